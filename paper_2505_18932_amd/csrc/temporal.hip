// Colour-difference masks between consecutive frames (Eq. 1, §3.2) and the
// temporally filtered depth (Eq. 2).  Three streaming passes per call:
//   1. one thread per low-resolution pixel: the factor x factor box sums of
//      both frames (exact integers), the channel mean of |I - I'| and the
//      clamped mask;
//   2. one thread per low-resolution pixel: the 3 x 3 maximum;
//   3. one thread per four full-resolution pixels (one where four are not
//      aligned): bilinear upsampling, and the depth filter fused in (one read
//      of D and of the previous filtered depth, one write of each output).
// The low-resolution planes (1/16 of a frame) stay in L2 between passes.
// Bound by latency and instructions, not bytes (4 x 1280 x 720, factor 4: 42 us
// with a pixel per thread, 64-bit index divisions and byte loads, 25 with four
// pixels per thread, a grid without divisions and word loads; the bytes take 16).
// Every step follows the FP32 operation order stated in the header, so the
// outputs are bitwise those of that definition.
#include "ggeom_internal.h"

namespace gg {

// Workgroups of 64 x 4 threads over one view: a row of low-resolution pixels
// or of groups of four full-resolution ones per wavefront, no index division.
constexpr int kMaskX = 64, kMaskY = 4;

// kWords: the factor and the width are multiples of 4 and the frames 4-byte
// aligned, so that a box's rows are whole words (a third of the loads of
// single bytes a third as wide).
template <bool kWords>
__global__ __launch_bounds__(256) void mask_low_kernel(MaskArgs a) {
  const int aa = (int)(blockIdx.x * kMaskX + (threadIdx.x & 63u));
  const int b = (int)(blockIdx.y * kMaskY + (threadIdx.x >> 6)), k = (int)blockIdx.z;
  if (aa >= a.Wq || b >= a.Hq) return;
  const int j0 = b * a.factor, i0 = aa * a.factor;
  const int j1 = min(j0 + a.factor, a.H), i1 = min(i0 + a.factor, a.W);
  const GG_GLOBAL uint8_t *f0 = gmem(a.rgb) + (size_t)k * a.W * a.H * 3;
  const GG_GLOBAL uint8_t *f1 = gmem(a.rgb_prev) + (size_t)k * a.W * a.H * 3;
  int st[3] = {0, 0, 0}, sp[3] = {0, 0, 0};
  if constexpr (kWords) {
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
      const size_t row = ((size_t)j * a.W + i0) * 3;
      const GG_GLOBAL uint32_t *w0 = (const GG_GLOBAL uint32_t *)(f0 + row);
      const GG_GLOBAL uint32_t *w1 = (const GG_GLOBAL uint32_t *)(f1 + row);
      for (int q = 0; q < (i1 - i0) / 4; ++q) {  // four pixels
        const uint32_t x[3] = {w0[3 * q], w0[3 * q + 1], w0[3 * q + 2]};
        const uint32_t y[3] = {w1[3 * q], w1[3 * q + 1], w1[3 * q + 2]};
#pragma unroll
        for (int c = 0; c < 12; ++c) {
          st[c % 3] += (int)((x[c / 4] >> (8 * (c % 4))) & 255u);
          sp[c % 3] += (int)((y[c / 4] >> (8 * (c % 4))) & 255u);
        }
      }
    }
  } else {
    for (int j = j0; j < j1; ++j) {
      const size_t row = ((size_t)j * a.W) * 3;
      for (int i = i0 * 3; i < i1 * 3; i += 3) {
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
          st[ch] += f0[row + i + ch];
          sp[ch] += f1[row + i + ch];
        }
      }
    }
  }
  const int cnt = (j1 - j0) * (i1 - i0);
  const int d = abs(st[0] - sp[0]) + abs(st[1] - sp[1]) + abs(st[2] - sp[2]);
  const float dI = (float)d / (float)(765 * cnt);
  const float tq = dI / a.lambda_t;
  gmem(a.low)[((size_t)k * a.Hq + b) * a.Wq + aa] = fminf(tq + a.beta, 1.0f);
}

__global__ __launch_bounds__(256) void mask_pool_kernel(MaskArgs a) {
  const int aa = (int)(blockIdx.x * kMaskX + (threadIdx.x & 63u));
  const int b = (int)(blockIdx.y * kMaskY + (threadIdx.x >> 6)), k = (int)blockIdx.z;
  if (aa >= a.Wq || b >= a.Hq) return;
  const GG_GLOBAL float *low = gmem(a.low) + (size_t)k * a.Wq * a.Hq;
  // rows and columns past the plane repeat its own: no bounds in the maximum
  const int x0 = max(aa - 1, 0), x1 = min(aa + 1, a.Wq - 1);
  float m = 0.0f;
#pragma unroll
  for (int dy = -1; dy <= 1; ++dy) {
    const GG_GLOBAL float *row = low + (size_t)min(max(b + dy, 0), a.Hq - 1) * a.Wq;
    const float r = fmaxf(fmaxf(row[x0], row[aa]), row[x1]);
    m = dy < 0 ? r : fmaxf(m, r);
  }
  gmem(a.pool)[((size_t)k * a.Hq + b) * a.Wq + aa] = m;
}

// kPer pixels of a row per thread: four by 16-byte accesses (the width a
// multiple of 4, the planes aligned), else one, so that a wavefront's single
// floats are neighbours (measured, 4 x 1283 x 721 factor 4: 36 us with four
// single floats per thread, 30 with one).  kWide: of four pixels at a factor
// of at least 4 the low-resolution columns are three neighbours, loaded once.
// (i + 0.5) / factor is the product with 1 / factor, exact, for a power of two.
template <bool kWide, int kPer>
__global__ __launch_bounds__(256) void mask_up_kernel(MaskArgs a) {
  const int i0 = kPer * (int)(blockIdx.x * kMaskX + (threadIdx.x & 63u));
  const int j = (int)(blockIdx.y * kMaskY + (threadIdx.x >> 6)), k = (int)blockIdx.z;
  if (i0 >= a.W || j >= a.H) return;
  const float fac = (float)a.factor, xmax = (float)(a.Wq - 1), ymax = (float)(a.Hq - 1);
  const bool pow2 = (a.factor & (a.factor - 1)) == 0;
  const float inv = 1.0f / fac;
  const size_t o = ((size_t)k * a.H + j) * a.W + i0;
  float D[kPer] = {}, pv[kPer] = {};
  if (a.depth) {
    if constexpr (kPer == 4) {
      const gg_v4f d = *(const GG_GLOBAL gg_v4f *)(a.depth + o);
      D[0] = d.x; D[1] = d.y; D[2] = d.z; D[3] = d.w;
      if (a.prev) {
        const gg_v4f p = *(const GG_GLOBAL gg_v4f *)(a.prev + o);
        pv[0] = p.x; pv[1] = p.y; pv[2] = p.z; pv[3] = p.w;
      }
    } else {
      D[0] = gmem(a.depth)[o];
      if (a.prev) pv[0] = gmem(a.prev)[o];
    }
  }
  auto low = [&](int i, float most) {  // the low-resolution coordinate
    const float q = (float)i + 0.5f;
    const float x = (pow2 ? q * inv : q / fac) - 0.5f;
    return x < 0.0f ? 0.0f : (x > most ? most : x);
  };
  const float y = low(j, ymax);
  const int y0 = (int)floorf(y), y1 = min(y0 + 1, a.Hq - 1);
  const float fy = y - (float)y0;
  const GG_GLOBAL float *p0 = gmem(a.pool) + ((size_t)k * a.Hq + y0) * a.Wq;
  const GG_GLOBAL float *p1 = gmem(a.pool) + ((size_t)k * a.Hq + y1) * a.Wq;
  const int first = (int)floorf(low(i0, xmax));
  float t[3], u[3];  // the three columns from `first`, of both rows
  if constexpr (kWide) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      t[c] = p0[min(first + c, a.Wq - 1)];
      u[c] = p1[min(first + c, a.Wq - 1)];
    }
  }
  float M[kPer], out[kPer];
#pragma unroll
  for (int v = 0; v < kPer; ++v) {
    const float x = low(i0 + v, xmax);
    const int x0 = (int)floorf(x), x1 = min(x0 + 1, a.Wq - 1);
    const float fx = x - (float)x0;
    const bool next = kWide && x0 > first;
    const float m00 = kWide ? (next ? t[1] : t[0]) : p0[x0], m10 = kWide ? (next ? t[2] : t[1]) : p0[x1];
    const float m01 = kWide ? (next ? u[1] : u[0]) : p1[x0], m11 = kWide ? (next ? u[2] : u[1]) : p1[x1];
    const float top = m00 + fx * (m10 - m00);
    const float bot = m01 + fx * (m11 - m01);
    M[v] = top + fy * (bot - top);
    out[v] = 0.0f;
    if (depth_ok(D[v]))
      out[v] = (pv[v] > 0.0f && pv[v] < INFINITY) ? fmaf(M[v], D[v], (1.0f - M[v]) * pv[v]) : D[v];
  }
  if constexpr (kPer == 4) {
    *(GG_GLOBAL gg_v4f *)(a.mask + o) = (gg_v4f){M[0], M[1], M[2], M[3]};
    if (a.depth) *(GG_GLOBAL gg_v4f *)(a.filtered + o) = (gg_v4f){out[0], out[1], out[2], out[3]};
  } else {
    gmem(a.mask)[o] = M[0];
    if (a.depth) gmem(a.filtered)[o] = out[0];
  }
}

int launch_difference_masks(const MaskArgs &a, hipStream_t s) {
  KernelTimer t("difference_masks", s);
  const auto grid = [&](int w, int h) {
    return dim3((w + kMaskX - 1) / kMaskX, (h + kMaskY - 1) / kMaskY, a.K);
  };
  const dim3 gq = grid(a.Wq, a.Hq), b(kMaskX * kMaskY);
  if (a.factor % 4 == 0 && a.W % 4 == 0 &&
      (((uintptr_t)a.rgb | (uintptr_t)a.rgb_prev) & 3u) == 0)
    hipLaunchKernelGGL(mask_low_kernel<true>, gq, b, 0, s, a);
  else
    hipLaunchKernelGGL(mask_low_kernel<false>, gq, b, 0, s, a);
  if (int rc = check_hip(hipGetLastError(), "mask_low_kernel")) return rc;
  hipLaunchKernelGGL(mask_pool_kernel, gq, b, 0, s, a);
  if (int rc = check_hip(hipGetLastError(), "mask_pool_kernel")) return rc;
  const bool vec = a.W % 4 == 0 && (((uintptr_t)a.depth | (uintptr_t)a.prev | (uintptr_t)a.mask |
                                     (uintptr_t)a.filtered) & 15u) == 0;
  void (*const up)(MaskArgs) = !vec ? mask_up_kernel<false, 1>
                               : a.factor >= 4 ? mask_up_kernel<true, 4> : mask_up_kernel<false, 4>;
  hipLaunchKernelGGL(up, grid(vec ? a.W / 4 : a.W, a.H), b, 0, s, a);
  return check_hip(hipGetLastError(), "mask_up_kernel");
}

}  // namespace gg
