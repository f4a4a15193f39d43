// Frustum-volume TSDF for gfx950: fusion weight map, depth bins, fused
// integrate + extraction, standalone extraction, adjoints.
//
// Paper passages: Suppl. A.1 (projection, signed distance, truncation,
// noise-aware weight, occlusion rule, sign change along the ray), Suppl. A.2
// (temporal weight), §3.2 (image-based TSDF guiding the target depth).
//
// Arithmetic is FP32 in a fixed operation order (no contraction; fused
// multiply-adds are explicit fmaf; divide and square root are correctly
// rounded) so that the volume and the extracted bins are bitwise
// reproducible and equal to the plain definition.
#include "fuse_device.h"

namespace gg {

// ---------------------------------------------------------------------------
// depth bins: z_d = 1 / (1/z_near - d du), tau_d = trunc du z_d^2 (in bins)

// (the last bin repeated to a multiple of kFuseBins, so that every chunk of
// the fusion reads whole), and the start values of the cells' depth ranges.

__global__ void bins_kernel(int32_t D, float z_near, float z_far, float trunc, int32_t in_bins,
                            float2 *out, uint32_t *cells, uint32_t ncells) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 2 * ncells) cells[i] = cell_start(i, ncells);
  if (i < padded_bins(D)) out[i] = bin_record((int)i, D, z_near, z_far, trunc, in_bins);
}

int launch_bins(const gg_tsdf_params &p, float2 *bins, uint32_t *cells, uint32_t ncells,
                hipStream_t s) {
  KernelTimer t("bins", s);
  const uint32_t n = 2 * ncells > padded_bins(p.num_bins) ? 2 * ncells : padded_bins(p.num_bins);
  hipLaunchKernelGGL(bins_kernel, dim3((n + 255) / 256), dim3(256), 0, s, p.num_bins,
                     p.z_near, p.z_far, p.trunc, p.trunc_in_bins, bins, cells, ncells);
  return check_hip(hipGetLastError(), "bins_kernel");
}

// ---------------------------------------------------------------------------
// fusion weight (Suppl. A.1): one workgroup per 32 x 8 kRows pixels of one
// view, the tile plus its halo staged in LDS by coalesced row loads.  Output:
// the view table (usable depth, or -inf for a hole so that the occlusion test
// drops it; omega), one 8-byte record per pixel, gathered by the fusion.
// Bound by the vector unit: four operations per term, 49 terms at the default
// window.  Four pixels per thread read a staged row once for up to four
// windows, and the halo is 1.4 of the tile against 2.1.  Tiles at the image's
// edge take the same unrolled windows.  Measured, before (one pixel per
// thread, loops with bounds checks at the edge) and after: 1920 x 1080 K=8 149
// and 97 us (one pixel per thread: 127), 960 x 540 K=8 42 and 33, 640 x 360
// K=4 18.3 and 14.6 (15.9), 333 x 200 K=4 11.5 and 9.7 (four: 10.1), 160 x 100
// K=1 10.8 and 7.5 (9.2).

template <int kRows>
__global__ __launch_bounds__(256) void conf_kernel(ConfArgs a) {
  __shared__ float tile[conf_tile_floats(kRows)];
  conf_tile<kRows>(a, blockIdx.z, blockIdx.x, blockIdx.y, tile);
}

template <int kRows>
static void launch_conf_rows(const ConfArgs &a, hipStream_t s) {
  const int ty = kConfTY * kRows;
  hipLaunchKernelGGL(conf_kernel<kRows>, dim3((a.Ws + kConfTX - 1) / kConfTX, (a.Hs + ty - 1) / ty,
                                              a.K),
                     dim3(kConfTX * kConfTY), 0, s, a);
}

int launch_conf(const ConfArgs &a, hipStream_t s) {
  KernelTimer t("conf", s);
  // one pixel per thread where four would leave the device too few workgroups
  if ((size_t)a.Ws * (size_t)a.Hs * (size_t)a.K >= 600000)
    launch_conf_rows<4>(a, s);
  else
    launch_conf_rows<1>(a, s);
  return check_hip(hipGetLastError(), "conf_kernel");
}

template <int kForm>
__global__ __launch_bounds__(64 * kFuseMaxWaves, form_waves(kForm)) void integrate_kernel(IntegrateArgs args) {
  extern __shared__ __align__(16) float smem[];
  // the record is read in the argument segment (offset 0: the only argument)
  const FuseArgs a = (FuseArgs)__builtin_amdgcn_kernarg_segment_ptr();
  integrate_tile<kForm>(a, band_tile(args, xcd_tile(blockIdx.x, args.nblocks)), smem);
}

// Structured view-table loads take three vector instructions per sample less
// than range-checked raw ones; their resource's 14-bit stride holds rows of
// at most 2047 records.
int integrate_form(const IntegrateArgs &a) {
  auto al = [](const void *p) { return ((uintptr_t)p & 15u) == 0; };
  const bool vec = a.D % 4 == 0 && al(a.F) && al(a.W) && al(a.F_prev) && al(a.W_prev);
  const bool lines = vec && a.D % 32 == 0, carry = a.F_prev != nullptr;
  return (vec ? kFormVec : 0) | (lines ? kFormLines : 0) | (table_rows_ok(a.Ws) ? kFormRows : 0) |
         (carry ? kFormCarry : 0) |
         (!lines && !carry && fuse_windows(a.K, a.D, vec, a.npix) ? kFormWindows : 0);
}

template <int kForm>
static void launch_form(IntegrateArgs &a, int form, hipStream_t s) {
  if constexpr (kForm < kFuseForms) {
    if (form != kForm) return launch_form<kForm + 1>(a, form, s);
    if constexpr (form_exists(kForm)) {
      const FuseShape shape = fuse_shape(kForm, a.K, a.D, a.nblocks);
      a.row = shape.row;
      a.span = shape.span;
      hipLaunchKernelGGL(integrate_kernel<kForm>, dim3(a.nblocks), dim3(64 * shape.waves),
                         shape.lds, s, a);
    }
  }
}

int launch_integrate(IntegrateArgs &a, hipStream_t s) {
  KernelTimer t("integrate", s);
  launch_form<0>(a, integrate_form(a), s);
  return check_hip(hipGetLastError(), "integrate_kernel");
}

// ---------------------------------------------------------------------------
// standalone extraction.  Bound by the volume's bytes: a wavefront takes
// kGroups pixels per load, the lanes of a group one 128-byte line of their
// pixel's F, and walks the bins only until every pixel has its crossing; of W
// it reads the lines in which F changes sign.  The lines come kLines at a time
// for kPixels pixels per group: one by one where the volume is larger than the
// caches (the fewest bytes), four at once in small launches, whose time is the
// chain of loads (launch_extract).  Measured, before (all of F and W read) and
// after: 960 x 540 D=128 92 and 66 us, 637 x 359 D=75 72 and 26, 1280 x 720
// D=128 166 and 94 (F alone: 91 at the copy's rate), 333 x 200 D=100 13.8 and
// 11.7.

template <uint32_t kWide, int kAux = 0>
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, uint32_t off, float (&o)[kWide]) {
  if constexpr (kWide == 4) {
    const gg_v4f v = __builtin_bit_cast(gg_v4f, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kAux));
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
  } else if constexpr (kWide == 2) {
    const gg_v2f v = __builtin_bit_cast(gg_v2f, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, kAux));
    o[0] = v.x; o[1] = v.y;
  } else {
    o[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kAux));
  }
}

// kWide: floats per lane and load, 4 or 2 (D a multiple, the volume aligned to them) or 1.
// kLanes: lanes of a group, 32 / kWide (a line) or, where they hold all D bins, fewer.
// kW: when W is loaded.
enum : int {
  kWhereNeeded,  // where F changes sign: a second trip to memory, but few lines
  kWithF,        // the group holds all D bins, a fraction of a line or one: the trip costs more
  kStreamed,     // with F, both non-temporal
};
template <uint32_t kWide, uint32_t kLanes, uint32_t kPixels, uint32_t kLines, int kW>
__global__ __launch_bounds__(256) void extract_kernel(ExtractArgs a) {
  constexpr uint32_t kGroups = 64 / kLanes, kLine = kLanes * kWide;
  constexpr uint64_t kGroup = (1ull << kLanes) - 1;
  constexpr bool kBoth = kW != kWhereNeeded;
  constexpr int kAux = kW == kStreamed ? 2 : 0;
  const uint32_t lane = threadIdx.x & 63u, group = lane / kLanes, sub = lane % kLanes;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t p0 = (xcd_tile(blockIdx.x, gridDim.x) * 4u + wave) * (kGroups * kPixels);
  if (p0 >= a.npix) return;
  const uint32_t D = (uint32_t)a.D, np = min(a.npix - p0, kGroups * kPixels);
  const auto F = buffer_of(a.F + (size_t)p0 * D, np * D * 4u);
  const auto W = buffer_of(a.W + (size_t)p0 * D, np * D * 4u);
  float prev[kPixels], prevw[kPixels];  // F and W of the bin before the lines
  bool done[kPixels];
#pragma unroll
  for (uint32_t p = 0; p < kPixels; ++p) {
    prev[p] = prevw[p] = 0.0f;
    done[p] = p * kGroups + group >= np;
  }
  for (uint32_t d0 = 0; d0 < D; d0 += kLine * kLines) {
    float f[kPixels][kLines][kWide], left[kPixels][kLines];
    float w[kPixels][kLines][kWide], wl[kPixels][kLines][1];
#pragma unroll
    for (uint32_t p = 0; p < kPixels; ++p)
#pragma unroll
      for (uint32_t l = 0; l < kLines; ++l) {
        const uint32_t d = d0 + kLine * l + sub * kWide;
        const uint32_t off =
            !done[p] && d < D ? ((p * kGroups + group) * D + d) * 4u : kOutOfRange;
        bload<kWide, kAux>(F, off, f[p][l]);
        if constexpr (kBoth) bload<kWide, kAux>(W, off, w[p][l]);
      }
    // crossings of F between bins d - 1 and d: F of the first, and whether there is one
    bool cross[kPixels][kLines], any = false;
#pragma unroll
    for (uint32_t p = 0; p < kPixels; ++p)
#pragma unroll
      for (uint32_t l = 0; l < kLines; ++l) {
        const uint32_t d = d0 + kLine * l + sub * kWide;
        const float up = __shfl_up(f[p][l][kWide - 1], 1, kLanes);
        left[p][l] = sub == 0 ? prev[p] : up;
        prev[p] = __shfl(f[p][l][kWide - 1], kLanes - 1, kLanes);
        if constexpr (kBoth) {
          const float upw = __shfl_up(w[p][l][kWide - 1], 1, kLanes);
          wl[p][l][0] = sub == 0 ? prevw[p] : upw;
          prevw[p] = __shfl(w[p][l][kWide - 1], kLanes - 1, kLanes);
        }
        bool c = false;
#pragma unroll
        for (uint32_t v = 0; v < kWide; ++v)
          c = c | ((v ? f[p][l][v ? v - 1 : 0] : left[p][l]) > 0.0f && f[p][l][v] <= 0.0f);
        cross[p][l] = c & !done[p] & (d < D);
        any |= cross[p][l];
      }
    if (__builtin_amdgcn_ballot_w64(any) == 0) continue;
    // both bins observed?
    if constexpr (!kBoth) {
#pragma unroll
      for (uint32_t p = 0; p < kPixels; ++p)
#pragma unroll
        for (uint32_t l = 0; l < kLines; ++l) {
          const uint32_t d = d0 + kLine * l + sub * kWide;
          const uint32_t off = ((p * kGroups + group) * D + d) * 4u;
          bload<kWide>(W, cross[p][l] ? off : kOutOfRange, w[p][l]);
          bload<1>(W, cross[p][l] && d ? off - 4u : kOutOfRange, wl[p][l]);
        }
    }
    bool all = true;
#pragma unroll
    for (uint32_t p = 0; p < kPixels; ++p) {
#pragma unroll
      for (uint32_t l = 0; l < kLines; ++l) {
        int best = -1;
        float f0 = 1.0f, f1 = 0.0f;
#pragma unroll
        for (int v = (int)kWide - 1; v >= 0; --v) {
          const float g0 = v ? f[p][l][v ? v - 1 : 0] : left[p][l];
          const float w0 = v ? w[p][l][v ? v - 1 : 0] : wl[p][l][0];
          if (g0 > 0.0f && f[p][l][v] <= 0.0f && w0 > 0.0f && w[p][l][v] > 0.0f) {
            best = (int)(d0 + kLine * l + sub * kWide) + v - 1;
            f0 = g0;
            f1 = f[p][l][v];
          }
        }
        const bool hit = cross[p][l] && best >= 0 && !done[p];
        const uint64_t mask = (__builtin_amdgcn_ballot_w64(hit) >> (group * kLanes)) & kGroup;
        if (hit && sub == (uint32_t)__builtin_ctzll(mask)) {  // the pixel's first
          const uint32_t pix = p0 + p * kGroups + group;
          const float za = bin_depth(best, a.D, a.z_near, a.z_far);
          const float zb = bin_depth(best + 1, a.D, a.z_near, a.z_far);
          const float frac = f0 / (f0 - f1);
          gmem(a.out_depth)[pix] = za + (zb - za) * frac;
          gmem(a.out_bin)[pix] = best;
        }
        done[p] = done[p] || mask != 0;
      }
      all &= done[p];
    }
    if (__builtin_amdgcn_ballot_w64(!all) == 0) return;
  }
#pragma unroll
  for (uint32_t p = 0; p < kPixels; ++p)
    if (!done[p] && sub == 0) {
      gmem(a.out_depth)[p0 + p * kGroups + group] = 0.0f;
      gmem(a.out_bin)[p0 + p * kGroups + group] = -1;
    }
}

template <uint32_t kWide, uint32_t kLanes, uint32_t kPixels, uint32_t kLines, int kW>
static void launch_extract_form(const ExtractArgs &a, hipStream_t s) {
  const uint32_t per = 4u * (64u / kLanes) * kPixels;
  hipLaunchKernelGGL((extract_kernel<kWide, kLanes, kPixels, kLines, kW>),
                     dim3((a.npix + per - 1) / per), dim3(256), 0, s, a);
}

// Few bins: the fewest lanes, a power of two, that hold them.
template <uint32_t kWide, uint32_t kPixels, uint32_t kLanes>
static void launch_extract_few(const ExtractArgs &a, hipStream_t s) {
  constexpr uint32_t kHalf = kLanes / 2;
  if constexpr (kHalf * kWide >= 2)
    if ((uint32_t)a.D <= kHalf * kWide) return launch_extract_few<kWide, kPixels, kHalf>(a, s);
  launch_extract_form<kWide, kLanes, kPixels, 1, kWithF>(a, s);
}

// Up to 16 bins (32 by vector loads), groups of as many lanes as hold them (measured, whole lines
// of 8 or 32 lanes as for more bins, and this: 1280 x 720 D=3 58 and 11.1 us, D=4 22.7 and 6.6, D=8
// 24.0 and 12.6, D=14 60 and 22, D=24 33.4 and 28.9; 333 x 200 D=4 4.6 and 3.2), streamed where F
// and W exceed the 256 MB cache (1920 x 1080 D=24: 75 us, 67 streamed; 1280 x 720 D=24: 29.1 and
// 30.5).  Of more bins, small volumes take two or four lines at once (one line and this: 160 x 100
// D=48 4.7 and 3.9 us, D=255 11.7 and 7.0, 333 x 200 D=100 12.2 and 11.7; but 420 x 260 D=48 10.3
// and 12.7, 512 x 288 D=96 19.3 and 21.5, 1280 x 720 D=128 95 and 117).
int launch_extract(const ExtractArgs &a, hipStream_t s) {
  KernelTimer t("extract", s);
  const uintptr_t base = (uintptr_t)a.F | (uintptr_t)a.W;
  const bool vec = a.D % 4 == 0 && (base & 15u) == 0, vec2 = a.D % 2 == 0 && (base & 7u) == 0;
  const size_t voxels = (size_t)a.npix * (size_t)a.D;
  if (vec && a.D <= 16)
    launch_extract_few<4, 1, 4>(a, s);
  else if (vec && a.D <= 32)
    voxels > (size_t)32 << 20 ? launch_extract_form<4, 8, 2, 1, kStreamed>(a, s)
    : a.npix > 1u << 17       ? launch_extract_form<4, 8, 2, 1, kWithF>(a, s)
                              : launch_extract_form<4, 8, 1, 1, kWithF>(a, s);
  else if (vec2 && a.D <= 32)
    launch_extract_few<2, 2, 16>(a, s);
  else if (a.D <= 16)
    a.npix > 1u << 17 ? launch_extract_few<1, 4, 16>(a, s) : launch_extract_few<1, 2, 16>(a, s);
  else if (a.D > 64 && voxels <= (size_t)8 << 20)
    vec ? launch_extract_form<4, 8, 1, 4, kWhereNeeded>(a, s)
        : launch_extract_form<1, 32, 2, 4, kWhereNeeded>(a, s);
  else if (a.D > 32 && voxels <= (size_t)1 << 20)
    vec ? launch_extract_form<4, 8, 1, 2, kWhereNeeded>(a, s)
        : launch_extract_form<1, 32, 2, 2, kWhereNeeded>(a, s);
  else
    vec ? launch_extract_form<4, 8, 2, 1, kWhereNeeded>(a, s)
        : launch_extract_form<1, 32, 4, 1, kWhereNeeded>(a, s);
  return check_hip(hipGetLastError(), "extract_kernel");
}

// Adjoint of the interpolation z* = z_d + (z_{d+1} - z_d) F_d / (F_d - F_{d+1}).
__global__ void extract_backward_kernel(ExtractArgs a) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.npix) return;
  const int d = a.bin[p];
  float2 out = make_float2(0.0f, 0.0f);
  if (d >= 0 && d < a.D - 1) {
    const float f0 = a.F[(size_t)p * a.D + d], f1 = a.F[(size_t)p * a.D + d + 1];
    const float za = bin_depth(d, a.D, a.z_near, a.z_far);
    const float zb = bin_depth(d + 1, a.D, a.z_near, a.z_far);
    const float dz = zb - za, delta = f0 - f1, g = a.g_depth[p];
    out.x = g * ((-dz * f1) / (delta * delta));
    out.y = g * ((dz * f0) / (delta * delta));
  }
  reinterpret_cast<float2 *>(a.g_F2)[p] = out;
}

int launch_extract_backward(const ExtractArgs &a, hipStream_t s) {
  KernelTimer t("extract_backward", s);
  hipLaunchKernelGGL(extract_backward_kernel, dim3((a.npix + 255) / 256), dim3(256), 0, s, a);
  return check_hip(hipGetLastError(), "extract_backward_kernel");
}

// ---------------------------------------------------------------------------
// adjoint of the fusion.  (1) per pixel with a crossing, bound |contribution|
// of its two voxels' per-view terms from the voxels alone; (2) recompute the
// terms and scatter them into per-source-pixel 64-bit fixed-point
// accumulators scaled by that bound (integer addition is associative: the
// result does not depend on arrival order); (3) chain the weight gradient
// through nu of its window; (4) gather the window terms.

__global__ void zero_u64_kernel(unsigned long long *p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0ull;
}

// Calls f(k, q, dD, dw) for each view sample of voxel (pix, d) whose
// contribution is live, with dD = dL/dD_k[q] through the clamp and
// dw = dL/domega_k[q].
template <typename Fn>
__device__ __forceinline__ void voxel_adjoint(const TsdfBackArgs &a, uint32_t pix, int d, float gF,
                                              Fn f) {
  const uint32_t y = fdiv(pix, a.wt_div), x = pix - y * a.wt_div.d;
  const float px = (float)x + 0.5f, py = (float)y + 0.5f;
  const float2 b = a.bins[d];
  const float z = b.x, tau = b.y;
  const size_t o = (size_t)pix * a.D + d;
  const float Wn = a.W[o], Fv = a.F[o];
  const float fWs = (float)a.Ws, fHs = (float)a.Hs;
  for (int k = 0; k < a.K; ++k) {
    const Proj &P = a.views[k];
    float h0, h1, h2;
    ray_of(P, px, py, h0, h1, h2);
    const float X0 = fmaf(z, h0, P.c[0]), X1 = fmaf(z, h1, P.c[1]), Z = fmaf(z, h2, P.c[2]);
    if (!(Z > 0.0f)) continue;
    const float inv = 1.0f / Z;
    const float u = X0 * inv, w = X1 * inv;
    if (!(u >= 0.0f && u < fWs && w >= 0.0f && w < fHs)) continue;
    const uint32_t q = (uint32_t)w * (uint32_t)a.Ws + (uint32_t)u;
    const float2 e = a.table[(size_t)k * table_view_records(a.Ws, a.Hs) +
                             (size_t)(uint32_t)w * table_pitch(a.Ws) + (uint32_t)u];
    const float s = e.x - Z;
    if (s < -tau) continue;
    const float c = fminf(s, tau);
    const float dD = (s < tau) ? (gF * e.y) / Wn : 0.0f;
    const float dw = (gF * (c - Fv)) / Wn;
    f(k, q, dD, dw);
  }
}

// An upper bound on |dD| and |dw| over every view sample of the pixel's two
// voxels, from the voxel alone: the table weight is at most 1 and the clamp
// keeps |c| <= tau, so |dD| <= |gF| / W and |dw| <= |gF| (tau + |F|) / W.
// Rounding is monotone, so the bound evaluated in FP32 also bounds the
// FP32 terms voxel_adjoint computes.
__device__ __forceinline__ float voxel_bound(const TsdfBackArgs &a, uint32_t pix, int d,
                                             float gF) {
  const size_t o = (size_t)pix * a.D + d;
  const float Wn = gmem(a.W)[o], Fv = gmem(a.F)[o];
  const float tau = gload2(a.bins + d).y, ag = fabsf(gF);
  return fmaxf(ag / Wn, (ag * (tau + fabsf(Fv))) / Wn);
}

__global__ __launch_bounds__(256) void tsdf_bwd_max_kernel(TsdfBackArgs a) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  float m = 0.0f;
  if (p < a.npix) {
    const int d = gmem(a.bin)[p];
    if (d >= 0) {
      const float2 g = reinterpret_cast<const float2 *>(a.g_F2)[p];
      m = fmaxf(voxel_bound(a, p, d, g.x), voxel_bound(a, p, d + 1, g.y));
    }
  }
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  __shared__ float red[4];
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = red[0];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) r = fmaxf(r, red[i]);
    atomicMax(a.maxbits, __float_as_uint(r));  // non-negative floats order as integers
  }
}

// Fixed-point exponent: every accumulated sum stays below 2^61 in magnitude.
__device__ __forceinline__ int fixed_exponent(const TsdfBackArgs &a) {
  const float m = __uint_as_float(*a.maxbits);
  if (!(m > 0.0f)) return INT_MIN;
  int e;
  frexp((double)m * 2.0 * (double)a.npix, &e);
  return 61 - e;
}

__device__ __forceinline__ unsigned long long to_fixed(float v, int E) {
  return (unsigned long long)(long long)llrint(ldexp((double)v, E));
}

__global__ __launch_bounds__(256) void tsdf_bwd_scatter_kernel(TsdfBackArgs a) {
  const uint32_t p = blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= a.npix) return;
  const int d = a.bin[p];
  if (d < 0) return;
  const int E = fixed_exponent(a);
  if (E == INT_MIN) return;
  const float2 g = reinterpret_cast<const float2 *>(a.g_F2)[p];
  auto sc = [&](int k, uint32_t q, float dD, float dw) {
    const size_t i = (size_t)k * a.ns + q;
    if (dD != 0.0f) atomicAdd(&a.acc_D[i], to_fixed(dD, E));
    if (dw != 0.0f) atomicAdd(&a.acc_w[i], to_fixed(dw, E));
  };
  voxel_adjoint(a, p, d, g.x, sc);
  voxel_adjoint(a, p, d + 1, g.y, sc);
}

__device__ __forceinline__ float from_fixed(unsigned long long v, int E) {
  return (float)ldexp((double)(long long)v, -E);
}

// The window parameters of the backward as the confidence kernel's record,
// so both share the tile staging and the window statistic.
__device__ __forceinline__ ConfArgs conf_of(const TsdfBackArgs &a) {
  ConfArgs c{};
  c.depth = a.depth;
  c.Ws = a.Ws;
  c.Hs = a.Hs;
  c.K = a.K;
  c.radius = a.radius;
  c.tw2 = a.tw2;
  c.n2 = a.n2;
  c.scale = a.scale;
  return c;
}

// dL/dnu at each source pixel: dL/domega * domega/dnu where the min(., 1)
// of the weight is inactive and nu > 0.  nu is the confidence kernel's
// window statistic (same tile staging, same terms in the same order); one
// 32 x 8 tile of view blockIdx.z per workgroup.
__global__ __launch_bounds__(256) void tsdf_bwd_nu_kernel(TsdfBackArgs a) {
  __shared__ float tile[conf_lds(1)];
  const ConfArgs c = conf_of(a);
  const int k = blockIdx.z, i0 = blockIdx.x * kConfTX, j0 = blockIdx.y * kConfTY;
  stage_rows<kDepths, 1>(tile, a.depth + (size_t)k * a.ns, i0, j0, c);
  __syncthreads();
  const int lx = threadIdx.x & (kConfTX - 1), ly = threadIdx.x / kConfTX;
  const int i = i0 + lx, j = j0 + ly;
  const bool edge = tile_at_edge<1>(c, i0, j0);
  if (i >= a.Ws || j >= a.Hs) return;
  const size_t o = (size_t)k * a.ns + (size_t)j * a.Ws + i;
  const int E = fixed_exponent(a);
  float out = 0.0f;
  const float gw = (E == INT_MIN) ? 0.0f : from_fixed(gmem(a.acc_w)[o], E);
  const int li = lx + kMaxR, lj = ly + kMaxR;
  const float dq[1] = {tile[lj * kConfLW + li]};  // NaN for a hole
  if (gw != 0.0f && depth_ok(dq[0])) {
    float nu[1];
    window_nu<1>(tile, edge, li, lj, dq, c, nu);
    if (nu[0] > 0.0f) {
      const float raw = a.scale / sqrtf(nu[0] / a.n2);
      if (raw < 1.0f) out = gw * ((-0.5f * raw) / nu[0]);
    }
  }
  gmem(a.gnu)[o] = out;
}

// The window terms of g_depth_in for a pixel with a usable depth dr, in
// row-major order over the window without its centre: the pixel as the centre
// (g2 = 2 gnu of it) and as a neighbour of each n (2 gnu_n in gtile).  A
// hole's NaN, also staged outside the image, makes dd NaN and fails dd^2 <
// tau^2; terms that fail add +0, with no branch around them (measured, 1920 x
// 1080 K=8: 309 us with branches, 181 without).  -2 gnu_n (d_n - d_r) is
// added as 2 gnu_n (d_r - d_n), the same value.
template <int R>
__device__ __forceinline__ void finish_window_r(const float *tile, const float *gtile, int li,
                                                int lj, float dr, float g2, float tw2, float &g) {
  const int at = (lj - R) * kConfLW + (li - R);
#pragma unroll
  for (int y = 0; y <= 2 * R; ++y) {
    float dn[2 * R + 1], gn[2 * R + 1];
#pragma unroll
    for (int x = 0; x <= 2 * R; ++x) {
      dn[x] = tile[at + y * kConfLW + x];
      gn[x] = gtile[at + y * kConfLW + x];
    }
#pragma unroll
    for (int x = 0; x <= 2 * R; ++x) {
      if (y == R && x == R) continue;
      const float dd = dr - dn[x];
      const bool in = dd * dd < tw2;
      g += in ? g2 * dd : 0.0f;
      g += in ? gn[x] * dd : 0.0f;
    }
  }
}

__device__ __forceinline__ void finish_window(const float *tile, const float *gtile, int li,
                                              int lj, float dr, float g2, const TsdfBackArgs &a,
                                              float &g) {
  switch (a.radius) {
    case 0: return finish_window_r<0>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    case 1: return finish_window_r<1>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    case 2: return finish_window_r<2>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    case 3: return finish_window_r<3>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    case 4: return finish_window_r<4>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    case 5: return finish_window_r<5>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    case 6: return finish_window_r<6>(tile, gtile, li, lj, dr, g2, a.tw2, g);
    default: return finish_window_r<kMaxR>(tile, gtile, li, lj, dr, g2, a.tw2, g);
  }
}

__global__ __launch_bounds__(256) void tsdf_bwd_finish_kernel(TsdfBackArgs a) {
  __shared__ float tile[conf_lds(1)];
  __shared__ float gtile[conf_lds(1)];
  const ConfArgs c = conf_of(a);
  const int k = blockIdx.z, i0 = blockIdx.x * kConfTX, j0 = blockIdx.y * kConfTY;
  stage_rows<kNeighbours, 1>(tile, a.depth + (size_t)k * a.ns, i0, j0, c);
  stage_rows<kTwice, 1>(gtile, a.gnu + (size_t)k * a.ns, i0, j0, c);
  const int lx = threadIdx.x & (kConfTX - 1), ly = threadIdx.x / kConfTX;
  const int i = i0 + lx, j = j0 + ly, li = lx + kMaxR, lj = ly + kMaxR;
  const size_t o = (size_t)k * a.ns + (size_t)j * a.Ws + i;
  const bool in = i < a.Ws && j < a.Hs;
  const int E = fixed_exponent(a);
  const float g = in && E != INT_MIN ? from_fixed(gmem(a.acc_D)[o], E) : 0.0f;
  __syncthreads();
  const float dr = tile[lj * kConfLW + li];
  float sum = g;
  finish_window(tile, gtile, li, lj, dr, gtile[lj * kConfLW + li], a, sum);
  if (in) gmem(a.g_depth_in)[o] = depth_ok(dr) ? sum : g;
}

int launch_tsdf_backward(const TsdfBackArgs &a, hipStream_t s) {
  {
    KernelTimer t("tsdf_bwd_zero", s);
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1024), dim3(256), 0, s, a.acc_D,
                       (size_t)a.K * a.ns * 2 + 1);
    if (int rc = check_hip(hipGetLastError(), "zero_u64_kernel")) return rc;
  }
  const dim3 gp((a.npix + 255) / 256);
  {
    KernelTimer t("tsdf_bwd_max", s);
    hipLaunchKernelGGL(tsdf_bwd_max_kernel, gp, dim3(256), 0, s, a);
    if (int rc = check_hip(hipGetLastError(), "tsdf_bwd_max_kernel")) return rc;
  }
  {
    KernelTimer t("tsdf_bwd_scatter", s);
    hipLaunchKernelGGL(tsdf_bwd_scatter_kernel, gp, dim3(256), 0, s, a);
    if (int rc = check_hip(hipGetLastError(), "tsdf_bwd_scatter_kernel")) return rc;
  }
  const dim3 gt((a.Ws + kConfTX - 1) / kConfTX, (a.Hs + kConfTY - 1) / kConfTY, a.K);
  {
    KernelTimer t("tsdf_bwd_nu", s);
    hipLaunchKernelGGL(tsdf_bwd_nu_kernel, gt, dim3(kConfTX * kConfTY), 0, s, a);
    if (int rc = check_hip(hipGetLastError(), "tsdf_bwd_nu_kernel")) return rc;
  }
  KernelTimer t("tsdf_bwd_finish", s);
  hipLaunchKernelGGL(tsdf_bwd_finish_kernel, gt, dim3(kConfTX * kConfTY), 0, s, a);
  return check_hip(hipGetLastError(), "tsdf_bwd_finish_kernel");
}

// ---------------------------------------------------------------------------
// self-check of the fast reciprocal against IEEE division (test hook)

__global__ void recip_selftest_kernel(uint32_t e_lo, uint32_t n_exp,
                                      unsigned long long *mismatches) {
  const uint64_t n = (uint64_t)n_exp << 23;
  unsigned long long bad = 0;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t bits = ((e_lo + (uint32_t)(i >> 23)) << 23) | (uint32_t)(i & 0x7fffffu);
    const float z = __uint_as_float(bits);
    const float a = recip_rn(z);
    const float b = 1.0f / z;
    bad += (__float_as_uint(a) != __float_as_uint(b)) ? 1ull : 0ull;
  }
  for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off);
  if ((threadIdx.x & 63) == 0 && bad) atomicAdd(mismatches, bad);
}

__global__ void fast_recip_kernel(const float *in, float *out, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    out[i] = recip_pos(in[i]);
}

int launch_recip_selftest(uint32_t e_lo, uint32_t n_exp, unsigned long long *mismatches,
                          hipStream_t s) {
  hipLaunchKernelGGL(recip_selftest_kernel, dim3(2048), dim3(256), 0, s, e_lo, n_exp, mismatches);
  return check_hip(hipGetLastError(), "recip_selftest_kernel");
}

int launch_fast_recip(const float *in, float *out, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(fast_recip_kernel, dim3(1024), dim3(256), 0, s, in, out, n);
  return check_hip(hipGetLastError(), "fast_recip_kernel");
}

}  // namespace gg
