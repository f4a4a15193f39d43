// Device functions of the fusion (Suppl. A.1, A.2) shared by the plain
// kernels (tsdf.hip) and the batched persistent kernels (batch.hip): one
// definition, so both paths perform the identical operation sequence.
#pragma once

#include <climits>

#include "ggeom_internal.h"

namespace gg {

// depth bins: z_d = 1 / (1/z_near - d du)
__device__ __forceinline__ float bin_depth(int d, int D, float z_near, float z_far) {
  const float un = 1.0f / z_near;
  const float uf = 1.0f / z_far;
  const float du = (un - uf) / (float)(D - 1);
  const float u = un - (float)d * du;
  return 1.0f / u;
}

// Entry d of the bin table: (z_d, tau_d), entries past D - 1 repeating it.
__host__ __device__ constexpr uint32_t padded_bins(int32_t D) { return ((uint32_t)D + 7u) & ~7u; }

__device__ __forceinline__ float2 bin_record(int d, int D, float z_near, float z_far, float trunc,
                                             int in_bins) {
  const float un = 1.0f / z_near;
  const float uf = 1.0f / z_far;
  const float du = (un - uf) / (float)(D - 1);
  const float z = bin_depth(d < D ? d : D - 1, D, z_near, z_far);
  return make_float2(z, in_bins ? (trunc * du) * (z * z) : trunc);
}

// ---------------------------------------------------------------------------
// fusion weight (Suppl. A.1)

constexpr int kConfTX = 32, kConfTY = 8, kMaxR = (GG_MAX_WINDOW - 1) / 2;
constexpr int kConfLW = kConfTX + 2 * kMaxR, kConfLH = kConfTY + 2 * kMaxR;
// the staged tile, then two floats per row of 16 lanes
constexpr int kConfRows = kConfTX * kConfTY / 16;
constexpr int kConfTileFloats = kConfLH * kConfLW + 2 * kConfRows;

// nu of Suppl. A.1 at pixel (i, j) with centre depth dq, reading the staged
// tile (origin at image (i0 - r, j0 - r)); row-major over the window.
__device__ __forceinline__ float window_nu(const float *tile, int li, int lj, int i, int j,
                                           float dq, const ConfArgs &a) {
  const int r = a.radius;
  float nu = 0.0f;
  for (int dy = -r; dy <= r; ++dy) {
    const int jj = j + dy;
    if (jj < 0 || jj >= a.Hs) continue;
    for (int dx = -r; dx <= r; ++dx) {
      const int ii = i + dx;
      if (ii < 0 || ii >= a.Ws) continue;
      const float dn = tile[(lj + dy) * kConfLW + (li + dx)];
      float term;
      if (depth_ok(dn)) {
        const float dd = dq - dn;
        term = fminf(dd * dd, a.tw2);
      } else {
        term = a.tw2;
      }
      nu = nu + term;
    }
  }
  return nu;
}

// nu for a pixel whose whole window lies inside the image (radius R known
// at compile time): the same terms in the same row-major order, with holes
// staged as NaN -- d_q - NaN is NaN and fminf(NaN, tau^2) = tau^2, which is
// exactly a hole's term -- so no test is needed per neighbour.
template <int R>
__device__ __forceinline__ float window_nu_interior(const float *tile, int li, int lj, float dq,
                                                    float tw2) {
  const float *w = tile + (lj - R) * kConfLW + (li - R);
  float nu = 0.0f;
#pragma unroll
  for (int dy = 0; dy <= 2 * R; ++dy)
#pragma unroll
    for (int dx = 0; dx <= 2 * R; ++dx) {
      const float dd = dq - w[dy * kConfLW + dx];
      nu = nu + fminf(dd * dd, tw2);
    }
  return nu;
}

__device__ __forceinline__ float window_nu_fast(const float *tile, int li, int lj, float dq,
                                                const ConfArgs &a) {
  switch (a.radius) {
    case 0: return window_nu_interior<0>(tile, li, lj, dq, a.tw2);
    case 1: return window_nu_interior<1>(tile, li, lj, dq, a.tw2);
    case 2: return window_nu_interior<2>(tile, li, lj, dq, a.tw2);
    case 3: return window_nu_interior<3>(tile, li, lj, dq, a.tw2);
    case 4: return window_nu_interior<4>(tile, li, lj, dq, a.tw2);
    case 5: return window_nu_interior<5>(tile, li, lj, dq, a.tw2);
    case 6: return window_nu_interior<6>(tile, li, lj, dq, a.tw2);
    default: return window_nu_interior<kMaxR>(tile, li, lj, dq, a.tw2);
  }
}

// The window's tile staged in LDS; pixels without a usable depth are staged
// as NaN (both window forms treat NaN as a hole), pixels outside the image
// as 0 (only the bounds-checked form can reach them, and it skips them).
// A staged row is at most 46 floats: one wavefront's lanes take its columns
// and the workgroup's wavefronts (blockDim a multiple of 64) step down the
// rows, so no lane divides by the row width.  kDepth: the source is a depth
// map, whose holes are staged as NaN; otherwise values are staged as read.
template <bool kDepth>
__device__ __forceinline__ void stage_rows(float *tile, const float *src, int i0, int j0,
                                           const ConfArgs &a) {
  static_assert(kConfTX + 2 * kMaxR <= 64, "a staged row fits one wavefront");
  const int r = a.radius;
  const int tw = kConfTX + 2 * r, th = kConfTY + 2 * r;
  const int lx = (int)(threadIdx.x & 63u), waves = (int)(blockDim.x >> 6);
  const int gi = i0 - r + lx;
  const bool in_col = gi >= 0 && gi < a.Ws;
  // stored at (ly + kMaxR - r, lx + kMaxR - r) so that window offsets are
  // relative to the fixed centre origin
  float *dst = tile + (kMaxR - r) * kConfLW + (lx + kMaxR - r);
  if (lx < tw) {
    for (int ly = (int)(threadIdx.x >> 6); ly < th; ly += waves) {
      const int gj = j0 - r + ly;
      float v = 0.0f;
      if (in_col && gj >= 0 && gj < a.Hs) {
        v = gmem(src)[(size_t)gj * a.Ws + gi];
        if (kDepth && !depth_ok(v)) v = __builtin_nanf("");
      }
      dst[ly * kConfLW] = v;
    }
  }
}

__device__ __forceinline__ void stage_tile(float *tile, const float *dk, int i0, int j0,
                                           const ConfArgs &a) {
  stage_rows<true>(tile, dk, i0, j0, a);
}

// The largest value of each row of 16 lanes, in all of them (lane swizzles of
// the vector unit: by 1, by 2, mirrored in 8, mirrored in 16).
template <int kCtrl>
__device__ __forceinline__ float row_swizzle(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kCtrl, 0xf, 0xf, true));
}
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, row_swizzle<0xb1>(v));    // quad: lanes 1 0 3 2
  v = fmaxf(v, row_swizzle<0x4e>(v));    // quad: lanes 2 3 0 1
  v = fmaxf(v, row_swizzle<0x141>(v));   // half-row mirror
  return fmaxf(v, row_swizzle<0x140>(v));  // row mirror
}

// Start value of word i of ConfArgs::cells.
__device__ __forceinline__ uint32_t cell_start(uint32_t i, uint32_t ncells) {
  return i < ncells ? 0u : 0x7f800000u;
}

// The tile's largest and least usable depth into every 3 x 3 window of cells
// that holds the tile's cell (float bits of non-negative values order as
// integers).  A tile lies in one cell: tiles are kCell wide and divide it in
// height.  d: the thread's depth, 0 if it has none.
__device__ __forceinline__ void cell_range(const ConfArgs &a, int k, int i0, int j0, float d,
                                           float *red) {
  static_assert(kConfTX == kCell && kCell % kConfTY == 0, "a tile lies in one cell");
  const float hi = row_max(d), lo = -row_max(d > 0.0f ? -d : -INFINITY);
  if ((threadIdx.x & 15u) == 0) {
    red[threadIdx.x >> 4] = hi;
    red[kConfRows + (threadIdx.x >> 4)] = lo;
  }
  __syncthreads();
  const int t = (int)threadIdx.x, cx = i0 / kCell - t % 3, cy = j0 / kCell - t / 3;
  if (t < 9 && cx >= 0 && cy >= 0) {
    float hi = red[0], lo = red[kConfRows];
#pragma unroll
    for (int w = 1; w < kConfRows; ++w) {
      hi = fmaxf(hi, red[w]);
      lo = fminf(lo, red[kConfRows + w]);
    }
    const uint32_t c = ((uint32_t)k * cells_across(a.Hs) + (uint32_t)cy) * cells_across(a.Ws) +
                       (uint32_t)cx;
    if (hi > 0.0f) {
      __hip_atomic_fetch_max(gmem(a.cells) + c, __float_as_uint(hi), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_fetch_min(gmem(a.cells) + a.ncells + c, __float_as_uint(lo), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// One 32 x 8 tile (bx, by) of view k; tile: LDS of kConfTileFloats floats.
__device__ __forceinline__ void conf_tile(const ConfArgs &a, int k, int bx, int by, float *tile) {
  const int i0 = bx * kConfTX, j0 = by * kConfTY;
  const float *dk = a.depth + (size_t)k * a.Ws * a.Hs;
  stage_tile(tile, dk, i0, j0, a);
  __syncthreads();
  const int lx = threadIdx.x & (kConfTX - 1), ly = threadIdx.x / kConfTX;
  const int i = i0 + lx, j = j0 + ly;
  // every window of the tile inside the image: the unchecked form
  const bool interior = i0 >= a.radius && j0 >= a.radius &&
                        i0 + kConfTX + a.radius <= a.Ws && j0 + kConfTY + a.radius <= a.Hs;
  float dusable = 0.0f;
  if (ly < kConfTY && i < a.Ws && j < a.Hs) {
    const int li = lx + kMaxR, lj = ly + kMaxR;
    const float dq = tile[lj * kConfLW + li];
    float2 rec = make_float2(-INFINITY, 0.0f);
    if (depth_ok(dq)) {
      const float nu = interior ? window_nu_fast(tile, li, lj, dq, a)
                                : window_nu(tile, li, lj, i, j, dq, a);
      const float om = (nu == 0.0f) ? 1.0f : fminf(a.scale / sqrtf(nu / a.n2), 1.0f);
      rec = make_float2(dq, om);
      dusable = dq;
    }
    float2 *row = a.table + (size_t)k * table_view_records(a.Ws, a.Hs) + (size_t)j * table_pitch(a.Ws);
    gstore2(row + i, rec);
    if (i == a.Ws - 1) gstore2(row + a.Ws, make_float2(0.0f, 0.0f));  // the row's closing record
  }
  if (a.cells) cell_range(a, k, i0, j0, dusable, tile + kConfLH * kConfLW);
}

// Fusion tile at position s of the launch's visiting order.  Far source
// views see a target ray as a long epipolar segment spanning many source
// rows, so one target row gathers from a large part of each view table;
// the rows below it gather from nearly the same lines.  Visiting vertical
// bands of band_B tiles across, each row by row from the top, keeps the
// lines that the tiles in flight share within cache, where row-major order
// would have walked the whole target width before returning to them.
// Every full band comes before the narrower last one (band_T = 0:
// row-major order).
__host__ __device__ __forceinline__ uint32_t band_tile(const IntegrateArgs &a, uint32_t s) {
  if (a.band_T == 0) return s;
  const uint32_t span = a.band_B * a.band_H;  // tiles of a full band
  const uint32_t b = s / span;
  const uint32_t b0 = b * a.band_B;
  const uint32_t w = a.band_T - b0 < a.band_B ? a.band_T - b0 : a.band_B;
  const uint32_t rem = s - b * span;
  const uint32_t r = rem / w;
  return r * a.band_T + b0 + (rem - r * w);
}

// ---------------------------------------------------------------------------
// sampling of a view table

// How the samples find their pixels.  The pixel of the point (X0, X1, Z)
// (homogeneous pixel coordinates) is (floor(X0 / Z), floor(X1 / Z)) with the
// quotient evaluated as X * (1 / Z), none if Z <= 0 or outside the image.
// 1 / Z is correctly rounded in every mode: by recip_rn where it is exact
// (2^-100 < Z < 2^100; the upper end is checked on the host), by IEEE division
// where a depth may lie in (0, 2^-100].
enum : int {
  kChecked = 0,  // no sample has Z in (0, 2^-100]: recip_rn, Z tested
  kDivide = 1,   // IEEE division
};

// Byte offset of the sample's view-table record within the view's table
// (rows of `pitch` records), kOutOfRange if none.
template <int kMode>
__device__ __forceinline__ uint32_t sample_offset(float X0, float X1, float Z, uint32_t Ws,
                                                  uint32_t Hs, uint32_t pitch, float fWs,
                                                  float fHs) {
  if constexpr (kMode == kDivide) {
    uint32_t off = kOutOfRange;
    if (Z > 0.0f) {
      const float iv = 1.0f / Z;
      const float u = X0 * iv, w = X1 * iv;
      if (u >= 0.0f && u < fWs && w >= 0.0f && w < fHs)
        off = ((uint32_t)w * pitch + (uint32_t)u) << 3;
    }
    return off;
  } else {
    const float inv = recip_rn(Z);
    const uint32_t i = (uint32_t)floor_i32(X0 * inv), j = (uint32_t)floor_i32(X1 * inv);
    const bool ok = i < Ws && j < Hs && Z > kRecipLo;
    // sizes are at most 16384 (host check): pitch * 8 < 2^24, the offset < 2^31
    return ok ? __umul24(j, pitch << 3) + (i << 3) : kOutOfRange;
  }
}

}  // namespace gg
