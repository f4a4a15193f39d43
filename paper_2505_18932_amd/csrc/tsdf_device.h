// Device functions of the fusion (Suppl. A.1, A.2) shared by the plain
// kernels (tsdf.hip) and the batched kernels (batch.hip): one definition, so
// both paths perform the identical operation sequence.
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

// Keeps the loads on their side of this point of the program.
__device__ __forceinline__ void schedule_fence() { __builtin_amdgcn_sched_barrier(0); }

// A tile of the window kernels: 32 x 8 kRows pixels, thread (x, y) of 32 x 8
// with the kRows pixels from row kRows y down.
constexpr int kConfTX = 32, kConfTY = 8, kMaxR = (GG_MAX_WINDOW - 1) / 2;
constexpr int kConfLW = kConfTX + 2 * kMaxR;
constexpr int conf_lds(int rows) { return (kConfTY * rows + 2 * kMaxR) * kConfLW; }  // floats
// the staged tile, then two floats per row of 16 lanes
constexpr int kConfRows = kConfTX * kConfTY / 16;
constexpr int conf_tile_floats(int rows) { return conf_lds(rows) + 2 * kConfRows; }

// nu of Suppl. A.1 (window radius R) of kRows pixels one below the other,
// centre depths dq, the first at (li, lj) of the staged tile; each pixel's
// terms in row-major order.  A staged row is read once for all the pixels
// whose window it crosses.  Holes are staged as NaN -- dq - NaN is NaN and
// fminf(NaN, tau^2) = tau^2, exactly a hole's term -- and pixels outside the
// image as -1: kEdge drops their terms (+0 changes no sum); a tile whose
// windows all lie inside the image has none.
template <int R, int kRows, bool kEdge>
__device__ __forceinline__ void window_rows(const float *tile, int li, int lj,
                                            const float (&dq)[kRows], float tw2,
                                            float (&nu)[kRows]) {
  const float *w = tile + (lj - R) * kConfLW + (li - R);
#pragma unroll
  for (int r = 0; r < kRows; ++r) nu[r] = 0.0f;
#pragma unroll
  for (int y = 0; y < kRows + 2 * R; ++y) {
    float dn[2 * R + 1];
#pragma unroll
    for (int dx = 0; dx <= 2 * R; ++dx) dn[dx] = w[y * kConfLW + dx];
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      if (y < r || y > r + 2 * R) continue;
#pragma unroll
      for (int dx = 0; dx <= 2 * R; ++dx) {
        const float dd = dq[r] - dn[dx];
        const float term = fminf(dd * dd, tw2);
        nu[r] = nu[r] + (kEdge && dn[dx] < 0.0f ? 0.0f : term);
      }
    }
  }
}

template <int R, int kRows>
__device__ __forceinline__ void window_nu_r(const float *tile, bool edge, int li, int lj,
                                            const float (&dq)[kRows], float tw2,
                                            float (&nu)[kRows]) {
  if constexpr (R <= 3) {
    if (edge)
      window_rows<R, kRows, true>(tile, li, lj, dq, tw2, nu);
    else
      window_rows<R, kRows, false>(tile, li, lj, dq, tw2, nu);
  } else {  // a pixel at a time: the code of the larger windows stays within the cache
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      const float d[1] = {dq[r]};
      float n[1];
      if (edge)
        window_rows<R, 1, true>(tile, li, lj + r, d, tw2, n);
      else
        window_rows<R, 1, false>(tile, li, lj + r, d, tw2, n);
      nu[r] = n[0];
    }
  }
}

template <int kRows>
__device__ __forceinline__ void window_nu(const float *tile, bool edge, int li, int lj,
                                          const float (&dq)[kRows], const ConfArgs &a,
                                          float (&nu)[kRows]) {
  switch (a.radius) {
    case 0: return window_nu_r<0>(tile, edge, li, lj, dq, a.tw2, nu);
    case 1: return window_nu_r<1>(tile, edge, li, lj, dq, a.tw2, nu);
    case 2: return window_nu_r<2>(tile, edge, li, lj, dq, a.tw2, nu);
    case 3: return window_nu_r<3>(tile, edge, li, lj, dq, a.tw2, nu);
    case 4: return window_nu_r<4>(tile, edge, li, lj, dq, a.tw2, nu);
    case 5: return window_nu_r<5>(tile, edge, li, lj, dq, a.tw2, nu);
    case 6: return window_nu_r<6>(tile, edge, li, lj, dq, a.tw2, nu);
    default: return window_nu_r<kMaxR>(tile, edge, li, lj, dq, a.tw2, nu);
  }
}

// Whether a tile's windows reach past the image.
template <int kRows>
__device__ __forceinline__ bool tile_at_edge(const ConfArgs &a, int i0, int j0) {
  return i0 < a.radius || j0 < a.radius || i0 + kConfTX + a.radius > a.Ws ||
         j0 + kConfTY * kRows + a.radius > a.Hs;
}

// The windows of a tile staged in LDS.  A depth map's pixels without a usable
// depth are staged as NaN, places outside the image as -1 (kDepths) or NaN as
// well (kNeighbours); of another map twice the value, and 0.  A staged row
// is at most 46 floats: one wavefront's lanes take its columns and the
// workgroup's four wavefronts step down the rows, so no lane divides by the
// row width; four or five rows' loads are in flight together.
enum : int { kDepths, kNeighbours, kTwice };
template <int kWhat, int kRows>
__device__ __forceinline__ void stage_rows(float *tile, const float *src, int i0, int j0,
                                           const ConfArgs &a) {
  static_assert(kConfTX + 2 * kMaxR <= 64, "a staged row fits one wavefront");
  constexpr int kBatch = kRows == 1 ? 4 : 5;
  const int r = a.radius;
  const int tw = kConfTX + 2 * r, th = kConfTY * kRows + 2 * r;
  const int lx = (int)(threadIdx.x & 63u);
  const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gi = i0 - r + lx;
  const bool in_col = lx < tw && gi >= 0 && gi < a.Ws;
  // at most 16384 x 16384 pixels (host check)
  const auto image = buffer_of(src, (uint32_t)a.Ws * (uint32_t)a.Hs * 4u);
  // stored at (ly + kMaxR - r, lx + kMaxR - r) so that window offsets are
  // relative to the fixed centre origin
  float *dst = tile + (kMaxR - r) * kConfLW + (lx + kMaxR - r);
  for (int y0 = wave; y0 < th; y0 += 4 * kBatch) {
    float v[kBatch];
#pragma unroll
    for (int n = 0; n < kBatch; ++n) {
      const int gj = j0 - r + y0 + 4 * n;
      const bool in = in_col && gj >= 0 && gj < a.Hs;
      v[n] = bload1(image, in ? ((uint32_t)gj * (uint32_t)a.Ws + (uint32_t)gi) * 4u : kOutOfRange);
      if (kWhat == kTwice)
        v[n] = v[n] * 2.0f;
      else if (!depth_ok(v[n]))
        v[n] = __builtin_nanf("");
      if (kWhat == kDepths && !in) v[n] = -1.0f;
    }
    if (lx < tw) {
#pragma unroll
      for (int n = 0; n < kBatch; ++n)
        if (y0 + 4 * n < th) dst[(y0 + 4 * n) * kConfLW] = v[n];
    }
  }
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

// Start value of word i of ConfArgs::cells: the empty range.
__device__ __forceinline__ uint32_t cell_start(uint32_t i, uint32_t ncells) {
  return i < ncells ? 0u : 0x7f800000u;
}

// The record that closes each row of a view table: no weight, so its depth changes no sum (0 times
// a finite clamp) and says whether the cells' ranges were formed with the table.  A fusion may be
// given a table that another call built without them, and a workspace long enough to hold them:
// it must not read what nothing wrote.
__device__ __forceinline__ float2 closing_record(bool ranges) {
  return make_float2(ranges ? 1.0f : 0.0f, 0.0f);
}

// The tile's largest and least usable depth into every 3 x 3 window of cells
// that holds the tile's cell (float bits of non-negative values order as
// integers).  A tile lies in one cell: tiles are kCell wide and divide it in
// height.  The thread's largest depth, 0 if it has none, and its least, inf.
__device__ __forceinline__ void cell_range(const ConfArgs &a, int k, int i0, int j0, float dmax,
                                           float dmin, float *red) {
  const float hi = row_max(dmax), lo = -row_max(-dmin);
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

// One 32 x 8 kRows tile (bx, by) of view k; tile: LDS of conf_tile_floats(kRows) floats.
template <int kRows>
__device__ __forceinline__ void conf_tile(const ConfArgs &a, int k, int bx, int by, float *tile) {
  static_assert(kConfTX == kCell && kCell % (kConfTY * kRows) == 0, "a tile lies in one cell");
  const int i0 = bx * kConfTX, j0 = by * kConfTY * kRows;
  stage_rows<kDepths, kRows>(tile, a.depth + (size_t)k * a.Ws * a.Hs, i0, j0, a);
  __syncthreads();
  const int lx = threadIdx.x & (kConfTX - 1), ly = threadIdx.x / kConfTX * kRows;
  const int i = i0 + lx, j = j0 + ly;
  const int li = lx + kMaxR, lj = ly + kMaxR;
  float dq[kRows], nu[kRows], dmax = 0.0f, dmin = INFINITY;
#pragma unroll
  for (int r = 0; r < kRows; ++r) dq[r] = tile[(lj + r) * kConfLW + li];
  window_nu<kRows>(tile, tile_at_edge<kRows>(a, i0, j0), li, lj, dq, a, nu);
  float2 *row = a.table + (size_t)k * table_view_records(a.Ws, a.Hs) + (size_t)j * table_pitch(a.Ws);
#pragma unroll
  for (int r = 0; r < kRows; ++r, row += table_pitch(a.Ws)) {
    if (i >= a.Ws || j + r >= a.Hs) continue;
    float2 rec = make_float2(-INFINITY, 0.0f);
    if (depth_ok(dq[r])) {
      const float om = (nu[r] == 0.0f) ? 1.0f : fminf(a.scale / sqrtf(nu[r] / a.n2), 1.0f);
      rec = make_float2(dq[r], om);
      dmax = fmaxf(dmax, dq[r]);
      dmin = fminf(dmin, dq[r]);
    }
    gstore2(row + i, rec);
    if (i == a.Ws - 1) gstore2(row + a.Ws, closing_record(a.cells != nullptr));
  }
  if (a.cells) cell_range(a, k, i0, j0, dmax, dmin, tile + conf_lds(kRows));
}

// Fusion tile at position s of the launch's visiting order.  Far source
// views see a target ray as a long epipolar segment spanning many source
// rows, so one target row gathers from a large part of each view table;
// the rows below it gather from nearly the same lines.  Visiting vertical
// bands of band_B tiles across, each row by row from the top, keeps the
// lines that the tiles in flight share within cache, where row-major order
// would have walked the whole target width before returning to them.
// band_N full bands come before the narrower last one (band_B = 0: row-major
// order).  A row's tiles of a band are those that start in it: of a full band
// always band_B, of the last, wl columns wide, ceil(r wl / 64) in the rows
// before row r, whether or not whole tiles make up a row (1529 x 1031 K=8 D=36
// carried: row-major 912 us, in bands 690).
__host__ __device__ __forceinline__ uint32_t band_tile(const IntegrateArgs &a, uint32_t s) {
  if (a.band_B == 0) return s;
  const uint32_t w = a.wt_div.d, across = a.band_B * kFusePix, span = a.band_B * a.band_H;
  uint32_t b = s / span;
  if (b > a.band_N) b = a.band_N;
  const uint32_t m = s - b * span, wl = b < a.band_N ? across : w - a.band_N * across;
  const uint32_t r = kFusePix * m / wl;
  return (r * w + b * across + kFusePix - 1) / kFusePix + m - (r * wl + kFusePix - 1) / kFusePix;
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
