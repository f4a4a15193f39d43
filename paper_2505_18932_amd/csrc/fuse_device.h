// Fused integrate + extraction (Suppl. A.1, A.2): the device function shared
// by the plain kernel (tsdf.hip) and the batched kernel (batch.hip), so both
// paths perform the identical operation sequence.
//
// A workgroup is 64 consecutive target pixels and 1 to 16 wavefronts; it walks
// the depth bins in slabs of 8 bins per wavefront.  In a slab each wavefront
// takes one chunk of 8 bins for all 64 pixels: lane = pixel, so the chunk's
// depths and truncations are wave-uniform (scalar registers), one gather
// instruction reads a row of neighbouring source pixels at one depth, and the
// wavefront's samples of a view project into a small patch of that view's
// image, which one test (find_live) can find to hold nothing to keep, or to
// lie in free space.  The volume moves in the other layout: the workgroup
// streams each pixel's run of the slab's bins (whole 128-byte lines with four
// wavefronts where D allows), and LDS exchanges the two.  Volumes written
// without a carry whose bins make no whole lines go by integrate_windows.
#pragma once

#include <type_traits>

#include "tsdf_device.h"

namespace gg {

constexpr int kFuseBins = 8;        // per lane and slab
constexpr int kFuseMaxWaves = 16;   // of a workgroup (LDS of slabs: 79 KB)

// Wavefronts per workgroup for D bins and a launch of nblocks workgroups:
// four, where a slab is one 128-byte line of each pixel if D is a multiple of
// 32.  The more workgroups share a compute unit, the better they hide each
// other's latencies and barriers (measured, video: 517 us with eight, 447 us
// with four).  Launches of no more workgroups than run at once take eight or
// sixteen: their slabs would run one after the other beside idle wavefronts
// (measured, 160 x 100 K=4 D=256: 54 us with four, 27 with sixteen).  Without a
// carry, whose registers leave room for six wavefronts per SIMD, eight run at
// once in up to 768 (240 x 150 K=4 D=128 32.2 us with four, 29.8 with eight;
// carried, 2% slower over D = 16 to 192).
__host__ __device__ inline int fuse_waves(int D, uint32_t nblocks, bool direct, bool carry) {
  const int chunks = (D + kFuseBins - 1) / kFuseBins;
  // 256 compute units of 16 to 24 wavefronts: one workgroup of 16, or two or three of 8
  int w = nblocks <= 256 ? (direct ? 8 : 16) : (nblocks <= (carry ? 512 : 768) ? 8 : 4);
  while (w > 1 && w / 2 >= chunks) w /= 2;
  return w;
}

// Whether a launch reads the cells' depth ranges (find_live).  The more views
// and the more chunks of 64 pixels x 8 bins there are, the more it drops and
// the better the test's chain of loads is hidden.  Measured, with and without:
// 1280 x 720 K=1 D=128 207 and 185 us, 640 x 400 K=2 D=64 43 and 40; 420 x 260
// K=3 D=48 (10 242 chunks) 35.5 and 30.9, 640 x 360 K=4 D=64 (28 800) 72.1 and
// 69.5, K=6 D=48 (21 600) 88.4 and 85.0, but K=4 D=100 (46 800) 95.3 and 96.3,
// 800 x 450 K=3 D=128 (90 000) 124.8 and 131.4.
__host__ __device__ inline bool fuse_ranges(int K, uint32_t nblocks, int D) {
  const uint64_t chunks = (uint64_t)nblocks * (uint32_t)((D + kFuseBins - 1) / kFuseBins);
  return K > 2 && chunks * (uint32_t)(K - 2) > 80000;
}

// LDS of a workgroup, in floats: F and W of the slab, F of each chunk's last
// bin by slab parity, and the first crossings (64-bit).
struct FuseLds {
  float *vol[2];             // 16-byte aligned
  float *edge;               // [parity][wave][pixel]
  unsigned long long *best;  // per pixel: bin << 32 | depth bits

  // of F or W: 8 waves floats per pixel, and 4 more per pixel or block of
  // pixels against bank conflicts (SlabRows, SlabDirect)
  static __host__ __device__ constexpr int array(int waves) { return (int)kFusePix * (8 * waves + 4); }
  static __host__ __device__ constexpr size_t bytes(int waves) {
    return sizeof(float) * (2 * array(waves) + 2 * waves * kFusePix + 2 * kFusePix);
  }
  __device__ __forceinline__ FuseLds(float *p, int waves) {
    vol[0] = p;
    vol[1] = p + array(waves);
    edge = vol[1] + array(waves);
    best = reinterpret_cast<unsigned long long *>(edge + 2 * waves * kFusePix);
  }
};

// Forms of the fusion kernel (integrate_form).
enum : int {
  kFormVec = 1,    // 16-byte accesses of the volume
  kFormLines = 2,  // and slabs of whole lines; a carried volume is loaded straight into LDS
  kFormRows = 4,   // structured view-table loads
  kFormCarry = 8,  // the previous volume is carried
  kFormWindows = 16,  // neither carry nor whole lines: integrate_windows
  kFuseForms = 32
};
__host__ __device__ constexpr bool form_exists(int f) {
  if (f & kFormWindows) return !(f & (kFormCarry | kFormLines));
  return (f & kFormVec) || ((f & kFormCarry) && !(f & kFormLines));
}
__host__ __device__ constexpr bool form_direct(int f) {
  return (f & kFormLines) && (f & kFormCarry);
}
// Wavefronts per SIMD that the registers must leave room for: three workgroups of eight.
__host__ __device__ constexpr int form_waves(int f) { return f & kFormWindows ? 6 : 4; }

// The bins of which one window holds a whole row in LDS, and of which two workgroups still fit a
// compute unit.
constexpr int kFuseWhole = 312, kFuseWholeTwice = 156;
constexpr uint32_t kFuseCuLds = 160u << 10;  // LDS of a compute unit

// Whether a launch without a carry, whose bins are not whole lines, goes by windows instead of
// slabs (integrate_windows).  Measured, slabs and windows: 1920 x 1080 K=1 D=100 831 and 351 us,
// K=8 D=75 1389 and 865; 1280 x 720 K=4 D=200 815 and 568; 637 x 359 K=6 D=104 131 and 118.  But
// with more bins than two workgroups have room for, few views and a volume that the 256 MB cache
// absorbs: 637 x 359 D=164 K=1 80 and 103, K=2 95 and 111.
__host__ __device__ constexpr bool fuse_windows(int K, int D, bool vec, size_t npix) {
  return !(vec && D > kFuseWholeTwice && K <= 3 && npix * (size_t)D <= (size_t)40 << 20);
}

// A launch's workgroups: wavefronts and LDS; of windows also their bins and LDS row.
struct FuseShape {
  int waves, span;
  uint32_t row;
  size_t lds;
};

// Windows of all bins where LDS holds them, the wavefronts taking their chunks in two rounds up to
// 64 bins, then eight or twelve of them (measured, 1280 x 720 K=1: D=48 with 3, 4 and 8 96, 101 and
// 117 us; D=100 with 7, 8, 12 and 13 180, 169, 187 and 266; D=125 with 8, 12 and 16 239, 225 and
// 320).  More than 156 bins leave one workgroup per compute unit: vector accesses of two or more
// views then take windows of 64 bins, three workgroups (1280 x 720 D=200 K=4 734 and 566, K=2 580
// and 461; K=1 446 and 452; single floats of D=233 K=4 821 and 1065: one window).  Small launches
// take as many wavefronts as run at once, few bins a wavefront per chunk (240 x 150 K=4 D=16 with
// one 18.4 us, with two 14.9), in rounds of as many chunks each: 333 x 200 K=4 D=48 with five, one
// chunk left for a second round, 29.4 us, with three 25.4; 240 x 150 K=4 D=100 29.0 with ten, 25.5
// with eight.  But where two rounds of workgroups share the LDS, the most (240 x 150 K=8 D=108 38.2
// with ten, 41.3 with eight).
__host__ inline FuseShape fuse_shape(int form, int K, int D, uint32_t nblocks) {
  FuseShape s{fuse_waves(D, nblocks, form_direct(form), (form & kFormCarry) != 0), 0, 0u, 0};
  s.lds = FuseLds::bytes(s.waves);
  if (form & kFormWindows) {
    const int chunks = (D + kFuseBins - 1) / kFuseBins;
    const bool more = D > kFuseWholeTwice;
    if (nblocks > 512) {
      const int rounds = (chunks + kFuseMaxWaves - 1) / kFuseMaxWaves;
      s.waves = D > 64 && D <= 108 ? 8 : D > 64 && !more ? 12 : (chunks - 1) / (rounds > 2 ? rounds : 2) + 1;
      // all that run at once, and a chunk each where there are few
      const int room = (int)(256u * 24u / nblocks);
      int least = D <= 24 ? chunks : (room < chunks ? room : chunks);
      // equal rounds, if the LDS has room for all workgroups at once
      const uint32_t lds = (uint32_t)sizeof(float) * 2u * kFusePix * (uint32_t)(D + 1);
      if (least > 0 && least < chunks && nblocks <= 256u * (kFuseCuLds / lds)) {
        const int r = (chunks - 1) / least + 1;
        least = (chunks - 1) / r + 1;
      }
      if (s.waves < least) s.waves = least;
    }
    s.span = kFuseBins * chunks;
    if (D > kFuseWhole || (more && K > 1 && nblocks > 512 && (form & kFormVec))) {
      s.waves = nblocks <= 256 ? 16 : 8;
      s.span = kFuseBins * s.waves;
    }
    s.row = (uint32_t)(s.span < D ? s.span + 36 : D);  // a ring's padded against bank conflicts
    s.lds = sizeof(float) * (2 * kFusePix * s.row + 2 * kFusePix);
  }
  return s;
}

// Read-only data addressed with wave-uniform addresses through the scalar
// unit: the argument record in the kernel's argument segment (or, batched, an
// item's descriptor) and the bin table.
#define GG_CONSTANT __attribute__((address_space(4)))
typedef const GG_CONSTANT IntegrateArgs *FuseArgs;

// The pointer itself, opaque to the compiler: fields read through it are read
// again from here on (scalar loads), not held in scalar registers, of which
// the tile needs more than there are.
__device__ __forceinline__ FuseArgs reread(FuseArgs a) {
  asm volatile("" : "+s"(a));
  return a;
}

// A wave-uniform value, for the compiler to hold in scalar registers.
__device__ __forceinline__ uint64_t uniform64(uint64_t v) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v) |
         ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32);
}

// ---------------------------------------------------------------------------
// samples of the wavefront's chunk

struct Chunk {
  float z[kFuseBins], tau[kFuseBins];  // wave-uniform
};

// One view for the lane's pixel: its ray and its table.
struct FuseView {
  float h0, h1, h2, c0, c1, c2;
  __amdgpu_buffer_rsrc_t table;
  uint32_t Ws, Hs, pitch8;
};

template <bool kRows>
__device__ __forceinline__ FuseView fuse_view(FuseArgs a, int k, float px, float py) {
  const GG_CONSTANT Proj &P = a->views[k];
  FuseView v;
  v.h0 = fmaf(P.H[0], px, fmaf(P.H[1], py, P.H[2]));  // ray_of
  v.h1 = fmaf(P.H[3], px, fmaf(P.H[4], py, P.H[5]));
  v.h2 = fmaf(P.H[6], px, fmaf(P.H[7], py, P.H[8]));
  v.c0 = P.c[0];
  v.c1 = P.c[1];
  v.c2 = P.c[2];
  v.Ws = (uint32_t)a->Ws;
  v.Hs = (uint32_t)a->Hs;
  v.pitch8 = table_pitch(a->Ws) * 8u;
  const uint32_t bytes = v.Hs * v.pitch8;
  const char *table = reinterpret_cast<const char *>(a->table) + (uint64_t)(uint32_t)k * bytes;
  v.table = kRows ? rows_of(table, v.pitch8, v.Hs) : buffer_of(table, bytes);
  return v;
}

// The record of the sample at pixel (i, j), of weight 0 where that lies
// outside the image (which drops it).  kRows: a structured load, row index
// and byte offset in the row; a row outside [0, Hs) -- a negative floor is a
// huge unsigned row -- is dropped by the load's range check, and a column
// outside [0, Ws) is clamped to Ws, the row's closing record (weight 0).  Else
// a range-checked raw load.
template <bool kRows>
__device__ __forceinline__ float2 load_record(const FuseView &v, uint32_t i, uint32_t j) {
  if constexpr (kRows) return rload2(v.table, j, min(i, v.Ws) << 3);
  // sizes are at most 16384 (host check): pitch8 < 2^24, the offset < 2^31
  return bload2(v.table, i < v.Ws && j < v.Hs ? __umul24(j, v.pitch8) + (i << 3) : kOutOfRange);
}

// A view's sample at depth z, every lane's in front (Z > 2^-100).
template <bool kRows>
__device__ __forceinline__ float2 front_sample(const FuseView &v, float z, float &Z) {
  const float X0 = fmaf(z, v.h0, v.c0), X1 = fmaf(z, v.h1, v.c1);
  Z = fmaf(z, v.h2, v.c2);
  const float inv = recip_rn(Z);
  return load_record<kRows>(v, (uint32_t)floor_i32(X0 * inv), (uint32_t)floor_i32(X1 * inv));
}

// The same wherever the lanes' points lie.  1 / Z is correctly rounded: for
// Z <= 2^-100 through the reciprocal of 2^100 Z, whose scaling is exact, and
// by IEEE division where the host found depths that may reach 2^99.
template <bool kRows>
__device__ __forceinline__ float2 any_sample(const FuseView &v, bool divide, float z, float &Z) {
  const float X0 = fmaf(z, v.h0, v.c0), X1 = fmaf(z, v.h1, v.c1);
  Z = fmaf(z, v.h2, v.c2);
  const float scale = Z > kRecipLo ? 1.0f : 0x1p100f;
  float inv = recip_rn(Z * scale) * scale;
  if (divide) inv = 1.0f / Z;
  const float u = X0 * inv, w = X1 * inv;
  const bool ok = Z > 0.0f && u >= 0.0f && u < (float)v.Ws && w >= 0.0f && w < (float)v.Hs;
  return load_record<kRows>(v, ok ? (uint32_t)u : v.Ws, ok ? (uint32_t)w : 0xffffffffu);
}

// Accumulate one sample: s = D_k - z_k, occlusion cut (s < -tau: dropped),
// clamp min(s, tau).  Branch-free: the clamp to [-tau, tau] equals
// min(s, tau) for every kept sample and stays finite for dropped ones (a
// hole's depth is -inf), which add (+0) * c and +0 and so leave S and Wo
// bitwise unchanged (both start at +0 and never become -0).
__device__ __forceinline__ void accumulate(float Z, float2 e, float tau, float &S, float &Wo) {
  const float s = e.x - Z;
  const float c = __builtin_amdgcn_fmed3f(s, -tau, tau);
  const float w = (s < -tau) ? 0.0f : e.y;
  S = fmaf(w, c, S);
  Wo = Wo + w;
}

// One view in front of every lane (each view by itself: one that reaches behind
// its camera leaves the others this form): the eight gathers are issued as their
// addresses are formed (two at a time: few registers, and the other
// wavefronts fill the latencies), then accumulated.  kFree: every usable
// sample lies at least tau in front of its surface, so the clamp gives tau
// whatever the depth and only the weights count (no pixel or a hole: 0).
// Whole records all the same: 4-byte gathers at this stride hold the texture
// address unit longer than 8-byte ones (measured: 76 to 97 us at 640 x 360 K=4 D=96).
// kN: the chunk's bins, the last chunk's four where it has no more.
template <bool kRows, bool kFree, int kN>
__device__ __forceinline__ void fuse_front(FuseArgs a, int k, float px, float py, const Chunk &b,
                                           float (&S)[kFuseBins], float (&Wo)[kFuseBins]) {
  const FuseView view = fuse_view<kRows>(a, k, px, py);
  float Z[kN];
  float2 e[kN];
#pragma unroll
  for (int v = 0; v < kN; ++v) {
    e[v] = front_sample<kRows>(view, b.z[v], Z[v]);
    if (v & 1) schedule_fence();
  }
#pragma unroll
  for (int v = 0; v < kN; ++v) {
    if constexpr (kFree) {
      asm volatile("" ::"v"(e[v].x));  // keeps the whole record's load
      S[v] = fmaf(e[v].y, b.tau[v], S[v]);
      Wo[v] = Wo[v] + e[v].y;
    } else {
      accumulate(Z[v], e[v], b.tau[v], S[v], Wo[v]);
    }
  }
}

template <bool kRows>
__device__ __forceinline__ void fuse_any(FuseArgs a, int k, float px, float py, const Chunk &b,
                                         float (&S)[kFuseBins], float (&Wo)[kFuseBins]) {
  const FuseView view = fuse_view<kRows>(a, k, px, py);
  const bool divide = a->exact_only != 0;
  float Z[kFuseBins];
  float2 e[kFuseBins];
#pragma unroll
  for (int v = 0; v < kFuseBins; ++v) {
    e[v] = any_sample<kRows>(view, divide, b.z[v], Z[v]);
    schedule_fence();
  }
#pragma unroll
  for (int v = 0; v < kFuseBins; ++v) accumulate(Z[v], e[v], b.tau[v], S[v], Wo[v]);
}

// ---------------------------------------------------------------------------
// views with nothing to keep, views in free space

// Minimum and maximum over each quad of lanes.
__device__ __forceinline__ float quad_min(float v) {
  v = fminf(v, row_swizzle<0xb1>(v));
  return fminf(v, row_swizzle<0x4e>(v));
}
__device__ __forceinline__ float quad_max(float v) {
  v = fmaxf(v, row_swizzle<0xb1>(v));
  return fmaxf(v, row_swizzle<0x4e>(v));
}

// Which views may keep a sample of the wavefront's patches, the tile's pixels
// times its chunk of 8 bins, for the next `slabs()` slabs at once.
//
// Lane (j, k, c), c fastest, holds corner c (first or last pixel, first or
// last bin) of view k's patch in slab slab0 + j.  The view's homogeneous
// coordinates are monotone in the pixel column and in the depth, also after
// rounding, so the corners bound Z exactly; and the patch is planar, so where
// Z > 0 its image lies in the corners' box, up to rounding: the rays'
// roundings (slack, an absolute bound that the host forms, over the least Z)
// and the quotients' (relative).  A tile over several target rows is taken at
// their middle, its half extent added to the slack and to the bounds of Z.  A
// view is dropped
//   - when no sample has Z > 0, or the box misses the image: no pixel;
//   - when the largest usable depth of the image cells that the box touches
//     lies more than tau in front of the least Z: with D <= max, every
//     s = D - Z rounds to at most max - Zlo < -tau, the occlusion cut.
// A dropped sample adds (+0) c and +0, which changes neither sum, so leaving
// it out gives the same bits.  And a view is in free space when the cells'
// least usable depth lies more than tau beyond the greatest Z: s > tau
// throughout.  The cells' extremes are over windows of 3 x 3 cells
// (cell_range), the lane's corner choosing the window: four of them cover a
// box of up to 6 x 6 cells; a larger box leaves its view as it is.
// Measured on the video, streaming and 960 x 540 K=8 cases it drops 37%, 49%
// and 41% of the (wavefront, view) pairs (42%, 54% and 46% hold nothing to
// keep) and finds 32%, 37% and 34% in free space; of the 640 x 360 parallel
// rig's, 5% and 71%.
struct TileRect {
  float x0, x1, y, ext;  // pixel columns, row; half extent in rows times a bound of the depths
};

struct LiveViews {
  // bits as the lanes: bit 4 (j << shift | k); free: in free space; behind:
  // not every sample in front
  uint64_t live, free, behind;
  uint32_t shift;  // log2 of the lanes' views (a power of two, at least K)

  __device__ __forceinline__ uint32_t slabs() const { return 16u >> shift; }
  __device__ __forceinline__ uint64_t of(uint64_t bits, uint32_t j, int K) const {
    return uniform64((bits >> (j << (shift + 2))) & (0x1111111111111111ull >> (64 - 4 * K)));
  }
};

__device__ __forceinline__ void find_live(FuseArgs a, const TileRect &rect, int chunk0, int waves,
                                          LiveViews &r) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t k = min((lane >> 2) & ((1u << r.shift) - 1u), (uint32_t)(a->K - 1));
  const GG_CONSTANT Proj &P = a->views[k];
  const float cx = (lane & 1u) ? rect.x1 : rect.x0;
  float h[3], e[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    h[i] = fmaf(P.H[3 * i], cx, fmaf(P.H[3 * i + 1], rect.y, P.H[3 * i + 2]));
    e[i] = fmaf(fabsf(P.H[3 * i + 1]), rect.ext, a->slack[k][i]);
  }
  const float ez = rect.ext > 0.0f ? e[2] : 0.0f;  // one row: Z's bounds are exact
  const int d0 = (chunk0 + (int)(lane >> (r.shift + 2)) * waves) * kFuseBins;
  const float2 b0 = gload2(a->bins + min(d0, a->D - 1)),
               b1 = gload2(a->bins + min(d0 + kFuseBins - 1, a->D - 1));
  const float zc = (lane & 2u) ? b1.x : b0.x;
  const float X0 = fmaf(zc, h[0], P.c[0]), X1 = fmaf(zc, h[1], P.c[1]), Z = fmaf(zc, h[2], P.c[2]);
  const float inv = __builtin_amdgcn_rcpf(Z);
  const float u = X0 * inv, v = X1 * inv;
  const float Zlo = quad_min(Z) - ez, Zhi = quad_max(Z) + ez;
  float u0 = quad_min(u), u1 = quad_max(u), v0 = quad_min(v), v1 = quad_max(v);
  // rounding of u, v over the patch, with a factor of two or more to spare
  const float ilo = __builtin_amdgcn_rcpf(Zlo) * (1.0f + 0x1p-20f);
  const float um = fmaxf(fabsf(u0), fabsf(u1)), vm = fmaxf(fabsf(v0), fabsf(v1));
  const float mu = fmaf(fmaf(um, e[2], e[0]), ilo, fmaf(um, 0x1p-20f, 0x1p-6f));
  const float mv = fmaf(fmaf(vm, e[2], e[1]), ilo, fmaf(vm, 0x1p-20f, 0x1p-6f));
  u0 -= mu;
  u1 += mu;
  v0 -= mv;
  v1 += mv;
  const float xl = (float)(a->Ws - 1), yl = (float)(a->Hs - 1);
  bool dead = u1 < 0.0f || u0 > xl + 1.0f || v1 < 0.0f || v0 > yl + 1.0f;
  bool free = false;
  // formed with this table (closing_record)?
  if (a->cells && ((const GG_CONSTANT float *)(const float *)a->table)[2 * a->Ws] != 0.0f) {
    const int a0 = (int)(fminf(fmaxf(u0, 0.0f), xl) * (1.0f / kCell));
    const int a1 = (int)(fminf(fmaxf(u1, 0.0f), xl) * (1.0f / kCell));
    const int c0 = (int)(fminf(fmaxf(v0, 0.0f), yl) * (1.0f / kCell));
    const int c1 = (int)(fminf(fmaxf(v1, 0.0f), yl) * (1.0f / kCell));
    const int ax = (lane & 1u) ? max(a0, a1 - 2) : a0, ay = (lane & 2u) ? max(c0, c1 - 2) : c0;
    const uint32_t cell =
        (k * cells_across(a->Hs) + (uint32_t)ay) * cells_across(a->Ws) + (uint32_t)ax;
    const float far = gmem(a->cells)[cell], near = gmem(a->cells)[a->ncells + cell];
    // no branch: a load that only one side waits for would have every slab's
    // first view wait for all memory traffic before it, the stores too
    const bool fits = (a1 - a0 < 6) & (c1 - c0 < 6);
    dead |= fits & (quad_max(far) - Zlo < -b1.y);
    free = fits & (quad_min(near) - Zhi > b1.y);
  }
  // far enough from the camera plane for the bounds above
  const bool clear = Zlo > 0x1p-40f;
  dead = (dead && clear) || !(Zhi > 0.0f);
  r.free = __builtin_amdgcn_ballot_w64(free && clear);
  r.live = ~__builtin_amdgcn_ballot_w64(dead);
  r.behind = __builtin_amdgcn_ballot_w64(!(Zlo > kRecipLo));
}

// ---------------------------------------------------------------------------
// the tile

// A slab's F or W between memory, LDS and the fusing lanes.  The workgroup's
// threads take the slab's accesses in order, pixel after pixel, each the same
// places of the runs whether it loads or stores them.  The volume is read and
// written once per launch: its accesses are non-temporal, so that they pass
// through the caches without evicting the view-table lines that the gathers
// of neighbouring tiles reuse (measured: the video fusion 447 us against 490
// with either direction temporal).
//
// Where slabs cut lines (kLines false) they are not: the line's other part
// follows a slab later.
template <bool kLines, typename T>
__device__ __forceinline__ T stream_load(const GG_GLOBAL T *p) {
  if constexpr (kLines) return __builtin_nontemporal_load(p);
  return *p;
}
template <bool kLines, typename T>
__device__ __forceinline__ void stream_store(T v, GG_GLOBAL T *p) {
  if constexpr (kLines)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

// SlabRows: a row of 8 waves + 4 floats per pixel; loads through registers.
// kVec: 16-byte accesses (D a multiple of 4, the volume 16-byte aligned),
// else single floats.
template <bool kVec, bool kLines>
struct SlabRows {
  static constexpr uint32_t kWide = kVec ? 4 : 1;
  static constexpr int kIssues = kVec ? 2 : 8;
  static constexpr uint32_t kStep = kFusePix / kIssues;
  struct Held {
    float v[kIssues][kWide];
  };
  uint32_t p, j;     // the thread's first pixel, and its bin in the runs
  uint32_t row;      // floats
  uint32_t last, D;  // the tile's last pixel

  __device__ __forceinline__ SlabRows(uint32_t waves, uint32_t last_, int D_)
      : row(8u * waves + 4u), last(last_), D((uint32_t)D_) {
    const uint32_t per = 8u / kWide * waves;  // accesses per run
    p = threadIdx.x / per;
    j = (threadIdx.x - p * per) * kWide;
  }
  // Unconditional (past the volume they repeat its last pixel or bin, which
  // nothing stores back): no branch separates them from the view gathers, so
  // the compiler's in-order wait counts need not assume that these
  // long-latency loads precede every gather.
  __device__ __forceinline__ void load(const float *tile, float *, int d0, Held &r) const {
    const uint32_t d = min((uint32_t)d0 + j, D - kWide);
#pragma unroll
    for (int h = 0; h < kIssues; ++h) {
      const uint32_t o = min(p + (uint32_t)h * kStep, last) * D + d;
      if constexpr (kVec) {
        const gg_v4f x = stream_load<kLines>((const GG_GLOBAL gg_v4f *)(tile + o));
        r.v[h][0] = x.x;
        r.v[h][1] = x.y;
        r.v[h][2] = x.z;
        r.v[h][3] = x.w;
      } else {
        r.v[h][0] = stream_load<kLines>((const GG_GLOBAL float *)(tile + o));
      }
    }
  }
  __device__ __forceinline__ void arrive(float *vol, const Held &r) const {
#pragma unroll
    for (int h = 0; h < kIssues; ++h) {
      float *q = vol + (p + (uint32_t)h * kStep) * row + j;
      if constexpr (kVec)
        *(gg_v4f *)q = (gg_v4f){r.v[h][0], r.v[h][1], r.v[h][2], r.v[h][3]};
      else
        *q = r.v[h][0];
    }
  }
  __device__ __forceinline__ void store(const float *vol, float *tile, int d0) const {
    if ((uint32_t)d0 + j >= D) return;
#pragma unroll
    for (int h = 0; h < kIssues; ++h) {
      const uint32_t q = p + (uint32_t)h * kStep;
      if (q > last) continue;
      const float *v = vol + q * row + j;
      float *o = tile + (q * D + (uint32_t)d0 + j);
      if constexpr (kVec)
        stream_store<kLines>(*(const gg_v4f *)v, (GG_GLOBAL gg_v4f *)o);
      else
        stream_store<kLines>(*v, (GG_GLOBAL float *)o);
    }
  }
  // four bins 8 wave + 4 q of the lane's pixel
  __device__ __forceinline__ uint32_t quad(uint32_t lane, int wave, int q) const {
    return lane * row + 8u * (uint32_t)wave + 4u * (uint32_t)q;
  }
};

// SlabDirect: 16-byte loads straight into LDS, which hold no registers (five
// wavefronts per SIMD instead of four).  Such a load puts a wavefront's 64 accesses one
// after the other, so a block of 64 / (2 waves) pixels lies contiguous; for
// the fusing lanes, one per pixel, the four-bin groups of a run are permuted
// by the pixel (group g at slot g xor p), and blocks are 4 floats apart more:
// no bank conflicts with four wavefronts.  1, 2, 4 or 8 wavefronts.
struct SlabDirect {
  static constexpr int kIssues = 2;
  static constexpr uint32_t kStep = kFusePix / kIssues, kBlock = 64 * 4 + 4;
  struct Held {};
  uint32_t p, j;     // the thread's first pixel, and its bin in the runs
  uint32_t slot;     // its place in LDS for the first access
  uint32_t mask, shift;  // groups per run - 1; log2 of pixels per block
  uint32_t last, D, waves;

  __device__ __forceinline__ SlabDirect(uint32_t waves_, uint32_t last_, int D_)
      : last(last_), D((uint32_t)D_), waves(waves_) {
    mask = 2u * waves - 1u;
    shift = 5u - (31u - (uint32_t)__builtin_clz(waves));  // 32 / waves pixels
    p = threadIdx.x >> (6u - shift);
    j = (((threadIdx.x & mask) ^ p) & mask) * 4u;
    slot = (threadIdx.x >> 6) * kBlock + (threadIdx.x & 63u) * 4u;
  }
  // Unconditional, as SlabRows.  The thread's second access is a whole number
  // of blocks on: the same group of the run (kStep is a multiple of the
  // groups' count).
  __device__ __forceinline__ void load(const float *tile, float *vol, int d0, Held &) const {
    const uint32_t d = min((uint32_t)d0 + j, D - 4u);
    const uint32_t block = (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
    for (int h = 0; h < kIssues; ++h) {
      const uint32_t o = min(p + (uint32_t)h * kStep, last) * D + d;
      // the wavefront's block; cache policy 2: non-temporal
      __builtin_amdgcn_global_load_lds(
          (const GG_GLOBAL void *)(tile + o),
          (__attribute__((address_space(3))) void *)(vol + (block + (uint32_t)h * waves) * kBlock),
          16, 0, 2);
    }
  }
  // The wavefront's own loads have landed (the barrier after covers the others').
  __device__ __forceinline__ void arrive(float *, const Held &) const {
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  }
  __device__ __forceinline__ void store(const float *vol, float *tile, int d0) const {
    if ((uint32_t)d0 + j >= D) return;
#pragma unroll
    for (int h = 0; h < kIssues; ++h) {
      const uint32_t q = p + (uint32_t)h * kStep;
      if (q > last) continue;
      const gg_v4f x = *(const gg_v4f *)(vol + slot + (uint32_t)h * waves * kBlock);
      __builtin_nontemporal_store(x, (GG_GLOBAL gg_v4f *)(tile + (q * D + (uint32_t)d0 + j)));
    }
  }
  __device__ __forceinline__ uint32_t quad(uint32_t lane, int wave, int q) const {
    const uint32_t g = ((2u * (uint32_t)wave + (uint32_t)q) ^ lane) & mask;
    return (lane >> shift) * kBlock + (lane & ((1u << shift) - 1u)) * 8u * waves + 4u * g;
  }
};

// The crossing between bins d and d + 1, of depths za and zb: the bin above,
// the interpolated depth below.
__device__ __forceinline__ unsigned long long crossing_key(int d, float za, float zb, float f0,
                                                           float f1) {
  const float frac = f0 / (f0 - f1);
  return ((unsigned long long)(uint32_t)d << 32) | __float_as_uint(za + (zb - za) * frac);
}

// The samples of every view in the wavefront's chunk of 8 bins from d0, the
// sub-th of the slabs that lv holds.  False: no view may keep any.  kWhole: D
// is a multiple of 8.  Else a last chunk of at most four bins samples only four
// (measured, all eight and four: 1280 x 720 K=4 D=2 64 and 52 us).
template <bool kRows, bool kWhole>
__device__ __forceinline__ bool fuse_chunk(FuseArgs a, const LiveViews &lv, uint32_t sub, int d0,
                                           float px, float py, float (&S)[kFuseBins],
                                           float (&Wo)[kFuseBins]) {
  Chunk b;  // bins past D repeat the last one
  const GG_CONSTANT float *bt = (const GG_CONSTANT float *)(const float *)(a->bins + d0);
#pragma unroll
  for (int v = 0; v < kFuseBins; ++v) {
    b.z[v] = bt[2 * v];
    b.tau[v] = bt[2 * v + 1];
  }
  uint64_t live = a->K ? 0x1111111111111111ull >> (64 - 4 * a->K) : 0ull, free = 0;
  uint64_t behind = a->front ? 0ull : live;
  if (a->test) {
    live = lv.of(lv.live, sub, a->K);
    free = lv.of(lv.free, sub, a->K);
    behind = lv.of(lv.behind, sub, a->K);
  }
  const bool some = live != 0, half = !kWhole && a->D - d0 <= 4;
#pragma nounroll
  while (live) {
    const int bit = __builtin_ctzll(live), k = __builtin_amdgcn_readfirstlane(bit >> 2);
    live = uniform64(live & (live - 1));
    if ((behind >> bit) & 1u)
      fuse_any<kRows>(a, k, px, py, b, S, Wo);
    else if (half)
      fuse_front<kRows, false, 4>(a, k, px, py, b, S, Wo);
    else if ((free >> bit) & 1u)
      fuse_front<kRows, true, kFuseBins>(a, k, px, py, b, S, Wo);
    else
      fuse_front<kRows, false, kFuseBins>(a, k, px, py, b, S, Wo);
  }
  return some;
}

// The place of a tile in the target.
struct FuseTile {
  uint32_t pix0, pix, last;  // first pixel, the lane's, the tile's last from the first
  float px, py;              // the lane's pixel
  TileRect rect;

  __device__ __forceinline__ FuseTile(FuseArgs a, uint32_t tile) {
    pix0 = tile * kFusePix;
    pix = pix0 + (threadIdx.x & 63u);
    last = min(kFusePix - 1u, a->npix - 1u - pix0);
    const FastDiv wt = {a->wt_div.d, a->wt_div.m, a->wt_div.s};
    const uint32_t y = fdiv(pix, wt), x = pix - y * wt.d;
    px = (float)x + 0.5f;
    py = (float)y + 0.5f;
    // its part of one target row, or every column of the rows it runs over, taken at their middle
    const uint32_t y0 = fdiv(pix0, wt), x0 = pix0 - y0 * wt.d, y1 = fdiv(pix0 + last, wt);
    rect.x0 = (float)(y1 > y0 ? 0u : x0) + 0.5f;
    rect.x1 = (float)(y1 > y0 ? wt.d - 1u : x0 + last) + 0.5f;
    rect.y = 0.5f * (float)(y0 + y1) + 0.5f;
    rect.ext = (float)(y1 - y0) * (0.5f * a->zfar);
  }
};

// A tile in windows of a->span bins held in LDS, without a carry: where bins
// do not make whole lines, so that a slab's stores would cut two lines of
// every pixel.  Lines cut in time leave the caches half written, and such
// stores bound the kernel.  Mostly one window holds all D bins: the tile's 64
// runs are one contiguous piece of the volume, stored at the end.  With more
// bins (a multiple of the wavefronts' per window) each pixel's run is stored
// up to the last line that the window completes; its other bins, less than a
// line, stay in LDS, a ring of span + 32 bins per pixel.
template <int kForm>
__device__ __forceinline__ void integrate_windows(FuseArgs a, uint32_t tile, float *smem) {
  constexpr bool kRows = (kForm & kFormRows) != 0;
  constexpr int kWide = (kForm & kFormVec) ? 4 : 1;
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const int wave = (int)__builtin_amdgcn_readfirstlane(t >> 6), waves = (int)(blockDim.x >> 6);
  const int D = a->D, step = waves * kFuseBins, span = a->span, ring = span < D ? span + 32 : D;
  const uint32_t row = a->row;
  float *vol[2] = {smem, smem + kFusePix * row};
  unsigned long long *best = reinterpret_cast<unsigned long long *>(smem + 2 * kFusePix * row);
  const FuseTile T(a, tile);
  if (t < kFusePix) best[t] = ~0ull;
  if (a->out_depth) __syncthreads();
  LiveViews lv;
  lv.shift = a->K > 1 ? 32u - (uint32_t)__builtin_clz((uint32_t)(a->K - 1)) : 0u;
  lv.live = lv.free = lv.behind = 0;
  int slab = 0, at0 = 0;  // at0: the place of bin w0 in the ring
  for (int w0 = 0; w0 < D; w0 += span) {
    const int w1 = min(w0 + span, D);
    for (int d0 = w0 + wave * kFuseBins; d0 < w1; d0 += step, ++slab) {
      a = reread(a);
      float S[kFuseBins], Wo[kFuseBins];
#pragma unroll
      for (int v = 0; v < kFuseBins; ++v) S[v] = Wo[v] = 0.0f;
      const uint32_t sub = (uint32_t)slab & (lv.slabs() - 1u);
      if (a->test && sub == 0) find_live(a, T.rect, d0 / kFuseBins, waves, lv);
      const bool some = fuse_chunk<kRows, false>(a, lv, sub, d0, T.px, T.py, S, Wo);
      a = reread(a);
      if (some) {
#pragma unroll
        for (int v = 0; v < kFuseBins; ++v) {
          float mean = S[v] / Wo[v];
          asm volatile("" : "+v"(mean));  // no branch around each division: they run abreast
          S[v] = Wo[v] > 0.0f ? mean : 0.0f;
        }
      }
      int at = at0 + (d0 - w0);  // (a chunk lies whole in the ring: both are multiples of 8)
      if (at >= ring) at -= ring;
      float *f = vol[0] + lane * row + at, *w = vol[1] + lane * row + at;
      if constexpr (kWide == 4) {
#pragma unroll
        for (int q = 0; q < kFuseBins; q += 4)
          if (d0 + q < w1) {
            *(gg_v4f *)(f + q) = (gg_v4f){S[q], S[q + 1], S[q + 2], S[q + 3]};
            *(gg_v4f *)(w + q) = (gg_v4f){Wo[q], Wo[q + 1], Wo[q + 2], Wo[q + 3]};
          }
      } else {
#pragma unroll
        for (int v = 0; v < kFuseBins; ++v)
          if (d0 + v < w1) f[v] = S[v], w[v] = Wo[v];
      }
      if (a->out_depth && some) {
        // the first crossing within the chunk
        const GG_CONSTANT float *bt = (const GG_CONSTANT float *)(const float *)(a->bins + d0);
        int d = -1;
        float f0 = 1.0f, f1 = 0.0f, za = 0.0f, zb = 0.0f;
#pragma unroll
        for (int v = kFuseBins - 1; v >= 1; --v)
          if (d0 + v < D && S[v - 1] > 0.0f && Wo[v] > 0.0f && S[v] <= 0.0f) {
            d = d0 + v - 1;
            f0 = S[v - 1];
            f1 = S[v];
            za = bt[2 * v - 2];
            zb = bt[2 * v];
          }
        if (d >= 0) atomicMin(&best[lane], crossing_key(d, za, zb, f0, f1));
      }
    }
    __syncthreads();  // the window is staged
    float *out[2] = {a->F + (size_t)T.pix0 * (size_t)D, a->W + (size_t)T.pix0 * (size_t)D};
    const uint32_t base[2] = {(uint32_t)((uintptr_t)out[0] >> 2), (uint32_t)((uintptr_t)out[1] >> 2)};
    if (span >= D && row == (uint32_t)D && ((base[0] | base[1]) & 3u) == 0) {
      // the tile's runs, as they lie in LDS
      const uint32_t n = (T.last + 1u) * (uint32_t)D;
      for (uint32_t e = 4u * t; e < n; e += 4u * blockDim.x) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          if (kWide == 4 || e + 4u <= n)
            __builtin_nontemporal_store(*(const gg_v4f *)(vol[h] + e), (GG_GLOBAL gg_v4f *)(out[h] + e));
          else
            for (uint32_t i = e; i < n; ++i) gmem(out[h])[i] = vol[h][i];
        }
      }
    } else {
      // run by run, from a line's start (or the run's) to another's (or the run's end)
      const int per = (span >= D ? D : span + 32) / kWide;  // accesses per run, at most
      const int dp = (int)blockDim.x / per, dj = (int)blockDim.x - dp * per;
      auto store_runs = [&](int h0, int h1) {
        int p = (int)t / per, j = (int)t - p * per;
        while (p <= (int)T.last) {
          const uint32_t b = base[h0] + (uint32_t)(p * D);
          const int lo = w0 > 0 ? w0 - (int)((b + (uint32_t)w0) & 31u) : 0;
          const int hi = w1 < D ? w1 - (int)((b + (uint32_t)w1) & 31u) : D;
          const int d = lo + j * kWide;
          if (d < hi) {
            int at = at0 + (d - w0);
            if (at < 0) at += ring;
            if (at >= ring) at -= ring;
            for (int h = h0; h < h1; ++h) {
              const float *from = vol[h] + (uint32_t)p * row + at;
              GG_GLOBAL float *to = gmem(out[h]) + (p * D + d);
              if constexpr (kWide == 4)
                __builtin_nontemporal_store(*(const gg_v4f *)from, (GG_GLOBAL gg_v4f *)to);
              else
                __builtin_nontemporal_store(*from, to);
            }
          }
          p += dp;
          j += dj;
          if (j >= per) {
            j -= per;
            ++p;
          }
        }
      };
      if (span >= D || ((base[0] ^ base[1]) & 31u) == 0) {  // F and W alike
        store_runs(0, 2);
      } else {
        store_runs(0, 1);
        store_runs(1, 2);
      }
    }
    if (a->out_depth) {
      // crossings between chunks (before the first bin of all there is none)
      for (int d = w0 + wave * kFuseBins; d < w1; d += step) {
        if (d == 0) continue;
        int at = at0 + (d - w0);
        if (at >= ring) at -= ring;
        const float *f = vol[0] + lane * row, *w = vol[1] + lane * row;
        const float f0 = f[at > 0 ? at - 1 : ring - 1], f1 = f[at];
        if (f0 > 0.0f && w[at] > 0.0f && f1 <= 0.0f) {
          const GG_CONSTANT float *bt = (const GG_CONSTANT float *)(const float *)(a->bins + d);
          atomicMin(&best[lane], crossing_key(d - 1, bt[-2], bt[0], f0, f1));
        }
      }
    }
    if (w1 < D) __syncthreads();  // the window has been read
    at0 += span;
    if (at0 >= ring) at0 -= ring;
  }
  if (a->out_depth) {
    __syncthreads();
    if (t < kFusePix && T.pix < a->npix) {
      const unsigned long long key = best[t];
      gmem(a->out_depth)[T.pix] = key == ~0ull ? 0.0f : __uint_as_float((uint32_t)key);
      gmem(a->out_bin)[T.pix] = key == ~0ull ? -1 : (int32_t)(key >> 32);
    }
  }
}

// Tile `tile` (kFusePix pixels) of one target, in the form of integrate_form.
template <int kForm>
__device__ __forceinline__ void integrate_tile(FuseArgs a, uint32_t tile, float *smem) {
  if constexpr ((kForm & kFormWindows) != 0) return integrate_windows<kForm>(a, tile, smem);
  constexpr bool kCarry = (kForm & kFormCarry) != 0, kRows = (kForm & kFormRows) != 0;
  constexpr bool kLines = (kForm & kFormLines) != 0, kVec = (kForm & kFormVec) != 0;
  constexpr bool kDirect = kCarry && kLines;
  const uint32_t t = threadIdx.x, lane = t & 63u;
  const int wave = (int)__builtin_amdgcn_readfirstlane(t >> 6), waves = (int)(blockDim.x >> 6);
  const FuseLds L(smem, waves);
  const int D = a->D;
  const FuseTile T(a, tile);
  if (t < kFusePix) L.best[t] = ~0ull;  // the first slab's barriers precede its use
  float m = 1.0f;
  if (kCarry && a->mask) m = fmaxf(1.0f - gmem(a->mask)[min(T.pix, a->npix - 1u)], 0.0f);

  typedef std::conditional_t<kDirect, SlabDirect, SlabRows<kVec, kLines>> Slab;
  const Slab slabs((uint32_t)waves, T.last, D);
  const size_t base = (size_t)T.pix0 * (size_t)D;
  typename Slab::Held rF, rW;
  // the previous volume's slab from s0
  auto load_volume = [&](int s0) {
    schedule_fence();
    slabs.load(a->F_prev + base, L.vol[0], s0, rF);
    slabs.load(a->W_prev + base, L.vol[1], s0, rW);
    schedule_fence();
  };
  if constexpr (kCarry) load_volume(0);
  LiveViews lv;
  lv.shift = a->K > 1 ? 32u - (uint32_t)__builtin_clz((uint32_t)(a->K - 1)) : 0u;
  lv.live = lv.free = lv.behind = 0;
  const int step = waves * kFuseBins;
  for (int s0 = 0, slab = 0; s0 < D; s0 += step, ++slab) {
    a = reread(a);
    const int d0 = s0 + wave * kFuseBins, par = slab & 1;  // the wavefront's chunk
    float S[kFuseBins], Wo[kFuseBins];
#pragma unroll
    for (int v = 0; v < kFuseBins; ++v) S[v] = Wo[v] = 0.0f;
    const uint32_t sub = (uint32_t)slab & (lv.slabs() - 1u);
    if (a->test && sub == 0) find_live(a, T.rect, slab * waves + wave, waves, lv);
    // without a view and a volume to carry, the chunk is zero and has no crossing
    bool some = kCarry;
    if (d0 < D) some |= fuse_chunk<kRows, kLines>(a, lv, sub, d0, T.px, T.py, S, Wo);
    a = reread(a);
    if constexpr (kCarry) {
      slabs.arrive(L.vol[0], rF);
      slabs.arrive(L.vol[1], rW);
      if constexpr (!kDirect) {
        if (s0 + step < D) load_volume(s0 + step);  // through registers: a slab ahead
      }
    }
    __syncthreads();  // the slab's previous F and W are in LDS; the last slab is stored
    const float decay = a->decay, cap = a->cap;
    float Fn[kFuseBins], Wn[kFuseBins];
    if (some) {
#pragma unroll
      for (int q = 0; q < kFuseBins / 4; ++q) {
        gg_v4f f = {0.0f, 0.0f, 0.0f, 0.0f}, w = f;
        const uint32_t at = slabs.quad(lane, wave, q);
        if constexpr (kCarry) {
          f = *(const gg_v4f *)(L.vol[0] + at);
          w = *(const gg_v4f *)(L.vol[1] + at);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int v = 4 * q + i;
          const float wp = kCarry ? fminf((decay * w[i]) * m, cap) : 0.0f;
          const float wn = wp + Wo[v];
          float mean = fmaf(wp, f[i], S[v]) / wn;
          asm volatile("" : "+v"(mean));  // no branch around each division: four run abreast
          Fn[v] = wn > 0.0f ? mean : 0.0f;
          Wn[v] = wn;
        }
        *(gg_v4f *)(L.vol[0] + at) = (gg_v4f){Fn[4 * q], Fn[4 * q + 1], Fn[4 * q + 2], Fn[4 * q + 3]};
        *(gg_v4f *)(L.vol[1] + at) = (gg_v4f){Wn[4 * q], Wn[4 * q + 1], Wn[4 * q + 2], Wn[4 * q + 3]};
        schedule_fence();
      }
    } else {
#pragma unroll
      for (int v = 0; v < kFuseBins; ++v) Fn[v] = Wn[v] = 0.0f;
#pragma unroll
      for (int q = 0; q < kFuseBins / 4; ++q) {
        const uint32_t at = slabs.quad(lane, wave, q);
        *(gg_v4f *)(L.vol[0] + at) = *(gg_v4f *)(L.vol[1] + at) = (gg_v4f){0.0f, 0.0f, 0.0f, 0.0f};
      }
    }
    // F of the last bin of the chunk before: the other wavefronts' after the
    // barrier, the previous slab's (kept by parity) before it
    float *edge = L.edge + lane;
    float Fprev = 0.0f;
    if (wave == 0 && slab > 0) Fprev = edge[((par ^ 1) * waves + waves - 1) * (int)kFusePix];
    edge[(par * waves + wave) * (int)kFusePix] = Fn[kFuseBins - 1];
    __syncthreads();  // the slab's new F and W are staged
    slabs.store(L.vol[0], a->F + base, s0);
    slabs.store(L.vol[1], a->W + base, s0);
    if constexpr (kDirect) {
      // into the places this thread has just read: its reads are done
      if (s0 + step < D) {
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        load_volume(s0 + step);
      }
    }
    if (a->out_depth && some && d0 < D) {
      // F > 0 means an observed bin (an unobserved one holds 0)
      if (wave > 0) Fprev = edge[(par * waves + wave - 1) * (int)kFusePix];
      uint64_t hit = 0;
#pragma unroll
      for (int v = 0; v < kFuseBins; ++v) {
        const float f0 = v ? Fn[v ? v - 1 : 0] : Fprev;
        const uint64_t h = __builtin_amdgcn_ballot_w64(f0 > 0.0f) &
                           __builtin_amdgcn_ballot_w64(Fn[v] <= 0.0f) &
                           __builtin_amdgcn_ballot_w64(Wn[v] > 0.0f);
        if (d0 + v < D) hit |= h;
      }
      if (hit) {
        // the chunk's first crossing (the first bin of all has Fprev = 0); the
        // smallest bin of the pixel wins (order-free).  The depths by scalar
        // loads: a vector load's wait would include the stores above.
        const GG_CONSTANT float *bt = (const GG_CONSTANT float *)(const float *)(a->bins + d0);
        int d = -1;
        float f0 = 1.0f, f1 = 0.0f, za = 0.0f, zb = 0.0f;
#pragma unroll
        for (int v = kFuseBins - 1; v >= 0; --v) {
          const float g0 = v ? Fn[v ? v - 1 : 0] : Fprev;
          if (d0 + v < D && g0 > 0.0f && Wn[v] > 0.0f && Fn[v] <= 0.0f) {
            d = d0 + v - 1;
            f0 = g0;
            f1 = Fn[v];
            za = v ? bt[2 * v - 2] : bt[d0 ? -2 : 0];
            zb = bt[2 * v];
          }
        }
        if (d >= 0) atomicMin(&L.best[lane], crossing_key(d, za, zb, f0, f1));
      }
    }
  }
  if (a->out_depth) {
    __syncthreads();
    if (t < kFusePix && T.pix < a->npix) {
      const unsigned long long key = L.best[t];
      gmem(a->out_depth)[T.pix] = key == ~0ull ? 0.0f : __uint_as_float((uint32_t)key);
      gmem(a->out_bin)[T.pix] = key == ~0ull ? -1 : (int32_t)(key >> 32);
    }
  }
}

}  // namespace gg
