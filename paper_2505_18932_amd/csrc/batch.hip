// Batched path: many target views of uneven resolution, view count and bin
// count fused by kernels over per-phase work lists, the whole batch captured
// once into a hipGraph and replayed with one launch.
//
// Each work item runs the same device function as the plain entry points
// (conf_tile, splat_bin_block, alloc_block, raster_tile,
// integrate_tile), so every output is bitwise identical to the
// corresponding plain call.  Work lists are grouped by item; each phase runs
// one workgroup per entry, and each XCD walks a contiguous part of a list.
#include <cstring>
#include <vector>

#include "batch_internal.h"

namespace gg {

// ---------------------------------------------------------------------------
// device phases

__global__ void batch_zero_kernel(uint32_t *p, size_t n) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

__global__ void batch_bins_kernel(const BatchItem *__restrict__ items) {
  const BatchItem &it = items[blockIdx.x];
  for (uint32_t d = threadIdx.x; d < padded_bins(it.D); d += blockDim.x)
    gstore2(it.bins + d, bin_record((int)d, it.D, it.z_near, it.z_far, it.trunc, it.trunc_in_bins));
  for (uint32_t c = threadIdx.x; c < 2 * it.conf.ncells; c += blockDim.x)
    gmem(it.conf.cells)[c] = cell_start(c, it.conf.ncells);
}

// The phases run one workgroup per entry, as their plain launches run one per
// tile: their lists hold far more entries than the device holds workgroups,
// so the dispatcher balances them as well as a work queue would, and gives
// the two branches' workgroups their turns as others end (measured, six items
// of 480 x 270 to 1280 x 720: 2225 us with the binning in persistent
// workgroups, which kept the fusion's out, 1521 without).  Entries go to the XCDs in
// contiguous parts (xcd_tile), so the tiles in flight on an XCD are
// neighbours in the list and share the lines in its L2.
__global__ __launch_bounds__(256) void batch_conf_kernel(const BatchItem *__restrict__ items,
                                                         const WorkItem *__restrict__ work,
                                                         uint32_t n) {
  __shared__ float tile[conf_tile_floats(kBatchConfRows)];
  const WorkItem wi = uniform_entry(work, xcd_tile(blockIdx.x, n));
  conf_tile<kBatchConfRows>(items[wi.item].conf, wi.k, wi.x, wi.y, tile);
}

template <bool kFill>
__global__ __launch_bounds__(256) void batch_bin_kernel(const BatchItem *__restrict__ items,
                                                        const WorkItem *__restrict__ work,
                                                        uint32_t n) {
  const WorkItem wi = uniform_entry(work, xcd_tile(blockIdx.x, n));
  splat_bin_block<kFill>(items[wi.item].splat, wi.k, work_tile(wi));
}

__global__ __launch_bounds__(kAllocThreads) void batch_alloc_kernel(
    const BatchItem *__restrict__ items, const uint32_t *__restrict__ list) {
  const SplatArgs &a = items[list[blockIdx.x]].splat;
  const uint32_t n = (uint32_t)a.K * a.ntiles;
  for (uint32_t base = blockIdx.y * kAllocTiles; base < n; base += gridDim.y * kAllocTiles)
    alloc_block(a.tile_count, a.tile_offset, a.tile_cursor, n, base);
}

__global__ __launch_bounds__(256) void batch_raster_kernel(const BatchItem *__restrict__ items,
                                                           const WorkItem *__restrict__ work,
                                                           uint32_t n) {
  __shared__ RasterLds lds;
  const WorkItem wi = uniform_entry(work, xcd_tile(blockIdx.x, n));
  raster_tile<false>(items[wi.item].splat, wi.k, work_tile(wi), lds);
}

// Fusion: one workgroup tile of one item per work entry, every entry of a
// launch in the same form of the plain kernel (so the same code); each
// item's tiles are listed in the plain launch's band order.
template <int kForm>
__global__ __launch_bounds__(64 * kFuseMaxWaves, form_waves(kForm)) void batch_integrate_kernel(
    const BatchItem *__restrict__ items, const WorkItem *__restrict__ work, uint32_t n) {
  extern __shared__ __align__(16) float smem[];
  const WorkItem wi = uniform_entry(work, xcd_tile(blockIdx.x, n));
  integrate_tile<kForm>((FuseArgs)(const IntegrateArgs *)&items[wi.item].integ, work_tile(wi), smem);
}

template <int kForm>
static void launch_integ_form(const BatchPlan &P, const IntegGroup &g, hipStream_t s) {
  if constexpr (kForm < kFuseForms) {
    if (g.form != kForm) return launch_integ_form<kForm + 1>(P, g, s);
    if constexpr (form_exists(kForm))
      hipLaunchKernelGGL(batch_integrate_kernel<kForm>, dim3(g.n), dim3(64 * g.waves),
                         g.lds, s, P.d_items, g.list, g.n);
  }
}

// ---------------------------------------------------------------------------
// plan

int batch_record(BatchPlan &P, hipStream_t s, hipStream_t side, hipEvent_t fork,
                 hipEvent_t join) {
  // tile counts and list allocators of every item
  hipLaunchKernelGGL(batch_zero_kernel, dim3(1024), dim3(256), 0, s, P.zero_ptr, P.zero_words);
  // The splat phases depend on the depth maps and the zeroed counts only: with a side stream
  // they form a second branch of the graph, beside the bins, weights and fusion of the main
  // branch, and the two overlap; the branches join before the graph ends.
  const bool branch = side && P.n_bin && P.branches != 1;
  if (branch) {
    if (int rc = check_hip(hipEventRecord(fork, s), "batch fork")) return rc;
    if (int rc = check_hip(hipStreamWaitEvent(side, fork, 0), "batch fork")) return rc;
  }
  const hipStream_t ss = branch ? side : s;
  if (P.n_bin) {
    hipLaunchKernelGGL(batch_bin_kernel<false>, dim3(P.n_bin), dim3(256), 0, ss, P.d_items, P.d_bin,
                       P.n_bin);
    hipLaunchKernelGGL(batch_alloc_kernel, dim3(P.n_splat_items, 16), dim3(kAllocThreads), 0, ss,
                       P.d_items, P.d_splat_items);
    hipLaunchKernelGGL(batch_bin_kernel<true>, dim3(P.n_bin), dim3(256), 0, ss, P.d_items, P.d_bin,
                       P.n_bin);
    if (P.n_raster)
      hipLaunchKernelGGL(batch_raster_kernel, dim3(P.n_raster), dim3(256), 0, ss, P.d_items,
                         P.d_raster, P.n_raster);
  }
  if (branch)
    if (int rc = check_hip(hipEventRecord(join, side), "batch join")) return rc;
  hipLaunchKernelGGL(batch_bins_kernel, dim3(P.n_items), dim3(256), 0, s, P.d_items);
  if (P.n_conf)
    hipLaunchKernelGGL(batch_conf_kernel, dim3(P.n_conf), dim3(256), 0, s, P.d_items, P.d_conf,
                       P.n_conf);
  for (const IntegGroup &g : P.integ)
    if (g.n) launch_integ_form<0>(P, g, s);
  if (branch)
    if (int rc = check_hip(hipStreamWaitEvent(s, join, 0), "batch join")) return rc;
  return check_hip(hipGetLastError(), "batch phases");
}

}  // namespace gg
