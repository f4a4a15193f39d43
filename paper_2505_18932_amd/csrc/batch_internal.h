// Batched path: device-resident item descriptors, work lists and the plan.
#pragma once

#include <vector>

#include "splat_device.h"
#include "fuse_device.h"

namespace gg {

constexpr int kBatchConfRows = 4;  // of the confidence phase's tiles (conf_tile)

// Everything one item's phases need, in device memory (read with scalar
// loads: the descriptor address is uniform per work entry).
struct BatchItem {
  IntegrateArgs integ;
  ConfArgs conf;
  SplatArgs splat;
  float2 *bins;
  int32_t D;
  float z_near, z_far, trunc;
  int32_t trunc_in_bins;
};

// One unit of work of one phase: item, view, and a tile / block coordinate.
struct WorkItem {
  uint16_t item, k;
  uint16_t x, y;  // conf: tile (x, y); splat bin: source block x; raster / fusion: tile x
};

// Entry e of a work list, read once and made uniform: the item index then
// addresses its descriptor through the scalar unit (SGPRs), instead of a
// vector register pair held for the whole tile.
__device__ __forceinline__ WorkItem uniform_entry(const WorkItem *work, uint32_t e) {
  static_assert(sizeof(WorkItem) == 8, "WorkItem is two dwords");
  const uint2 raw = reinterpret_cast<const uint2 *>(work)[e];
  const uint32_t lo = __builtin_amdgcn_readfirstlane(raw.x);
  const uint32_t hi = __builtin_amdgcn_readfirstlane(raw.y);
  WorkItem w;
  w.item = (uint16_t)(lo & 0xffffu);
  w.k = (uint16_t)(lo >> 16);
  w.x = (uint16_t)(hi & 0xffffu);
  w.y = (uint16_t)(hi >> 16);
  return w;
}

// The fusion and raster phases address tiles beyond 65535: they use x as
// the low 16 bits and y as the high 16 bits of a 32-bit tile index.
__device__ __forceinline__ uint32_t work_tile(const WorkItem &w) {
  return (uint32_t)w.x | ((uint32_t)w.y << 16);
}

// One fusion launch of the batch: the tiles of every item of one form and
// workgroup size.
struct IntegGroup {
  int form = 0, waves = 0;
  size_t lds = 0;              // the largest of its items'
  WorkItem *list = nullptr;    // device
  uint32_t n = 0;
};

struct BatchPlan {
  int32_t n_items = 0;
  int branches = 2;  // 2: splat phases beside the fusion; 1: one sequence
  // device memory owned by the plan
  void *dev = nullptr;
  size_t dev_bytes = 0;
  BatchItem *d_items = nullptr;
  WorkItem *d_conf = nullptr, *d_bin = nullptr, *d_raster = nullptr;
  uint32_t n_conf = 0, n_bin = 0, n_raster = 0;
  std::vector<IntegGroup> integ;
  uint32_t *d_splat_items = nullptr;
  uint32_t n_splat_items = 0;
  uint32_t *zero_ptr = nullptr;  // tile counts and list allocators of every item
  size_t zero_words = 0;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

// Record every phase on s (captured into the plan's graph); with a side
// stream and the two events the splat phases become a parallel branch.
int batch_record(BatchPlan &P, hipStream_t s, hipStream_t side, hipEvent_t fork,
                 hipEvent_t join);

}  // namespace gg
