// The super-kernel of Section 4: one launch serves every tenant.  Workgroup b reads work item b, which names its tile code and
// its tenant, and computes one output tile (or one split-K slice of it) of that tenant's layer with the tile code of
// st_tiles.hpp.  Included by one source file per kernel, which are compiled side by side.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "st_internal.h"
#include "st_launch.h"
#include "st_tiles.hpp"

namespace st {

template <uint32_t HAS>
__global__ __launch_bounds__(kThreads, 2) void st_conv_kernel(const TenantDev* __restrict__ tenants,
                                                          const st_work_item* __restrict__ items,
                                                          uint64_t* __restrict__ prof_base) {
  __shared__ __attribute__((aligned(16))) char smem[kSmemBytes];
  ConstItem* ip = (ConstItem*)(items + blockIdx.x);
  st_work_item it;
  it.tenant = ip->tenant;
  it.k_split_idx = ip->k_split_idx;
  it.tile_m = ip->tile_m;
  it.tile_n = ip->tile_n;
  it.reserved = ip->reserved;
  ConstOp& T = *(ConstOp*)(tenants + it.tenant);
  uint64_t* prof = prof_base ? prof_base + (size_t)blockIdx.x * kProfSlots : nullptr;
  run_item<HAS, std::conditional_t<(HAS & kHasGather) != 0u, RaggedActs, PlainActs>>(T, it, smem, prof);
}

template <uint32_t HAS>
int launch_conv_kernel(const TenantDev* tenants_dev, const st_work_item* items_dev, int64_t n_items, void* stream, uint64_t* prof_dev) {
  return (int)launch(st_conv_kernel<HAS>, (unsigned)n_items, kThreads, stream, tenants_dev, items_dev, prof_dev);
}

}  // namespace st
