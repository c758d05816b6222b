// Launch of the persistent chain kernel (st_chain_kernel.hpp).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "st_chain_args.h"
#include "st_internal.h"
#include "st_launch.h"

namespace st {

// Each kernel is instantiated in a source file of its own (st_chain_*.hip).
constexpr uint32_t kBf16Rows = (1u << ST_DT_BF16) | kHasRows | kHasPools;
static const void* kernel_for(uint32_t needs, bool columns) {
  if ((needs & ~kBf16Rows) == 0u) return columns ? chain_kernel<kBf16Rows, true>() : chain_kernel<kBf16Rows, false>();
  return columns ? chain_kernel<kHasEverything, true>() : chain_kernel<kHasEverything, false>();
}

int chain_max_workgroups(int* out_workgroups, int* out_xcds) {
  int dev = 0, per_cu = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, dev);
  if (e != hipSuccess) return (int)e;
  e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel_for(kHasEverything, true), kThreads, 0);      // (every chain kernel is compiled for the same occupancy)
  if (e != hipSuccess) return (int)e;
  if (per_cu < 1) per_cu = 1;
  *out_workgroups = per_cu * prop.multiProcessorCount;
  // an XCD has 32 compute units; a whole MI355X shows 256 of them (8 XCDs), a partition of it fewer
  *out_xcds = prop.multiProcessorCount / (kNumCUs / kNumXCDs);
  return 0;
}

int launch_chain(uint32_t needs, const TenantDev* ops_dev, const st_work_item* items_dev, uint32_t n_items, const uint32_t* colbegin_dev, const ChainDep* deps_dev, uint32_t n_queues, const ChainPrefetch* prefetch_dev,
                 const uint32_t* prefetch_begin, uint32_t* ctl, uint32_t* ctl_other, uint32_t ctl_slots, uint32_t* item_flags, uint32_t run_number,
                 uint32_t spin_limit_ticks, uint32_t flags, int grid, void* stream, uint64_t* prof_dev) {
  if (n_queues != 1u && n_queues != (uint32_t)kNumXCDs) return (int)hipErrorInvalidValue;
  if (grid <= 0 || n_items == 0u) return 0;
  if (((flags & kChainFlagLocalFlags) != 0u) != (n_queues > 1u)) return (int)hipErrorInvalidValue;
  if (n_queues > 1u && (item_flags == nullptr || run_number == 0u || colbegin_dev == nullptr || deps_dev == nullptr)) return (int)hipErrorInvalidValue;
  ChainArgs a;
  a.ops = ops_dev;
  a.items = items_dev;
  a.ctl = ctl;
  a.ctl_other = ctl_other;
  a.prof = prof_dev;
  a.item_flags = item_flags;
  a.run_number = run_number;
  a.ctl_slots = ctl_slots;
  a.spin_limit = spin_limit_ticks;
  a.flags = flags;
  a.n_queues = n_queues;
  a.q_end = n_items;
  a.colbegin = colbegin_dev;
  a.deps = deps_dev;
  a.prefetch = prefetch_dev;
  for (int x = 0; x <= kNumXCDs; ++x) a.prefetch_begin[x] = prefetch_dev ? prefetch_begin[x] : 0u;
  void* addresses[] = {(void*)&a, nullptr};
  return (int)hipLaunchKernel(kernel_for(needs, n_queues > 1u), dim3((unsigned)grid), dim3(kThreads), addresses, 0, (hipStream_t)stream);
}

// What a captured run needs to start from: its control block as the run before would have left it, and no flag set.
__global__ __launch_bounds__(256) void st_chain_reset_kernel(uint32_t* ctl, uint32_t ctl_slots, uint32_t* item_flags, uint32_t n_flags) {
  const uint32_t first = blockIdx.x * 256u + threadIdx.x, step = gridDim.x * 256u;
  for (uint32_t i = first; i < ctl_slots; i += step)
    if (i == (uint32_t)kChainCtlAbort || i >= (uint32_t)kChainCtlHead) ctl[i * kChainCtlStride] = 0u;
  for (uint32_t i = first; i < (uint32_t)kChainRankWords; i += step) ctl[ctl_slots * kChainCtlStride + i] = 0u;
  for (uint32_t i = first; i < n_flags; i += step) item_flags[i] = 0u;
}

int launch_chain_reset(uint32_t* ctl, uint32_t ctl_slots, uint32_t* item_flags, uint32_t n_flags, void* stream) {
  const uint32_t n = n_flags > (uint32_t)kChainRankWords ? n_flags : (uint32_t)kChainRankWords;      // (at most 4116 slots)
  const unsigned blocks = (n + 255u) / 256u < 256u ? (n + 255u) / 256u : 256u;
  return (int)launch(st_chain_reset_kernel, blocks, 256, stream, ctl, ctl_slots, item_flags, n_flags);
}

}  // namespace st
