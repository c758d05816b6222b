// Arguments of the persistent chain kernel.
#pragma once
#include <stdint.h>

#include "st_internal.h"

namespace st {

struct ChainArgs {
  const TenantDev* ops;
  const st_work_item* items;
  uint32_t* ctl;          // this run's control block
  uint32_t* ctl_other;    // the next run's: cleared by workgroup 0
  uint64_t* prof;         // kProfSlots stamps per queue entry, or nullptr
  uint32_t* item_flags;   // kChainFlagLocalFlags: one completion flag per work item, holding the number of the run that set it
  uint32_t run_number;    // this run's number (never 0)
  uint32_t ctl_slots;     // 256-byte slots of a control block (one live word each); kChainRankWords dense words follow them
  uint32_t spin_limit;    // ticks of the 100 MHz constant clock a dependency wait may last
  uint32_t flags;         // kChainFlag*
  uint32_t n_queues;      // 1: one queue for the whole chip, entries claimed one by one; kNumXCDs: columns (see st_chain_kernel)
  uint32_t q_end;         // one queue: it is items[0 .. q_end)
  const ChainPrefetch* prefetch;      // columns: XCD x's filters in stage order are prefetch[prefetch_begin[x] .. prefetch_begin[x + 1])
  uint32_t prefetch_begin[kNumXCDs + 1];
  const uint32_t* colbegin;   // columns: column j of XCD x is items[colbegin[x * 2 * kChainColumns + j] .. colbegin[.. + j + 1])
  const ChainDep* deps;       // columns: beside every entry of items
};

// The kernel compiled for HAS, to launch with one ChainArgs.
template <uint32_t HAS, bool COLUMNS> const void* chain_kernel();
extern template const void* chain_kernel<(1u << ST_DT_BF16) | kHasRows | kHasPools, false>();
extern template const void* chain_kernel<(1u << ST_DT_BF16) | kHasRows | kHasPools, true>();
extern template const void* chain_kernel<kHasEverything, false>();
extern template const void* chain_kernel<kHasEverything, true>();

}  // namespace st
