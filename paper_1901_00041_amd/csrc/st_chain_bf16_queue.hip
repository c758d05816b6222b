// st_chain_kernel for chains of bf16 vector, patch and row tiles (and max-pools), with one queue.
#include "st_chain_kernel.hpp"

template const void* st::chain_kernel<(1u << ST_DT_BF16) | st::kHasRows | st::kHasPools, false>();
