// st_chain_kernel for chains of bf16 vector, patch and row tiles (and max-pools), laid out per XCD.
#include "st_chain_kernel.hpp"

template const void* st::chain_kernel<(1u << ST_DT_BF16) | st::kHasRows | st::kHasPools, true>();
