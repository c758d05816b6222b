// st_chain_kernel for any chain, with one queue.
#include "st_chain_kernel.hpp"

template const void* st::chain_kernel<st::kHasEverything, false>();
