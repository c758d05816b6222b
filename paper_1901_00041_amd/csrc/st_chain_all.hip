// st_chain_kernel for any chain, laid out per XCD.
#include "st_chain_kernel.hpp"

template const void* st::chain_kernel<st::kHasEverything, true>();
