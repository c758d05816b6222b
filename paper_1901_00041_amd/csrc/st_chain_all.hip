// st_chain_kernel for chains of every type and form (and max-pools).
#include "st_chain_kernel.hpp"

template const void* st::chain_kernel<st::kHasEverything>();
