// st_conv_kernel for launches of bf16 with the row tile and max-pools.
#include "st_conv_kernel.hpp"

template int st::launch_conv_kernel<(1u << ST_DT_BF16) | st::kHasRows | st::kHasPools>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
