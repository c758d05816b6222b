// st_conv_kernel for launches of bf16 vector and patch tiles.
#include "st_conv_kernel.hpp"

template int st::launch_conv_kernel<1u << ST_DT_BF16>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
