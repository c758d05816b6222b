// st_conv_kernel for launches of fp32 vector tiles.
#include "st_conv_kernel.hpp"

template int st::launch_conv_kernel<1u << ST_DT_F32>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
