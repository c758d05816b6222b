// st_conv_kernel for launches of every type and form.
#include "st_conv_kernel.hpp"

template int st::launch_conv_kernel<st::kHasEverything>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
