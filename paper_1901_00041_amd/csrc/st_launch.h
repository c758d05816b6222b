// Kernel launches of the library (device sources only).
#pragma once
#include <hip/hip_runtime.h>

namespace st {

template <class T> struct ParamType { typedef T type; };

// Queues `kernel` and returns the launch's own error code.  hipGetLastError after a launch would also report, and clear,
// whatever failed before it on this thread: in an earlier call of this library or in any other user of the runtime.
template <class... P>
inline hipError_t launch(void (*kernel)(P...), unsigned blocks, unsigned threads, void* stream, typename ParamType<P>::type... args) {
  void* addresses[] = {(void*)&args..., nullptr};
  return hipLaunchKernel((const void*)kernel, dim3(blocks), dim3(threads), addresses, 0, (hipStream_t)stream);
}

}  // namespace st
