// Kernels of the fused multi-tenant convolution launch for gfx950 (MI355X) and their launchers.
//
// One launch serves every tenant (the "super-kernel" of Section 4): workgroup b reads work item b, looks up its
// tenant record with scalar loads, and computes one output tile (or one split-K slice of it) of that tenant's layer
// with the tile code of st_tiles.hpp.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <mutex>
#include <utility>

#include "st_internal.h"
#include "st_launch.h"
#include "st_tiles.hpp"

// Fixed scratch memory for the entry point that allocates nothing (st_conv_run_noalloc).  One array per GPU, held
// from the moment the code object is loaded on that GPU until the process ends.  Host code never uses the array's
// name as an address: the device address is looked up once per device (st::noalloc_scratch) and kept.
static __device__ __align__(256) unsigned char scratch[st::kNoallocScratchBytes];

namespace st {

__global__ void st_empty_kernel() {}

// NHWC max-pool of 16-byte channel vectors, tensors below 2^31 bytes: one thread per vector of the output, nine taps in flight
// (maxpool_vector).  Bound by memory; 16 images of 112x112x64: 10.5 us with one tap after another and 64-bit
// divisions, 9.25 so; inside a chain of eight networks of batch 8 the whole pass 1130 us -> 1108.
template <int DT>
__global__ __launch_bounds__(256) void st_maxpool_vector_kernel(const void* __restrict__ x, void* __restrict__ y, uint32_t x_bytes, uint32_t total,
                                                                int H, int W, int C, int P, int Q, int win, int stride, int pad) {
  const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
  if (idx < total) ((u32x4*)y)[idx] = maxpool_vector<DT, 0>(x, x_bytes, idx, H, W, C, P, Q, win, stride, pad);
}

// NHWC max-pool; padding never wins.  One thread per (output pixel, group of VEC channels): the window's
// 16-byte channel vectors are loaded whole.  VEC = 1 is the fallback for channel counts that are not a
// multiple of the vector width.
template <int DT, int VEC>
__global__ __launch_bounds__(256) void st_maxpool_kernel(const void* __restrict__ xv, void* __restrict__ yv, int N, int H,
                                                         int W, int C, int P, int Q, int win, int stride, int pad) {
  constexpr int ES = (DT == ST_DT_F32) ? 4 : 2;
  const int CV = C / VEC;
  const int64_t total = (int64_t)N * P * Q * CV;
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= total) return;
  const int cv = (int)(idx % CV);
  int64_t t = idx / CV;
  const int q = (int)(t % Q);
  t /= Q;
  const int p = (int)(t % P);
  const int n = (int)(t / P);
  float best[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) best[e] = -__builtin_inff();
  uint32_t bits[VEC];      // bit pattern of the current maximum, so the result is copied, not re-rounded
#pragma unroll
  for (int e = 0; e < VEC; ++e) bits[e] = 0u;
  bool any = false;
  for (int r = 0; r < win; ++r) {
    const int h = p * stride - pad + r;
    if ((unsigned)h >= (unsigned)H) continue;
    for (int s = 0; s < win; ++s) {
      const int w = q * stride - pad + s;
      if ((unsigned)w >= (unsigned)W) continue;
      const char* src = (const char*)xv + ((((int64_t)n * H + h) * W + w) * C + (int64_t)cv * VEC) * ES;
      uint32_t raw[VEC * ES / 4 > 0 ? VEC * ES / 4 : 1];
      if constexpr (VEC * ES == 16) {
        const u32x4 v = *(const u32x4*)src;
        raw[0] = v[0]; raw[1] = v[1]; raw[2] = v[2]; raw[3] = v[3];
      } else if constexpr (ES == 4) {
        raw[0] = *(const uint32_t*)src;
      } else {
        raw[0] = *(const uint16_t*)src;
      }
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        uint32_t b;
        float v;
        if constexpr (ES == 4) {
          b = raw[e];
          v = __builtin_bit_cast(float, b);
        } else {
          b = (raw[e >> 1] >> (16 * (e & 1))) & 0xffffu;
          v = (DT == ST_DT_BF16) ? bf16_bits_to_f32((uint16_t)b) : f16_bits_to_f32((uint16_t)b);
        }
        if (!any || v > best[e]) { best[e] = v; bits[e] = b; }
      }
      any = true;
    }
  }
  char* dst = (char*)yv + idx * (int64_t)(VEC * ES);
  if constexpr (VEC * ES == 16) {
    u32x4 o;
    if constexpr (ES == 4) { o = u32x4{bits[0], bits[1], bits[2], bits[3]}; }
    else { o = u32x4{bits[0] | (bits[1] << 16), bits[2] | (bits[3] << 16), bits[4] | (bits[5] << 16), bits[6] | (bits[7] << 16)}; }
    *(u32x4*)dst = o;
  } else if constexpr (ES == 4) {
    *(uint32_t*)dst = bits[0];
  } else {
    *(uint16_t*)dst = (uint16_t)bits[0];
  }
}

// Each kernel is instantiated in a source file of its own (st_conv_*.hip).
extern template int launch_conv_kernel<1u << ST_DT_BF16>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
extern template int launch_conv_kernel<1u << ST_DT_F16>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
extern template int launch_conv_kernel<1u << ST_DT_F32>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
extern template int launch_conv_kernel<(1u << ST_DT_BF16) | kHasRows | kHasPools>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);
extern template int launch_conv_kernel<kHasEverything>(const TenantDev*, const st_work_item*, int64_t, void*, uint64_t*);

int launch_conv(uint32_t needs, const TenantDev* tenants_dev, const st_work_item* items_dev, int64_t n_items, void* stream,
                uint64_t* prof_dev) {
  if (n_items <= 0) return 0;
  const auto fits = [=](uint32_t has) { return (needs & ~has) == 0u; };
  constexpr uint32_t kBf16 = 1u << ST_DT_BF16, kF16 = 1u << ST_DT_F16, kF32 = 1u << ST_DT_F32, kBf16Rows = kBf16 | kHasRows | kHasPools;
  const auto run = fits(kBf16)       ? launch_conv_kernel<kBf16>
                   : fits(kF16)      ? launch_conv_kernel<kF16>
                   : fits(kF32)      ? launch_conv_kernel<kF32>
                   : fits(kBf16Rows) ? launch_conv_kernel<kBf16Rows>
                                     : launch_conv_kernel<kHasEverything>;
  return run(tenants_dev, items_dev, n_items, stream, prof_dev);
}

// Plain 16-byte-per-lane copy: the reference kernel for scaling hardware traffic counters.
__global__ __launch_bounds__(256) void st_copy_kernel(const u32x4* __restrict__ src, u32x4* __restrict__ dst, int64_t n16) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (int64_t)gridDim.x * blockDim.x) dst[i] = src[i];
}

int launch_copy(const void* src, void* dst, int64_t bytes, void* stream) {
  const int64_t n16 = bytes / 16;
  if (n16 <= 0) return 0;
  const unsigned blocks = (unsigned)((n16 + 255) / 256 < 8192 ? (n16 + 255) / 256 : 8192);
  return (int)launch(st_copy_kernel, blocks, 256, stream, (const u32x4*)src, (u32x4*)dst, n16);
}

// ---- the entry point that allocates nothing: tables and split-K workspace in the fixed array `scratch` -------
namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Bytes that travel to the device inside the kernel arguments (a launch copies its arguments when it is issued, so
// the host buffer is free again as soon as the launch call returns, and no copy routine is involved).
constexpr int kPokeVecs = 224;                       // 3584 bytes per launch
struct PokePayload { u32x4 v[kPokeVecs]; };
}  // namespace

__global__ __launch_bounds__(256) void st_poke_kernel(PokePayload p, u32x4* __restrict__ dst, int nvec) {
  const int i = threadIdx.x;
  if (i < nvec) dst[i] = p.v[i];
}

// New tensor pointers for a plan's tenants, in stream order.  As a launch the update costs about what any launch costs;
// as a copy from pinned memory it took a copy routine with its barriers, and an event for every reuse of the memory (a
// step of 8 arriving tenants 13.4 -> 9.7 us).  The payload is copied with the arguments, so there is a small form too.
constexpr int kBindSmall = 16, kBindLarge = 112;
template <int N>
struct BindPayload { u32x4 v[2 * N]; };
static_assert(offsetof(TenantDev, x) == 0 && offsetof(TenantDev, res) == 24, "the pointers are a record's first 32 bytes");

template <int N>
__global__ __launch_bounds__(256) void st_bind_kernel(BindPayload<N> p, TenantDev* __restrict__ table, int n) {
  const int i = threadIdx.x;
  if (i < 2 * n) ((u32x4*)(table + (i >> 1)))[i & 1] = p.v[i];
}

template <int N>
static hipError_t bind(const TenantDev* host, int n, TenantDev* table, void* stream) {
  BindPayload<N> p;
  for (int i = 0; i < n; ++i) std::memcpy(&p.v[2 * i], host + i, 32);
  std::memset(&p.v[2 * n], 0, (size_t)(N - n) * 32);
  return launch(st_bind_kernel<N>, 1, 256, stream, p, table, n);
}

int launch_bind(const TenantDev* host, int n, TenantDev* table_dev, void* stream) {
  for (int done = 0; done < n; done += kBindLarge) {
    const int m = n - done < kBindLarge ? n - done : kBindLarge;
    const hipError_t e = m <= kBindSmall ? bind<kBindSmall>(host + done, m, table_dev + done, stream) : bind<kBindLarge>(host + done, m, table_dev + done, stream);
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}

__global__ __launch_bounds__(256) void st_zero_kernel(u32x4* __restrict__ dst, int64_t nvec) {
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec; i += (int64_t)gridDim.x * blockDim.x) dst[i] = z;
}

int noalloc_scratch(void** out_ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(::scratch));     // this device's copy of the array (the current device's)
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out_ptr = g_scratch_ptr[dev];
  return 0;
}

int launch_poke(const void* host_src, int64_t bytes, void* dst_dev, void* stream) {
  const char* src = (const char*)host_src;
  char* dst = (char*)dst_dev;
  PokePayload p;
  for (int64_t done = 0; done < bytes; done += (int64_t)sizeof(PokePayload)) {
    const int64_t n = bytes - done < (int64_t)sizeof(PokePayload) ? bytes - done : (int64_t)sizeof(PokePayload);
    std::memset(&p, 0, sizeof(p));
    std::memcpy(&p, src + done, (size_t)n);
    const hipError_t e = launch(st_poke_kernel, 1, 256, stream, p, (u32x4*)(dst + done), (int)((n + 15) / 16));
    if (e != hipSuccess) return (int)e;
  }
  return 0;
}

int launch_zero(void* dst_dev, int64_t bytes, void* stream) {
  const int64_t nvec = (bytes + 15) / 16;
  if (nvec <= 0) return 0;
  const unsigned blocks = (unsigned)((nvec + 255) / 256 < 1024 ? (nvec + 255) / 256 : 1024);
  return (int)launch(st_zero_kernel, blocks, 256, stream, (u32x4*)dst_dev, nvec);
}

int launch_empty(void* stream) {
  return (int)launch(st_empty_kernel, 1, 64, stream);
}

int launch_maxpool(const void* x, void* y, int N, int H, int W, int C, int P, int Q, int win, int stride, int pad,
                   int dtype, void* stream) {
  const int es = dtype == ST_DT_F32 ? 4 : 2;
  const int vec = (C % (16 / es) == 0) ? 16 / es : 1;
  const int64_t total = (int64_t)N * P * Q * (C / vec);
  if (total <= 0) return 0;
  const unsigned blocks = (unsigned)((total + 255) / 256);
  const int64_t x_bytes = (int64_t)N * H * W * C * es;
  if (vec > 1 && x_bytes < ((int64_t)1 << 31) && total * 16 < ((int64_t)1 << 31)) {
    auto kernel = dtype == ST_DT_F32 ? st_maxpool_vector_kernel<ST_DT_F32> : dtype == ST_DT_BF16 ? st_maxpool_vector_kernel<ST_DT_BF16> : st_maxpool_vector_kernel<ST_DT_F16>;
    return (int)launch(kernel, blocks, 256, stream, x, y, (uint32_t)x_bytes, (uint32_t)total, H, W, C, P, Q, win, stride, pad);
  }
  auto kernel = dtype == ST_DT_F32    ? (vec == 4 ? st_maxpool_kernel<ST_DT_F32, 4> : st_maxpool_kernel<ST_DT_F32, 1>)
                : dtype == ST_DT_BF16 ? (vec == 8 ? st_maxpool_kernel<ST_DT_BF16, 8> : st_maxpool_kernel<ST_DT_BF16, 1>)
                                      : (vec == 8 ? st_maxpool_kernel<ST_DT_F16, 8> : st_maxpool_kernel<ST_DT_F16, 1>);
  return (int)launch(kernel, blocks, 256, stream, x, y, N, H, W, C, P, Q, win, stride, pad);
}

}  // namespace st
