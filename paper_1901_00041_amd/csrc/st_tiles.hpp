// Device code shared by the convolution kernels: MFMA wrappers, the tile epilogue, the implicit-GEMM workgroup
// tile (conv_tile), the row tile for few-channel layers (conv_tile_rows) and the per-workgroup dispatch on
// (dtype, tile shape).  Included by st_kernels.hip (one launch per plan) and st_chain.hip (one persistent launch
// over a whole chain of layers).
//
// One workgroup computes one MT x NT output tile (or one split-K slice of it) of one tenant's layer.  The layer is
// the im2col product of Section 4.1 with M = output pixels, N = filters, K = C*R*S; the patch matrix is never
// materialised: each K step gathers a [MT x KB] slab of patches and a [NT x KB] slab of filters into LDS with
// 16-byte loads (NHWC / KRSC make the reduction index channel-contiguous), and the 4 wavefronts run bf16/f16/f32
// MFMA blocks on them with fp32 accumulators.
//
// MFMA operand roles: filters are operand A (block rows), pixels operand B (block columns), so each lane ends up
// with runs of 4 consecutive filters of one pixel, which are contiguous in the NHWC output.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "st_internal.h"

namespace st {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// Records and work items that no launch in flight modifies: the constant address space makes every read a scalar load,
// however many stores, atomics and barriers surround it.
typedef __attribute__((address_space(4))) const st_work_item ConstItem;
typedef __attribute__((address_space(4))) const TenantDev ConstOp;

// Has the fields of a record that the start of a tile needs loaded by here, together.  Read one by one where they are first
// needed, they cost a tile eight round trips of 75 ns, most of the 1300 clocks before its first load.
__device__ __forceinline__ void tile_fields_loaded(ConstOp& T) {
  asm volatile("" ::"s"(T.x), "s"(T.w), "s"(T.x_bytes), "s"(T.w_bytes), "s"(T.C), "s"(T.H), "s"(T.W), "s"(T.K), "s"(T.R), "s"(T.S), "s"(T.stride), "s"(T.pad),
               "s"(T.Q), "s"(T.PQ), "s"(T.M), "s"(T.Kg), "s"(T.shift_pq), "s"(T.shift_q), "s"(T.magic_pq), "s"(T.magic_q), "s"(T.k_steps),
               "s"(T.k_steps_per_split), "s"(T.k_order), "s"(T.epilogue), "s"(T.out_dtype), "s"(T.split_k));
}

// The thread's index in its workgroup, read afresh wherever a work item starts.  Inside a loop over work items the
// compiler would otherwise compute everything that depends only on the thread index (lane geometry, staging rows of
// every tile shape) once before the loop and keep it alive in registers through all of it.
__device__ __forceinline__ int work_thread_id() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  __builtin_assume(t >= 0 && t < kThreads);
  return t;
}

// The stamps every work item of a profiled launch leaves (one thread calls; slots as st_conv_run_profiled documents them).
__device__ __forceinline__ void stamp_start(uint64_t* prof) {
  prof[0] = __builtin_readcyclecounter();
  prof[4] = wall_clock64();
  prof[5] = ((uint64_t)__builtin_amdgcn_s_getreg(0x1814) << 32) | (uint32_t)__builtin_amdgcn_s_getreg(0xF804);
}
__device__ __forceinline__ void stamp_end(uint64_t* prof) {
  prof[3] = __builtin_readcyclecounter();
  prof[6] = wall_clock64();
}

template <int DT> struct ElemOf;
template <> struct ElemOf<ST_DT_F32> { static constexpr int ES = 4; };
template <> struct ElemOf<ST_DT_BF16> { static constexpr int ES = 2; };
template <> struct ElemOf<ST_DT_F16> { static constexpr int ES = 2; };

// ---- MFMA wrappers: one call consumes one 16-byte K fragment per lane ----------------------------
template <int DT, int MF> struct Mma;
template <> struct Mma<ST_DT_BF16, 32> {
  typedef f32x16 Acc;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<ST_DT_F16, 32> {
  typedef f32x16 Acc;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<ST_DT_F32, 32> {
  typedef f32x16 Acc;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], c, 0, 0, 0);
    return c;
  }
};
template <> struct Mma<ST_DT_BF16, 16> {
  typedef f32x4 Acc;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<ST_DT_F16, 16> {
  typedef f32x4 Acc;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
  }
};
template <> struct Mma<ST_DT_F32, 16> {
  typedef f32x4 Acc;
  static __device__ __forceinline__ Acc run(u32x4 a, u32x4 b, Acc c) {
    f32x4 fa = __builtin_bit_cast(f32x4, a), fb = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[j], fb[j], c, 0, 0, 0);
    return c;
  }
};

// compile-time loop: f(integral_constant<int, 0>) ... f(integral_constant<int, N-1>)
template <int... Is, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, Is...>, F&& f) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, static_cast<F&&>(f));
}

// nested conditionals: if (n > 0) { f(0); if (n > 1) { f(1); ... } } up to N levels
template <int I, int N, class F>
__device__ __forceinline__ void static_nest_impl(int n, F&& f) {
  if constexpr (I < N) {
    if (n > I) {
      f(std::integral_constant<int, I>{});
      static_nest_impl<I + 1, N>(n, static_cast<F&&>(f));
    }
  }
}
template <int N, class F>
__device__ __forceinline__ void static_nest(int n, F&& f) {
  static_nest_impl<0, N>(n, static_cast<F&&>(f));
}

// ---- output conversion (fp32 to 16 bits rounds to nearest even: v_cvt_pk_bf16_f32, v_cvt_f16_f32) ----
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) {
  return __builtin_bit_cast(float, (uint32_t)b << 16);
}
__device__ __forceinline__ uint16_t f32_to_f16_bits(float f) {
  _Float16 h = (_Float16)f;
  return __builtin_bit_cast(uint16_t, h);
}
__device__ __forceinline__ float f16_bits_to_f32(uint16_t b) {
  return (float)__builtin_bit_cast(_Float16, b);
}

// v > 0 ? v : 0, also for NaN, in one instruction: the median of v, 0 and infinity, which the compiler must not know to be one (it
// makes a maximum of it, behind another one that quiets NaNs).
__device__ __forceinline__ float relu_f32(float v) {
  float inf;
  asm("s_mov_b32 %0, 0x7f800000" : "=s"(inf));
  return __builtin_amdgcn_fmed3f(v, 0.f, inf);
}

// two fp32 values rounded to nearest even, packed; DT is one of the 16-bit types
template <int DT>
__device__ __forceinline__ uint32_t pack16(float a, float b) {
  if constexpr (DT == ST_DT_BF16) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
  } else {
    return (uint32_t)f32_to_f16_bits(a) | ((uint32_t)f32_to_f16_bits(b) << 16);
  }
}
template <int DT>
__device__ __forceinline__ float unpack16(uint32_t pair, int which) {
  const uint16_t h = (uint16_t)(pair >> (16 * which));
  if constexpr (DT == ST_DT_BF16) return bf16_bits_to_f32(h);
  else return f16_bits_to_f32(h);
}

// ---- cache-coherent partial-tile traffic for split-K -------------------------------------------------
// Split-K partial tiles travel between workgroups that may sit on different XCDs, whose L2 caches are
// not coherent with each other.  Instead of fences that write back and invalidate a whole L2, the
// partials themselves are stored and loaded with device-scope coherence (sc1: write through / miss
// always), so the only ordering needed is "my stores have completed" before the arrival counter is
// bumped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
constexpr int kAuxDeviceCoherent = 16;   // sc1
// How a tile reads activations (x and the residual): what another kernel wrote before this launch can be read
// through the caches (PlainActs); what other workgroups of the SAME launch write (the chain kernel) must be read
// with device-scope loads, which never stop at the compute unit's vector cache and take from the L2 only what that
// L2 itself holds newer than memory (CoherentActs).  Outputs are stored write-through (a launch per layer: they leave the L2
// while the kernel still runs, see tile_epilogue), unless everyone who reads them during the launch shares the L2
// (LocalActs: a chain laid out per XCD; the same goes for split-K partial tiles and their counters); filters never change
// during a launch and always go through the caches.
// kAnyFilters: whole vectors are stored for filter counts off the vector width, too (see tile_epilogue).
struct PlainActs { static constexpr int kActAux = 0, kOutAux = kAuxDeviceCoherent; static constexpr bool kOneL2 = false, kAnyFilters = false; };
struct RaggedActs : PlainActs { static constexpr bool kAnyFilters = true; };
struct CoherentActs { static constexpr int kActAux = kAuxDeviceCoherent, kOutAux = kAuxDeviceCoherent; static constexpr bool kOneL2 = false, kAnyFilters = false; };
struct LocalActs { static constexpr int kActAux = kAuxDeviceCoherent, kOutAux = 0; static constexpr bool kOneL2 = true, kAnyFilters = false; };

// floor(n / d) for 0 <= n < 2^31 with the planner's multiplier m = floor(2^(31+L)/d)+1, L = ceil(log2 d)
__device__ __forceinline__ int fast_div(int n, uint32_t m, int L) {
  return (int)(__umulhi((uint32_t)n << 1, m) >> L);      // the upper half of 2n * m: one multiplication, where n * m takes two
}

constexpr uint32_t kInvalidOffset = 0x80000000u;   // >= num_records of every buffer: the load returns 0
// Offsets of a tile's output and residual rows, each the one before plus a launch constant.  Rows past the last pixel are not compared
// with it but left to the tensor's end, so the sum stops at kPastEnd (a tensor is shorter than 2^31 bytes) instead of coming
// round into the tensor, however long the rows; the addition that saturates is one instruction like the other.
constexpr int kPastEnd = 0x7fffffff;
__device__ __forceinline__ int next_row(int off, int turn) { return __builtin_elementwise_add_sat(off, turn); }
template <int BYTES>                                             // BYTES times the number of filters (uniform)
__device__ __forceinline__ int row_turn(int filters) { return filters <= kPastEnd / BYTES ? filters * BYTES : kPastEnd; }

// ---- memory to LDS without registers -------------------------------------------------------------
// One instruction moves 16 bytes per lane from a buffer straight into LDS: lane l's bytes land at lds_base + 16 * l
// (lds_base is wave-uniform), lanes whose offset is out of range write zeros.  The compiler is not told about the LDS
// write: whoever reads the data first waits for the vector-memory counter (wait_loads_barrier) and for a barrier.
// (M0 is reserved: the compiler sets it right before each use of its own, and warns that an asm statement writes it.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int AUX, int OFF>
__device__ __forceinline__ void load_to_lds(const u32x4& rsrc, uint32_t voff, uint32_t soff, uint32_t lds_base) {   // to lds_base + OFF
  static_assert(AUX == 0 || AUX == kAuxDeviceCoherent, "cache policy");
  if constexpr (AUX == 0)
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff), "i"(OFF) : "memory", "scc", "m0");
  else
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen sc1 lds" ::"s"(lds_base), "v"(voff), "s"(rsrc), "s"(soff), "i"(OFF) : "memory", "scc", "m0");
}
#pragma clang diagnostic pop
// Waits until at most N of this wavefront's loads are outstanding and all its LDS reads are done, then for the other
// wavefronts to get there.
template <int N>
__device__ __forceinline__ void wait_loads_barrier() {
  static_assert(N >= 0 && N < 64, "the vector-memory counter has six bits");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory");
}
template <int MAXS, int PER>
__device__ __forceinline__ void wait_steps_barrier(int steps) {   // all but the `steps` most recent K steps have arrived
  if constexpr (MAXS <= 0) wait_loads_barrier<0>();
  else {
    if (steps >= MAXS) wait_loads_barrier<MAXS * PER>();
    else wait_steps_barrier<MAXS - 1, PER>(steps);
  }
}
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes) {
  const uint64_t a = (uint64_t)(uintptr_t)base;
  return u32x4{(uint32_t)a, (uint32_t)(a >> 32), bytes, 0x00020000u};
}

// LDS copy of a 16-bit residual tile, [pixel][filter] in rows of NT * 2 bytes: 16-byte chunk c of row r sits at position
// c ^ residual_swizzle(r), which spreads the 8-byte reads of 16 pixels over the banks.
template <int NT>
__device__ __forceinline__ int residual_swizzle(int row) {
  static_assert(NT == 64 || NT == 128, "residual rows of 128 or 256 bytes");
  return NT == 128 ? (row & 15) : ((row >> 1) & 7);
}
// Load instructions per wavefront that stage_residual issues.
template <int MT, int NT> constexpr int kResidualLoads = (MT * NT * 2 + 4095) / 4096;
// Puts the residual tile's loads in flight, to LDS offset lds_base (of this wavefront: + 1024 * wave); needs
// kResidualLoads * 4096 bytes there.
template <int MT, int NT, class POL>
__device__ __forceinline__ void stage_residual(ConstOp& T, int m0, int n0, int wave, int lane, uint32_t lds_base) {
  constexpr int CH = NT / 8, RPI = 64 / CH;
  const u32x4 rr = rsrc_words(T.res, T.y_bytes);
  // rows 4 * RPI apart have the same swizzle
  const int row0 = wave * RPI + lane / CH, ch = n0 + ((lane % CH) ^ residual_swizzle<NT>(row0)) * 8, turn = row_turn<4 * RPI * 2>(T.K);
  int off = (ch < T.K) & (m0 + row0 < T.M) ? (int)(((uint32_t)(m0 + row0) * (uint32_t)T.K + (uint32_t)ch) * 2u) : kPastEnd;
  static_for<kResidualLoads<MT, NT>>([&](auto I) {
    constexpr int i = decltype(I)::value;
    const bool ok = (i + 1) * 4 * RPI <= MT || i * 4 * RPI + row0 < MT;
    load_to_lds<POL::kActAux, i * 4096>(rr, (uint32_t)(ok ? off : kPastEnd), 0u, lds_base);
    off = next_row(off, turn);
  });
}

// ---- epilogue shared by all tile kernels: (+ residual) -> ReLU -> cast -> store ---------------------
// The transposed output rows are stored write-through (sc1), so they leave the L2 while the kernel still runs
// instead of waiting in it for the write-back at the end of the kernel, which the next launch on the stream
// would have to sit through.
// acc[i][j] is the MF x MF block at pixels wm0 + i*MF, filters wn0 + j*MF of the tile whose first pixel is
// im2col row m0 and first filter n0; rows at or past m_end are not stored.
// The transposition buffer `smem` holds MT/PASSES pixel rows; with PASSES > 1 the tile is written out in
// that many slices of consecutive pixel rows.
// DT is the operands' type: 16-bit outputs have the operands' type (out_dtype is fp32 or in_dtype).
// What bounds it, beside the two barriers, is the number of vector instructions: two wavefronts share a SIMD, so each costs a
// wavefront eight clocks.  ReLU in one instruction and only where asked for, and offsets by adding, took a third of them away
// (128x128 with a residual: 360 -> 230; eight networks of batch 1 as a chain 334.5 us -> 325, four of batch 4 as launches 532 -> 520).
// res_lds >= 0: the tile of a 16-bit residual is on its way to smem + res_lds (stage_residual); else a residual is loaded
// here, where its latency is in the open (128x128 tile, bf16, alone on its compute unit, clocks from the last MFMA to the last store:
// 7900 with the residual loaded here, 4500 with it staged, 3070 since a third of the instructions went; without a residual 5700,
// 3400 with packed conversions, now 1840; ReLU 240 more).
// TO_END: m_end is the number of pixels (rows past it lie past the tensor's end, which no store gets beyond).
template <int MT, int NT, int BM, int BN, int MF, int DT, int PASSES = 1, int CAP = kSmemBytes, class POL = PlainActs, bool TO_END = true, class Acc>
__device__ __forceinline__ void tile_epilogue(ConstOp& T, Acc (&acc)[BM][BN], int m0, int m_end, int n0, int wm0,
                                              int wn0, int lrow, int lk, int tid, char* smem, int res_lds = -1) {
  constexpr int NG = (MF == 32) ? 4 : 1;
  const bool relu = (T.epilogue & ST_EPI_RELU) != 0u;
  const bool has_res = (T.epilogue & ST_EPI_RESIDUAL) != 0u;
  const int Kf = T.K;
  const bool vec4 = (Kf & 3) == 0, whole = (Kf & 7) == 0;
  // Any number of filters: a row of the output is still mostly whole vectors (at element-aligned addresses); what is left of
  // it is stored element by element, by the lanes that hold it.  (With stores per lane and element instead, four of 2 bytes for
  // every four filters of a pixel, a 128x64 tile of 201 filters spent 9900 clocks after its last MFMA.)  Not with a
  // residual, not in row tiles, and only in the kernel for everything: the second way out costs other launches 2-3 % (16
  // unlike tenants 40.1 -> 41.2 us).
  constexpr bool kAnyFilters = POL::kAnyFilters && PASSES == 1;
  const bool rest = kAnyFilters && !whole && n0 + NT > Kf;       // this tile holds the end of the rows
  bool done16 = false;
  if constexpr (DT != ST_DT_F32) {
   if (T.out_dtype != ST_DT_F32 && (has_res ? whole && res_lds >= 0 : whole || kAnyFilters)) {
    // 16-bit output: the residual (if any, staged in LDS) is added to the accumulators, ReLU and the rounding are applied
    // to them, and the transposition buffer holds the finished 16-bit values, [pixel][filter], the whole tile at once.
    // Every lane then moves 16 bytes of one output row from LDS to memory.
    done16 = true;
    constexpr int PITCHB = NT * 2 + 16;   // bytes per pixel row; the pad spreads the 8-byte writes of 8 pixels over the banks
    static_assert(MT * PITCHB <= CAP, "16-bit output tile does not fit the transposition buffer");
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(T.y, T.y_bytes);
    if (has_res) {
      wait_loads_barrier<0>();
      const char* rs = smem + res_lds;
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j)
#pragma unroll
          for (int g = 0; g < NG; ++g) {
            const int row = wm0 + i * MF + lrow;
            const int chl = wn0 + j * MF + ((MF == 32) ? (8 * g + 4 * lk) : (4 * lk));
            const uint2 r = *(const uint2*)(rs + row * (NT * 2) + (((chl >> 3) ^ residual_swizzle<NT>(row)) << 4) + (chl & 4) * 2);
            acc[i][j][4 * g + 0] += unpack16<DT>(r.x, 0);
            acc[i][j][4 * g + 1] += unpack16<DT>(r.x, 1);
            acc[i][j][4 * g + 2] += unpack16<DT>(r.y, 0);
            acc[i][j][4 * g + 3] += unpack16<DT>(r.y, 1);
          }
    }
    if (relu) {
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j)
#pragma unroll
          for (int v = 0; v < 4 * NG; ++v) acc[i][j][v] = relu_f32(acc[i][j][v]);
    }
    __syncthreads();                // the buffer (operands, residual, or the previous tile) is no longer read
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const int row = wm0 + i * MF + lrow;
          const int chl = wn0 + j * MF + ((MF == 32) ? (8 * g + 4 * lk) : (4 * lk));
          uint2 pk;
          pk.x = pack16<DT>(acc[i][j][4 * g], acc[i][j][4 * g + 1]);
          pk.y = pack16<DT>(acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]);
          *(uint2*)(smem + row * PITCHB + chl * 2) = pk;
        }
    __syncthreads();
    constexpr int NV = NT / 8, ROWS = kThreads / NV;      // vectors of a row; rows stored at a time
    constexpr int IT = (MT + ROWS - 1) / ROWS;
    const int row0 = tid / NV, cv = tid % NV, ch = n0 + cv * 8, turn = row_turn<ROWS * 2>(Kf);
    auto store_rows = [&](auto REST) {       // REST: with the end of the rows
    int at = (ch < Kf) & (m0 + row0 < m_end) ? (int)(((uint32_t)(m0 + row0) * (uint32_t)Kf + (uint32_t)ch) * 2u) : kPastEnd;
#pragma unroll
    for (int u = 0; u < IT; ++u, at = next_row(at, turn)) {
      const int row = row0 + u * ROWS;
      const bool ok = ((u + 1) * ROWS <= MT || row < MT) & (TO_END || m0 + row < m_end) & (!decltype(REST)::value || ((m0 + row < m_end) & (ch < Kf)));
      const int off = ok ? at : kPastEnd;
      const u32x4 d = *(const u32x4*)(smem + (row < MT ? row : 0) * PITCHB + cv * 16);
      if constexpr (!decltype(REST)::value) {
        __builtin_amdgcn_raw_buffer_store_b128(d, ry, off, 0, POL::kOutAux);
      } else if (ok) {
        if (ch + 8 <= Kf) {
          __builtin_amdgcn_raw_buffer_store_b128(d, ry, off, 0, POL::kOutAux);
        } else {
#pragma unroll
          for (int e = 0; e < 7; ++e)
            if (ch + e < Kf) __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(d[e >> 1] >> (16 * (e & 1))), ry, off + 2 * e, 0, POL::kOutAux);
        }
      }
    }
    };
    if constexpr (kAnyFilters) {
      if (rest) store_rows(std::true_type{});
      else store_rows(std::false_type{});
    } else {
      store_rows(std::false_type{});
    }
   }
  }
  if (done16) return;
  if (whole || (kAnyFilters && !has_res && T.out_dtype == ST_DT_F32)) {
    // Transpose through LDS: accumulators go to an fp32 [pixel][filter] tile, then every lane handles 16
    // bytes of one output row, so residual loads and output stores are whole contiguous rows.
    constexpr int PITCH = NT + 4;   // floats; the pad keeps the 16-byte writes of 16 pixels on distinct banks
    constexpr int MP = MT / PASSES; // pixel rows per slice
    static_assert(MT % PASSES == 0 && MP % MF == 0, "slices must hold whole MFMA blocks");
    static_assert(MP * PITCH * 4 <= CAP, "output tile does not fit the transposition buffer");
    float* sC = (float*)smem;
    const __amdgpu_buffer_rsrc_t ry = make_rsrc(T.y, T.y_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(has_res ? T.res : T.y, T.y_bytes);
    // Residual vectors are requested before the accumulators are staged, so their latency overlaps the
    // transposition (single-slice tiles only).
    // Offset of the thread's first vector of slice `pass`, and from one of its rows to the next (ES: bytes of an element).
    auto first_row = [&](auto ES, int pass) -> int {
      constexpr int es = decltype(ES)::value, nv = NT * es / 16;
      const int m = m0 + tid / nv, ch = n0 + tid % nv * (16 / es);
      const uint32_t off0 = ((uint32_t)m * (uint32_t)Kf + (uint32_t)ch) * (uint32_t)es;
      return (ch < Kf) & (m + pass * MP < m_end) ? (int)(off0 + (uint32_t)(pass * MP) * (uint32_t)(Kf * es)) : kPastEnd;
    };
    auto turn_of = [&](auto ES) { return row_turn<kThreads / (NT * decltype(ES)::value / 16) * decltype(ES)::value>(Kf); };
    // ... of its u-th row, which `at` has come to
    auto row_off = [&](auto ES, int u, int pass, int at) -> int {
      constexpr int nv = NT * decltype(ES)::value / 16, rows = kThreads / nv;
      const int row = tid / nv + u * rows;
      return (MP % rows == 0 || row < MP) & (TO_END || m0 + pass * MP + row < m_end) ? at : kPastEnd;
    };
    constexpr std::integral_constant<int, 4> k4{};
    constexpr std::integral_constant<int, 2> k2{};
    constexpr int IT32 = (MP * (NT / 4) + kThreads - 1) / kThreads, IT16 = (MP * (NT / 8) + kThreads - 1) / kThreads;
    constexpr bool kPrefetchRes = (PASSES == 1);
    u32x4 rpre[kPrefetchRes ? IT32 : 1];
    if (kPrefetchRes && has_res) {
      if (T.out_dtype == ST_DT_F32) {
        const int turn = turn_of(k4);
        int at = first_row(k4, 0);
#pragma unroll
        for (int u = 0; u < IT32; ++u, at = next_row(at, turn)) rpre[u] = __builtin_amdgcn_raw_buffer_load_b128(rr, row_off(k4, u, 0, at), 0, POL::kActAux);
      } else if constexpr (DT != ST_DT_F32) {
        const int turn = turn_of(k2);
        int at = first_row(k2, 0);
#pragma unroll
        for (int u = 0; u < IT16; ++u, at = next_row(at, turn)) rpre[u] = __builtin_amdgcn_raw_buffer_load_b128(rr, row_off(k2, u, 0, at), 0, POL::kActAux);
      }
    }
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
    const int mp0 = m0 + pass * MP;   // first im2col row of this slice
    __syncthreads();                // the buffer (operands, split-K flag, or the previous slice) is no longer read
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const int row = wm0 + i * MF + lrow - pass * MP;
          const int chl = wn0 + j * MF + ((MF == 32) ? (8 * g + 4 * lk) : (4 * lk));
          if (PASSES == 1 || (row >= 0 && row < MP))
            *(f32x4*)(sC + row * PITCH + chl) = f32x4{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
        }
    __syncthreads();
    // Branch-free read-back: rows past the tile end or filters past K get an out-of-range offset, which
    // drops the store (and makes the residual load return zero).
    if (T.out_dtype == ST_DT_F32) {
      constexpr int NV = NT / 4;
      constexpr int IT = (MP * NV + kThreads - 1) / kThreads;
      constexpr int UB = IT < 4 ? IT : 4;        // vectors in flight per thread (bounds register use)
      const int turn = turn_of(k4);
      auto store_rows = [&](auto REST) {
      int at = first_row(k4, pass);
#pragma unroll
      for (int u0 = 0; u0 < IT; u0 += UB) {
        f32x4 a[UB];
        int off[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u, at = next_row(at, turn)) {
          const int v = (u0 + u) * kThreads + tid;
          const int row = v / NV, cv = v % NV;
          off[u] = row_off(k4, u0 + u, pass, at);
          if constexpr (decltype(REST)::value) off[u] = (mp0 + row < m_end) & (n0 + cv * 4 < Kf) ? off[u] : kPastEnd;
          a[u] = *(const f32x4*)(sC + (row < MP ? row : 0) * PITCH + cv * 4);
        }
        if (has_res) {
#pragma unroll
          for (int u = 0; u < UB; ++u)
            a[u] += __builtin_bit_cast(f32x4, kPrefetchRes ? rpre[u0 + u] : __builtin_amdgcn_raw_buffer_load_b128(rr, off[u], 0, POL::kActAux));
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          if (relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) a[u][e] = relu_f32(a[u][e]);
          }
          const u32x4 d = __builtin_bit_cast(u32x4, a[u]);
          const int ch = n0 + ((u0 + u) * kThreads + tid) % NV * 4;
          if constexpr (!decltype(REST)::value) {
            __builtin_amdgcn_raw_buffer_store_b128(d, ry, off[u], 0, POL::kOutAux);
          } else if (off[u] != kPastEnd) {
            if (ch + 4 <= Kf) {
              __builtin_amdgcn_raw_buffer_store_b128(d, ry, off[u], 0, POL::kOutAux);
            } else {
#pragma unroll
              for (int e = 0; e < 3; ++e)
                if (ch + e < Kf) __builtin_amdgcn_raw_buffer_store_b32(d[e], ry, off[u] + 4 * e, 0, POL::kOutAux);
            }
          }
        }
      }
      };
      if constexpr (kAnyFilters) {
        if (rest) store_rows(std::true_type{});
        else store_rows(std::false_type{});
      } else {
        store_rows(std::false_type{});
      }
    } else if constexpr (DT != ST_DT_F32) {
      constexpr int NV = NT / 8;
      constexpr int IT = (MP * NV + kThreads - 1) / kThreads;
      constexpr int UB = IT < 4 ? IT : 4;
      const int turn = turn_of(k2);
      int at = first_row(k2, pass);
#pragma unroll
      for (int u0 = 0; u0 < IT; u0 += UB) {
        f32x4 lo[UB], hi[UB];
        int off[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u, at = next_row(at, turn)) {
          const int v = (u0 + u) * kThreads + tid;
          const int row = v / NV, cv = v % NV;
          off[u] = row_off(k2, u0 + u, pass, at);
          const float* src = sC + (row < MP ? row : 0) * PITCH + cv * 8;
          lo[u] = *(const f32x4*)src;
          hi[u] = *(const f32x4*)(src + 4);
        }
        if (has_res) {
#pragma unroll
          for (int u = 0; u < UB; ++u) {
            const u32x4 r = kPrefetchRes ? rpre[u0 + u] : __builtin_amdgcn_raw_buffer_load_b128(rr, off[u], 0, POL::kActAux);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              lo[u][e] += unpack16<DT>(r[e >> 1], e & 1);
              hi[u][e] += unpack16<DT>(r[2 + (e >> 1)], e & 1);
            }
          }
        }
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          if (relu) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              lo[u][e] = relu_f32(lo[u][e]);
              hi[u][e] = relu_f32(hi[u][e]);
            }
          }
          u32x4 pk;
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            pk[e] = pack16<DT>(lo[u][2 * e], lo[u][2 * e + 1]);
            pk[2 + e] = pack16<DT>(hi[u][2 * e], hi[u][2 * e + 1]);
          }
          __builtin_amdgcn_raw_buffer_store_b128(pk, ry, off[u], 0, POL::kOutAux);
        }
      }
    }
    }   // slices
  } else {
  #pragma unroll
    for (int i = 0; i < BM; ++i) {
      const int m = m0 + wm0 + i * MF + lrow;
      if (m >= m_end) continue;
  #pragma unroll
      for (int j = 0; j < BN; ++j)
  #pragma unroll
        for (int g = 0; g < NG; ++g) {
          const int ch = n0 + wn0 + j * MF + ((MF == 32) ? (8 * g + 4 * lk) : (4 * lk));
          if (ch >= Kf) continue;
          float v[4] = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
          const int64_t o = (int64_t)m * Kf + ch;
          const int nv = (Kf - ch < 4) ? (Kf - ch) : 4;
          if (T.out_dtype == ST_DT_F32) {
            float* y = (float*)T.y + o;
            if (has_res) {
              const float* rp = (const float*)T.res + o;
_Pragma("unroll")
              for (int e = 0; e < 4; ++e)
                if (e < nv) {
                  if constexpr (POL::kActAux == 0) v[e] += rp[e];
                  else v[e] += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(T.res, T.y_bytes), (int)((uint32_t)(o + e) * 4u), 0, POL::kActAux));
                }
            }
            if (relu)
_Pragma("unroll")
              for (int e = 0; e < 4; ++e) v[e] = relu_f32(v[e]);
            if (vec4) *(f32x4*)y = f32x4{v[0], v[1], v[2], v[3]};
            else {
_Pragma("unroll")
              for (int e = 0; e < 4; ++e) if (e < nv) y[e] = v[e];
            }
          } else if constexpr (DT != ST_DT_F32) {
            uint16_t* y = (uint16_t*)T.y + o;
            if (has_res) {
              const uint16_t* rp = (const uint16_t*)T.res + o;
_Pragma("unroll")
              for (int e = 0; e < 4; ++e)
                if (e < nv) {
                  uint16_t rb;
                  if constexpr (POL::kActAux == 0) rb = rp[e];
                  else rb = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(make_rsrc(T.res, T.y_bytes), (int)((uint32_t)(o + e) * 2u), 0, POL::kActAux);
                  v[e] += unpack16<DT>(rb, 0);
                }
            }
            if (relu)
_Pragma("unroll")
              for (int e = 0; e < 4; ++e) v[e] = relu_f32(v[e]);
            uint2 pk;
            pk.x = pack16<DT>(v[0], v[1]);
            pk.y = pack16<DT>(v[2], v[3]);
            if (vec4) {
              *(uint2*)y = pk;
            } else {
_Pragma("unroll")
              for (int e = 0; e < 4; ++e) if (e < nv) y[e] = (uint16_t)((e < 2 ? pk.x : pk.y) >> (16 * (e & 1)));
            }
          }
        }
    }
  }
}

// ---- split-K hand-off ----------------------------------------------------------------------------
// Publishes this workgroup's partial tile; the last workgroup to arrive sums all slices in index order into acc and
// returns true (it goes on to the epilogue), the others return false.
template <int MT, int NT, int BM, int BN, int MF, class POL, class Acc>
__device__ __forceinline__ bool split_k_reduce(ConstOp& T, const st_work_item it, Acc (&acc)[BM][BN], int tid, char* smem, uint64_t* prof) {
  constexpr int NG = (MF == 32) ? 4 : 1;      // groups of 4 consecutive filters per block per lane
  {
    const int tile_id = (int)it.tile_m * T.tiles_n + (int)it.tile_n;
    constexpr uint32_t kTileBytes = MT * NT * 4;
    const __amdgpu_buffer_rsrc_t rs =
        make_rsrc(T.ws + (int64_t)tile_id * T.split_k * (MT * NT), (uint32_t)T.split_k * kTileBytes);
    const uint32_t my = (uint32_t)it.k_split_idx * kTileBytes;
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rs,
                                                 (((i * BN + j) * NG + g) * kThreads + tid) * 16, my, POL::kOutAux);
        }
    __builtin_amdgcn_s_waitcnt(0);       // every store of this thread has completed (written through)
    __syncthreads();
    uint32_t* flag = (uint32_t*)smem;
    if (tid == 0) {
      constexpr int scope = POL::kOneL2 ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT;      // in that L2, or at the memory side
      const uint32_t old = __hip_atomic_fetch_add(&T.counters[tile_id], 1u, __ATOMIC_RELAXED, scope);
      const uint32_t last = (old == (uint32_t)(T.split_k - 1));
      if (last) __hip_atomic_store(&T.counters[tile_id], 0u, __ATOMIC_RELAXED, scope);  // next run
      *flag = last;
    }
    __syncthreads();
    if (*flag == 0u) {
      if (prof && tid == 0) prof[6] = wall_clock64();
      return false;
    }
    // Sum the slices in index order.  Loads are issued in batches (GB groups x SB slices) so that the device-coherent reads, each
    // a trip to memory, overlap.  A load that is out of range still costs the compute unit's 16 clocks, so tiles of 32x32 blocks
    // with fewer slices than a batch holds load those there are (`pick`), and take the own one from the registers it is still in.
    // us, without and with, three 3x3 layers 256 -> 256 at 14x14: bf16 64x64 in 2, 4, 6, 7 slices 8.1, 7.7, 9.95, 9.9 -> 7.6, 7.3,
    // 9.35, 9.4; 64x128 in 2, 3 10.9, 10.65 -> 10.3, 10.05; fp32 1 to 2 %; 20 fp32 layers in 3 18.65 -> 17.95.  A full batch has one
    // load to spare and a branch for each (four batches in flight, their 7x7 layer 64x64 in 8 slices, 25.5 -> 25.8; 64x128 in 5 to 7, only
    // the rest picked from, 11.05 -> 11.25), so more slices are loaded in whole batches.  The small tiles have few loads, and the branches cost more than they
    // do where the slices come from memory (four 3x3 layers of batch 1, 16x64 in four: 7.21 us, 7.36 with branches), not where they
    // come from the L2 (eight networks of batch 1 as a chain 321.3 -> 319.6).  Chains pick in every batch: a second loop makes them spill
    // (320 -> 338).  Nor in the kernel for everything, which is short of scalar registers (24 layers off every round number 26.35 -> 26.55).
    constexpr int NGRP = BM * BN * NG;
    constexpr int GB = NGRP < 4 ? NGRP : 4;
    constexpr int SB = (NGRP > 4) ? 4 : 8;   // at most 32 partial vectors (128 registers) in flight
    static_assert(NGRP % GB == 0, "group batching");
    const int split = T.split_k, mine = (int)it.k_split_idx;
    auto sum_slices = [&](auto PICK, auto ONE_BATCH) {
      constexpr bool pick = decltype(PICK)::value, one = decltype(ONE_BATCH)::value;       // one: split < SB
      constexpr int SL = one ? SB - 1 : SB;
#pragma unroll
      for (int g0 = 0; g0 < NGRP; g0 += GB) {
        f32x4 sum[GB];
#pragma unroll
        for (int gg = 0; gg < GB; ++gg) sum[gg] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < (one ? 1 : split); s0 += SB) {
          f32x4 part[SB][GB];
#pragma unroll
          for (int ss = 0; ss < SL; ++ss) {
            if (!pick || (s0 + ss < split && s0 + ss != mine)) {
#pragma unroll
              for (int gg = 0; gg < GB; ++gg) {
                const uint32_t voff = pick || s0 + ss < split ? (uint32_t)(((g0 + gg) * kThreads + tid) * 16) : kInvalidOffset;
                part[ss][gg] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)voff, (s0 + ss) * (int)kTileBytes, kAuxDeviceCoherent));
              }
            } else {
#pragma unroll
              for (int gg = 0; gg < GB; ++gg) {
                const int grp = g0 + gg, i = grp / (BN * NG), j = (grp / NG) % BN, g = grp % NG;
#pragma unroll
                for (int e = 0; e < 4; ++e) part[ss][gg][e] = s0 + ss == mine ? acc[i][j][4 * g + e] : 0.f;
              }
            }
          }
#pragma unroll
          for (int ss = 0; ss < SL; ++ss)
#pragma unroll
            for (int gg = 0; gg < GB; ++gg) sum[gg] += part[ss][gg];
        }
#pragma unroll
        for (int gg = 0; gg < GB; ++gg) {
          const int grp = g0 + gg;
          const int i = grp / (BN * NG), j = (grp / NG) % BN, g = grp % NG;
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[i][j][4 * g + e] = sum[gg][e];
        }
      }
    };
    constexpr std::true_type yes;
    constexpr std::false_type no;
    constexpr bool in_chain = POL::kActAux == kAuxDeviceCoherent;
    if constexpr (POL::kOneL2 || (in_chain && MF == 32)) {
      sum_slices(yes, no);
      return true;
    }
    if constexpr (MF == 32 && !POL::kAnyFilters) {
      if (split < SB) {
        sum_slices(yes, yes);
        return true;
      }
    }
    sum_slices(no, no);
  }
  return true;
}

// ---- one workgroup tile --------------------------------------------------------------------------
// MT x NT output tile, 4 wavefronts as WPX x WCH, MFMA block edge MF, KB bytes of the reduction index staged per row
// per K step, ST steps of operands resident in LDS.  Operands go from memory to LDS directly (load_to_lds), so no
// register and no LDS-write instruction is spent on staging; the loads of ST - 1 further steps are in flight while one
// step's MFMAs run, and the MFMA operands of the next step are read from LDS during them.  A K step is one barrier.
// Out-of-range lanes load zeros, so padding, ragged tiles and the end of the K range need no branches.
// LDS rows are KB bytes without padding: 16-byte chunk c of row r sits at position c ^ swz(r), so that the 16 rows an
// MFMA operand read touches at a time fall into 16 different 16-byte bank groups; the swizzle is applied by choosing
// which chunk each lane fetches (a lane's LDS position is fixed).
//
// PIECES: layers whose channel count is no multiple of the vector.  The reduction index is then walked in two parts: the whole
// vectors of every tap's channels, which go straight to LDS like any others (an element-aligned address costs nothing where it is a
// multiple of four bytes, and twice the step where it is not), and at the end the few channels left over, a vector per tap
// through registers.  A 64x64 step of 3x3, 240 channels or so, alone: fp32 1295 clocks
// where conv_tile_gather takes 1780, bf16 462 (odd channel counts 961) for 1074 (1187).
template <int MT, int NT, int WPX, int WCH, int MF, int KB, int ST, int DT, bool PIECES, class POL = PlainActs>
__device__ __forceinline__ void conv_tile(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr int ES = ElemOf<DT>::ES;
  constexpr int VEC = 16 / ES;          // elements per 16-byte vector
  constexpr int KT = KB / ES;           // elements of K per step
  constexpr int CH = KB / 16;           // 16-byte chunks per row
  constexpr int RPI = 64 / CH;          // rows one load instruction of a wavefront covers
  constexpr int AW = MT / (4 * RPI), BW = NT / (4 * RPI);   // load instructions per wavefront and step
  constexpr int kStage = (MT + NT) * KB;
  constexpr int WM = MT / WPX, WN = NT / WCH;
  constexpr int BM = WM / MF, BN = WN / MF;
  constexpr int SUBB = (MF == 32) ? 32 : 64;   // row bytes one MFMA sub-step consumes
  constexpr int NSUB = KB / SUBB;
  typedef Mma<DT, MF> MMA;
  typedef typename MMA::Acc Acc;
  static_assert(WPX * WCH == 4 && WM % MF == 0 && WN % MF == 0, "bad tile shape");
  static_assert(MT % (4 * RPI) == 0 && NT % (4 * RPI) == 0, "every wavefront stages whole instructions");
  static_assert(ST >= 2 && ST * kStage <= kSmemBytes, "tile does not fit the LDS allocation");
  static_assert(kResidualLoads<MT, NT> * 4096 <= kStage, "a 16-bit residual tile must fit a stage");
  static_assert(KB == 64 || KB == 128 || KB == 256, "swizzles exist for these row lengths");
  static_assert(MF == 32 || KB >= 128, "the 64-byte swizzle is for 32x32 blocks");

  tile_fields_loaded(T);
  const int tid = work_thread_id();
  if (prof && tid == 0) stamp_start(prof);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = (int)it.tile_m * MT;
  const int n0 = (int)it.tile_n * NT;
  // Launches of fp32 layers alone: what the first loads do not need is read and worked out behind them.  us: 20 3x3 layers
  // 128 -> 128 at 16x16 18.10 -> 17.85, 30 1x1 layers 256 -> 256 11.46 -> 11.14, 13 of 136 -> 512 at 8x8 with a residual 6.97 -> 6.76, four 3x3
  // of 512 at 7x7 17.40 -> 17.08.  Others lose by it or gain nothing: 24 layers off every round number 26.05 -> 26.25, 32 unlike tenants
  // 78.6 -> 79.0, four networks of batch 4 as layer launches 511.5 -> 514.4, eight of batch 8 as a chain 1036 -> 1038.
  constexpr bool late = DT == ST_DT_F32 && std::is_same_v<POL, PlainActs>;
  // everything the K loop needs of the record, read once (the loads to LDS count as writes to any memory)
  const int C = T.C, W = T.W, WC = W * C, H = T.H, R = T.R, S = T.S, SC = S * C, step_dk0 = late ? 0 : T.step_dk, step_dr0 = late ? 0 : T.step_dr;
  const u32x4 rx = rsrc_words(T.x, T.x_bytes), rw = rsrc_words(T.w, T.w_bytes);

  // K-step range of this work item
  const int ks_begin = (int)it.k_split_idx * T.k_steps_per_split;
  int ks_end = ks_begin + T.k_steps_per_split;
  if (ks_end > T.k_steps) ks_end = T.k_steps;
  const int main_steps = PIECES ? (late ? T.step_dr : step_dr0) : ks_end;      // steps of whole vectors (of the layer), before those of left-over channels
  const int nsteps = (PIECES && main_steps < ks_end ? main_steps : ks_end) - ks_begin;

  // staging: which row of an instruction's block of RPI rows, and which 16-byte chunk of it, this lane fetches
  const int lr = lane / CH;
  const int swz = (KB == 256) ? ((4 * wave + lr) & 15) : (KB == 128) ? ((4 * (wave & 1) + (lr >> 1)) & 7) : ((lr >> 2) & 3);
  const int chunk = (lane % CH) ^ swz;
  // per-thread patch rows: first image row and column, and element offset of the patch (a 1x1 layer of stride 1 without
  // padding needs no position in the image: output pixel m is input pixel m)
  int a_h0[AW], a_w0[AW], a_base[AW];
  const bool same_pixels = !PIECES && T.k_order == kOrderLinear && T.stride == 1;
  if (!same_pixels) {
#pragma unroll
    for (int i = 0; i < AW; ++i) {
      const int m = m0 + (i * 4 + wave) * RPI + lr;
      const bool ok = m < T.M;
      const int mm = ok ? m : 0;
      const int n = fast_div(mm, T.magic_pq, T.shift_pq);
      const int pq = mm - n * T.PQ;
      const int p = fast_div(pq, T.magic_q, T.shift_q);
      const int q = pq - p * T.Q;
      const int h0 = p * T.stride - T.pad;
      a_w0[i] = q * T.stride - T.pad;
      a_base[i] = (n * H + h0) * WC + a_w0[i] * C;
      a_h0[i] = ok ? h0 : -(1 << 24);     // a dead row fails every bounds check
    }
  } else {
    const int m = m0 + wave * RPI + lr;
#pragma unroll
    for (int i = 0; i < AW; ++i) {
      a_w0[i] = 0;
      a_base[i] = i == 0 ? m * C : a_base[i - 1] + 4 * RPI * C;
      a_h0[i] = m + i * 4 * RPI < T.M ? 0 : -1;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + (uint32_t)wave * 1024u;

  // wavefront / lane geometry of the MFMA operands
  const int wm0 = (wave % WPX) * WM;
  const int wn0 = (wave / WPX) * WN;
  const int lrow = lane & (MF - 1);
  const int lk = lane / MF;          // 0..1 for 32x32 blocks, 0..3 for 16x16 blocks
  uint32_t a_lds[NSUB], b_lds[NSUB];     // LDS offset of this lane's first pixel and first filter fragment in stage 0, per sub-step
  auto operand_addresses = [&]() {
    const int rsw = (KB == 256) ? (lrow & 15) : (KB == 128) ? ((lrow >> 1) & 7) : ((lrow >> 2) & 3);
    const int rbase = lrow * KB + (lk ^ rsw) * 16;          // sub-step 0; sub-step u is this ^ (u * SUBB)
#pragma unroll
    for (int u = 0; u < NSUB; ++u) {
      a_lds[u] = (uint32_t)((rbase ^ (u * SUBB)) + wm0 * KB);
      b_lds[u] = (uint32_t)((rbase ^ (u * SUBB)) + MT * KB + wn0 * KB);
    }
  };
  if constexpr (!late) operand_addresses();

  // PIECES: two sums of each block, one over even and one over odd sub-steps.  Layers of this form are often split less than
  // with gathered tiles, and a longer chain of fp32 additions errs more (43 such layers against 64 bits, mean relative error
  // 2.79e-7 gathered, 3.12e-7 with one sum, 2.65e-7 with two).
  Acc acc[BM][BN], odd[PIECES ? BM : 1][PIECES ? BN : 1];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j)
#pragma unroll
      for (int v = 0; v < (int)(sizeof(Acc) / 4); ++v) {
        acc[i][j][v] = 0.f;
        if constexpr (PIECES) odd[i][j][v] = 0.f;
      }
  struct Frags { u32x4 w[NSUB][BN], x[NSUB][BM]; };
  auto read_one = [&](auto I, auto stage_off, Frags& f) {     // operand fragment I of the step: per sub-step filters, then pixels
    constexpr int u = decltype(I)::value / (BN + BM), q = decltype(I)::value % (BN + BM);
    if constexpr (q < BN) f.w[u][q] = *(const u32x4*)(smem + b_lds[u] + (stage_off + q * MF * KB));
    else f.x[u][q - BN] = *(const u32x4*)(smem + a_lds[u] + (stage_off + (q - BN) * MF * KB));
  };
  auto read_frags = [&](auto stage_off, Frags& f) { static_for<NSUB*(BN + BM)>([&](auto I) { read_one(I, stage_off, f); }); };
  constexpr int NMMA = NSUB * BM * BN;
  auto mma_one = [&](auto I, const Frags& f) {
    constexpr int u = decltype(I)::value / (BM * BN), i = decltype(I)::value / BN % BM, j = decltype(I)::value % BN;
    if constexpr (PIECES && u % 2 == 1) odd[i][j] = MMA::run(f.w[u][j], f.x[u][i], odd[i][j]);
    else acc[i][j] = MMA::run(f.w[u][j], f.x[u][i], acc[i][j]);
  };
  auto mma = [&](const Frags& f) { static_for<NMMA>([&](auto I) { mma_one(I, f); }); };

  // A 16-bit residual tile is loaded into the stage of the last step but one as soon as that is free (no later loads
  // are waited for by count), and added in the epilogue.
  int res_lds = -1;
  if constexpr (DT != ST_DT_F32 && !PIECES) {
    if ((T.epilogue & ST_EPI_RESIDUAL) != 0u && T.out_dtype != ST_DT_F32 && (T.K & 7) == 0 && T.split_k == 1)
      res_lds = (nsteps == 1 ? 1 : (nsteps - 2) % ST) * kStage;
  }
  // The reduction index k = (r*S + s)*C + c is walked in one of three orders (planner's k_order):
  //   kOrderTaps      ascending k; any C.  Every lane keeps the position of its own vector: filter row kr and element
  //                   kk = s*C + c inside it, which is also the element offset inside the image row, from the patch.
  //   kOrderChannels  C a multiple of the step, at most 32 taps: channel blocks outermost, the R*S taps of a block one
  //                   after another.  Tap and block are uniform, a row's valid taps are bits of one register.
  //   kOrderLinear    1x1 layers without padding: nothing changes from step to step but the scalar offset.
  //   kOrderPieces    ascending over the whole vectors of every tap (PIECES); the lane works its tap out afresh every step.
  // What bounds a step: 16 clocks of the vector-memory unit per load instruction (a 64x64 step is 256), MFMA time, and,
  // for a wavefront that has its SIMD to itself, four clocks or so per instruction of any kind.  Hence tap masks, immediate
  // LDS offsets and as little scalar arithmetic as possible.  Clocks per 64x64 step alone on a compute unit, 3x3 layers:
  // 634 staged through registers, 608 with loads straight to LDS, 500 with loads, LDS reads and MFMAs taking turns, 350
  // with masks and immediates, 295 with the MFMAs spread evenly (1x1 layers: 320).  128x128, two workgroups per unit: 1932
  // -> 1300 (777 -> 1040 TFLOP/s); rows of 64 bytes instead of 128 take 1830, half of every cache line fetched twice.
  auto k_loop = [&](auto ORDER) {
    constexpr int order = decltype(ORDER)::value;
    constexpr uint32_t kTop = 0x80000000u;
    const int step_dk = !late ? step_dk0 : order == kOrderTaps || order == kOrderPieces ? T.step_dk : 0;
    const int step_dr = !late ? step_dr0 : order == kOrderTaps ? T.step_dr : 0;
    int kr = 0, kk = 0, koff = 0;          // kOrderTaps: per lane
    int s_left = 0, r_left = 0;            // kOrderChannels: taps left in this filter row, rows left after it
    uint32_t a_soff = 0u, b_soff;          // byte offsets of the step; kOrderChannels: a_soff is added per lane (it may be negative)
    uint32_t va[AW], vb[BW], b_off[BW];    // byte offsets of the next step's vectors
    uint32_t bad[AW], bad0[AW];            // kOrderChannels: bit 31 - t: tap t of this row lies outside; bad: shifted to the next tap
    const uint32_t c_bytes = (uint32_t)(C * ES), wrap_row = (uint32_t)((WC - SC) * ES);
    const uint32_t wrap_a = (uint32_t)(KB - R * WC * ES), wrap_b = (uint32_t)(KB - R * SC * ES);
    if constexpr (order == kOrderPieces) {
      kk = ks_begin * KT + chunk * VEC;       // position among the whole vectors
      b_soff = 0u;
    } else if constexpr (order == kOrderTaps) {
      const int k = ks_begin * KT + chunk * VEC;
      kr = fast_div(fast_div(k, T.magic_c, T.shift_c), T.magic_s, T.shift_s);
      kk = k - kr * SC;
      koff = kr * WC + kk;
      b_soff = (uint32_t)(ks_begin * KB);
    } else {
      int block = ks_begin, tap = 0, r = 0, sx = 0;
      if constexpr (order == kOrderChannels) {
        if (ks_begin != 0) {
          const int taps = R * S;
          block = ks_begin / taps;
          tap = ks_begin - block * taps;
          r = tap / S;
          sx = tap - r * S;
        }
        s_left = S - 1 - sx;
        r_left = R - 1 - r;
      }
      a_soff = (uint32_t)((r * WC + sx * C) * ES + block * KB);
      b_soff = (uint32_t)(tap * C * ES + block * KB);
#pragma unroll
      for (int i = 0; i < AW; ++i) {
        a_base[i] = (a_base[i] + chunk * VEC) * ES;
        if constexpr (order == kOrderLinear) {
          va[i] = a_h0[i] >= 0 ? (uint32_t)a_base[i] : kInvalidOffset;
        } else {
          // filter rows and columns that lie inside: [h_lo, h_hi) and [w_lo, w_hi)
          const int h_lo = a_h0[i] < 0 ? -a_h0[i] : 0, h_hi = H - a_h0[i] < R ? H - a_h0[i] : R;
          const int w_lo = a_w0[i] < 0 ? -a_w0[i] : 0, w_hi = W - a_w0[i] < S ? W - a_w0[i] : S;
          const uint32_t cols = w_hi > w_lo ? ((w_hi < 32 ? (1u << w_hi) : 0u) - (1u << w_lo)) : 0u;
          const int b_lo = h_lo * S, b_hi = h_hi * S;
          const uint32_t rows = h_hi > h_lo && h_lo < R ? (((b_hi < 32 ? (1u << b_hi) : 0u) - (1u << b_lo)) & T.tap_rows) : 0u;
          bad0[i] = ~__builtin_bitreverse32(cols * rows);
          bad[i] = bad0[i] << tap;
        }
      }
    }
    const int b_row = n0 + wave * RPI + lr;
    const uint32_t b_first = (uint32_t)(b_row * T.Kg + (order == kOrderPieces ? 0 : chunk * VEC)) * ES, b_turn = (uint32_t)(4 * RPI * ES) * (uint32_t)T.Kg;
#pragma unroll
    for (int i = 0; i < BW; ++i) vb[i] = b_off[i] = b_row + i * 4 * RPI < T.K ? b_first + (uint32_t)i * b_turn : kInvalidOffset;
    auto addresses = [&]() {
      if constexpr (order == kOrderChannels) {
#pragma unroll
        for (int i = 0; i < AW; ++i) va[i] = (bad[i] & kTop) | ((uint32_t)a_base[i] + a_soff);
      } else if constexpr (order == kOrderPieces) {
        const int tap = fast_div(kk, T.magic_c, T.shift_c), c = kk - tap * step_dk;
        const int r = fast_div(tap, T.magic_s, T.shift_s), sx = tap - r * S;
        const bool kin = r < R;         // past the end nothing is loaded
        const int off = r * WC + sx * C + c;
#pragma unroll
        for (int i = 0; i < AW; ++i) {
          const bool ok = kin & ((unsigned)(a_h0[i] + r) < (unsigned)H) & ((unsigned)(a_w0[i] + sx) < (unsigned)W);
          va[i] = ok ? (uint32_t)(a_base[i] + off) * ES : kInvalidOffset;
        }
        const uint32_t b = kin ? (uint32_t)(tap * C + c) * ES : 0u, kmask = kin ? 0u : kInvalidOffset;
#pragma unroll
        for (int i = 0; i < BW; ++i) vb[i] = (b_off[i] + b) | kmask;
      } else if constexpr (order == kOrderTaps) {
        const bool kin = kr < R;        // past the end of the reduction index nothing is loaded
        const int hr = kin ? kr : (1 << 28);
        const uint32_t kmask = kin ? 0u : kInvalidOffset;
#pragma unroll
        for (int i = 0; i < AW; ++i) {
          const bool ok = ((unsigned)(a_h0[i] + hr) < (unsigned)H) & ((unsigned)(a_w0[i] * C + kk) < (unsigned)WC);
          va[i] = ok ? (uint32_t)(a_base[i] + koff) * ES : kInvalidOffset;
        }
#pragma unroll
        for (int i = 0; i < BW; ++i) vb[i] = b_off[i] | kmask;
      }
    };
    addresses();
    // one step on, after a step's loads were issued
    auto advance = [&]() {
      if constexpr (order == kOrderLinear) {
        a_soff += KB;
        b_soff += KB;
      } else if constexpr (order == kOrderChannels) {
        a_soff += c_bytes;
        b_soff += c_bytes;
#pragma unroll
        for (int i = 0; i < AW; ++i) bad[i] <<= 1;
        if (__builtin_expect(--s_left < 0, 0)) {
          s_left = S - 1;
          a_soff += wrap_row;
          if (--r_left < 0) {
            r_left = R - 1;
            a_soff += wrap_a;
            b_soff += wrap_b;
#pragma unroll
            for (int i = 0; i < AW; ++i) bad[i] = bad0[i];
          }
        }
      } else if constexpr (order == kOrderPieces) {
        kk += KT;
      } else {
        const bool wrap = kk + step_dk >= SC;
        kk += step_dk - (wrap ? SC : 0);
        kr += step_dr + (wrap ? 1 : 0);
        koff += step_dr * WC + step_dk + (wrap ? WC - SC : 0);
        b_soff += KB;
      }
      addresses();
    };
    auto issue_one = [&](auto I, auto stage_off) {     // load instruction I of the step
      constexpr int i = decltype(I)::value, off = i < AW ? i * 4096 : MT * KB + (i - AW) * 4096;
      if constexpr (i < AW) load_to_lds<POL::kActAux, off>(rx, va[i], order == kOrderLinear ? a_soff : 0u, lds0 + (uint32_t)stage_off);
      else load_to_lds<0, off>(rw, vb[i - AW], b_soff, lds0 + (uint32_t)stage_off);
    };

    // step s lives in stage s % ST.  The first ST steps go in flight at once.
    const int in_flight = nsteps < ST ? nsteps : ST;
    for (int s = 0; s < in_flight; ++s) {
      static_for<AW + BW>([&](auto I) { issue_one(I, s * kStage); });
      advance();
    }
    if constexpr (late) operand_addresses();
    if (res_lds >= 0 && nsteps == 1) {          // a one-step K loop: the residual follows the operands at once
      stage_residual<MT, NT, POL>(T, m0, n0, wave, lane, lds0 + (uint32_t)res_lds);
      wait_loads_barrier<kResidualLoads<MT, NT>>();
    } else {
      wait_steps_barrier<ST - 1, AW + BW>(in_flight - 1);
    }
    if (prof && tid == 0) prof[1] = __builtin_readcyclecounter();
    Frags f0, f1;
    read_frags(0, f0);
    // One K step: wait until step k + 1 has arrived and everyone has read step k's operands, read step k + 1's operands
    // and compute step k meanwhile, refill step k's stage with step k + ST.  The vector-memory unit takes 16 clocks
    // per load instruction (64 bytes per clock) and a wavefront stands still while the unit is busy, so loads, LDS reads
    // and MFMAs take turns.
    auto step = [&](const Frags& fc, Frags& fn, auto cur, auto nxt) {
      wait_loads_barrier<(ST - 2) * (AW + BW)>();
      constexpr int NL = AW + BW, NR = NSUB * (BN + BM);
      static_for<NL>([&](auto L) {
        constexpr int l = decltype(L)::value, b = l * NR / NL, e = (l + 1) * NR / NL, mb = l * NMMA / NL, me = (l + 1) * NMMA / NL;
        issue_one(L, cur);
        static_for<e - b>([&](auto I) { read_one(std::integral_constant<int, b + decltype(I)::value>{}, nxt, fn); });
        static_for<me - mb>([&](auto I) { mma_one(std::integral_constant<int, mb + decltype(I)::value>{}, fc); });
        __builtin_amdgcn_sched_barrier(0);
      });
      advance();
    };
    // the last ST steps of the range (and short ranges): nothing is left to refill
    auto last_step = [&](const Frags& fc, Frags& fn, int nxt, int left) {     // left = steps after this one
      if (left > 0) {
        wait_steps_barrier<ST - 2, AW + BW>(left - 1);
        if (left == 1 && res_lds >= 0) stage_residual<MT, NT, POL>(T, m0, n0, wave, lane, lds0 + (uint32_t)res_lds);
        read_frags(nxt, fn);
      }
      mma(fc);
    };
    int k = 0, cur = 0;              // cur: LDS offset of step k's stage
    auto after = [&](int off) { return off + kStage < ST * kStage ? off + kStage : 0; };
    constexpr int U = ST % 2 == 0 ? ST : 2 * ST;
    for (; k + U + ST <= nsteps; k += U)       // whole turns of the stages: their LDS offsets are immediates
      static_for<U>([&](auto J) {
        constexpr int j = decltype(J)::value;
        const std::integral_constant<int, j % ST * kStage> c{};
        const std::integral_constant<int, (j + 1) % ST * kStage> n{};
        if constexpr (j % 2 == 0) step(f0, f1, c, n);
        else step(f1, f0, c, n);
      });
    for (; k + 1 + ST < nsteps; k += 2) {
      const int n1 = after(cur), n2 = after(n1);
      step(f0, f1, cur, n1);
      step(f1, f0, n1, n2);
      cur = n2;
    }
    if (k + ST < nsteps) {
      const int n1 = after(cur);
      step(f0, f1, cur, n1);
      f0 = f1;
      cur = n1;
      ++k;
    }
    for (;; k += 2) {
      const int n1 = after(cur), n2 = after(n1);
      last_step(f0, f1, n1, nsteps - 1 - k);
      if (k + 1 >= nsteps) break;
      last_step(f1, f0, n2, nsteps - 2 - k);
      if (k + 2 >= nsteps) break;
      cur = n2;
    }
  };
  if constexpr (PIECES) {
    if (nsteps > 0) k_loop(std::integral_constant<int, kOrderPieces>{});
    else {
      if constexpr (late) operand_addresses();
      if (prof && tid == 0) prof[1] = __builtin_readcyclecounter();
    }
    // The channels left over: a vector per tap, the last one inside its channels, of which those that the whole vectors have are
    // cleared in both operands; 16 bytes at a time to where load_to_lds would have put them.
    const int left = C - (late ? T.step_dk : step_dk0), taps = R * S;
    uint32_t keep[4];
#pragma unroll
    for (int d = 0; d < 4; ++d)
      keep[d] = ES == 4 ? (d >= VEC - left ? 0xffffffffu : 0u) : (2 * d >= VEC - left ? 0x0000ffffu : 0u) | (2 * d + 1 >= VEC - left ? 0xffff0000u : 0u);
    const __amdgpu_buffer_rsrc_t bx = make_rsrc(T.x, T.x_bytes), bw = make_rsrc(T.w, T.w_bytes);
    u32x4 qa[AW], qb[BW];
    auto fetch_left = [&](int ts) {
      const int tap = (ts - main_steps) * CH + chunk;
      const int r = fast_div(tap, T.magic_s, T.shift_s), sx = tap - r * S;
      const bool kin = tap < taps;
#pragma unroll
      for (int i = 0; i < AW; ++i) {
        const bool ok = kin & ((unsigned)(a_h0[i] + r) < (unsigned)H) & ((unsigned)(a_w0[i] + sx) < (unsigned)W);
        qa[i] = __builtin_amdgcn_raw_buffer_load_b128(bx, (int)(ok ? (uint32_t)(a_base[i] + r * WC + sx * C + C - VEC) * ES : kInvalidOffset), 0, POL::kActAux);
      }
#pragma unroll
      for (int i = 0; i < BW; ++i) {
        const int row = n0 + (i * 4 + wave) * RPI + lr;
        qb[i] = __builtin_amdgcn_raw_buffer_load_b128(bw, (int)((kin & (row < T.K)) ? (uint32_t)(row * T.Kg + tap * C + C - VEC) * ES : kInvalidOffset), 0, 0);
      }
    };
    int ts = ks_begin > main_steps ? ks_begin : main_steps;
    if (ts < ks_end) fetch_left(ts);
    for (; ts < ks_end; ++ts) {
      __syncthreads();                // the stage is no longer read
#pragma unroll
      for (int i = 0; i < AW; ++i) *(u32x4*)(smem + wave * 1024 + i * 4096 + lane * 16) = u32x4{qa[i][0] & keep[0], qa[i][1] & keep[1], qa[i][2] & keep[2], qa[i][3] & keep[3]};
#pragma unroll
      for (int i = 0; i < BW; ++i) *(u32x4*)(smem + wave * 1024 + MT * KB + i * 4096 + lane * 16) = u32x4{qb[i][0] & keep[0], qb[i][1] & keep[1], qb[i][2] & keep[2], qb[i][3] & keep[3]};
      __syncthreads();
      if (ts + 1 < ks_end) fetch_left(ts + 1);
      Frags f;
      read_frags(0, f);
      mma(f);
    }
#pragma unroll
    for (int i = 0; i < BM; ++i)
#pragma unroll
      for (int j = 0; j < BN; ++j)
#pragma unroll
        for (int v = 0; v < (int)(sizeof(Acc) / 4); ++v) acc[i][j][v] += odd[i][j][v];
  } else {
  switch (T.k_order) {
    case kOrderLinear: k_loop(std::integral_constant<int, kOrderLinear>{}); break;
    case kOrderChannels: k_loop(std::integral_constant<int, kOrderChannels>{}); break;
    default: k_loop(std::integral_constant<int, kOrderTaps>{}); break;
  }
  }

  if (prof && tid == 0) prof[2] = __builtin_readcyclecounter();
  if (T.split_k > 1 && !split_k_reduce<MT, NT, BM, BN, MF, POL>(T, it, acc, tid, smem, prof)) return;

  // ---- epilogue: (+ residual) -> ReLU -> cast -> store ---------------------------------------------
  tile_epilogue<MT, NT, BM, BN, MF, DT, 1, kSmemBytes, POL>(T, acc, m0, T.M, n0, wm0, wn0, lrow, lk, tid, smem, res_lds);
  if (prof && tid == 0) stamp_end(prof);
}

// ---- workgroup tile with the input patch resident in LDS ---------------------------------------------
// For 3x3 stride-1 layers in 16-bit types.  conv_tile stages a pixel row once per tap; here the run of input pixels that
// the tile's taps touch (MT + 2 * W + 2 of them for a same-size layer: the output's linear order is the input's) is loaded
// once per block of KT channels, into one of two buffers, while the previous block's taps are computed, and only filters
// are staged per step.  A tap is an offset in LDS rows, its addresses computed once; a pixel whose tap lies outside the
// image reads the row after the last, which is zero.
// What it takes away: a good part of the 64 bytes per clock a compute unit can load, and half of the load instructions a
// lone workgroup issues.  A K step at 256 channels of 14x14, data not in the L2: 64x64 tile 335 -> 312 clocks alone and
// 444 -> 368 beside a second workgroup, 128x64 702 -> 550, 64x128 695 -> 625; first operands 3700 -> 2370.  What bounds it now:
// alone the LDS reads and the barrier, beside a second one the MFMAs (512 of 550 clocks at 128x64).
// LDS: [patch][patch, when there is more than one channel block][ST filter steps][NT][KB].
template <int MT, int NT, int WPX, int WCH, int MF, int KB, int ST, int DT, class POL = PlainActs>
__device__ __forceinline__ void conv_tile_patch(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr int ES = ElemOf<DT>::ES;
  constexpr int VEC = 16 / ES;
  constexpr int CH = KB / 16;
  constexpr int RPI = 64 / CH;          // LDS rows one load instruction of a wavefront covers
  constexpr int BW = NT / (4 * RPI);    // filter load instructions per wavefront and step
  constexpr int kStage = NT * KB;
  constexpr int WM = MT / WPX, WN = NT / WCH;
  constexpr int BM = WM / MF, BN = WN / MF;
  constexpr int SUBB = (MF == 32) ? 32 : 64;
  constexpr int NSUB = KB / SUBB;
  constexpr int kTaps = kPatchTaps;
  typedef Mma<DT, MF> MMA;
  typedef typename MMA::Acc Acc;
  static_assert(ES == 2 && (KB == 128 || KB == 256) && NT % (4 * RPI) == 0 && kTaps == 9 && ST < kTaps, "patch tile shape");

  tile_fields_loaded(T);
  const int tid = work_thread_id();
  if (prof && tid == 0) stamp_start(prof);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = (int)it.tile_m * MT;
  const int n0 = (int)it.tile_n * NT;
  const int W = T.W, H = T.H, pad = T.pad;
  const uint32_t c_bytes = (uint32_t)(T.C * ES);
  const int p_rows = T.patch_rows, p_loads = T.patch_loads;
  const uint32_t p_bytes = (uint32_t)(p_loads * 4 * RPI * KB);      // one patch buffer
  const u32x4 rx = rsrc_words(T.x, T.x_bytes), rw = rsrc_words(T.w, T.w_bytes);

  // channel blocks of this K slice
  const int block0 = (int)it.k_split_idx * T.patch_blocks;
  const int all_blocks = (int)(c_bytes / KB);
  const int blocks = all_blocks - block0 < T.patch_blocks ? all_blocks - block0 : T.patch_blocks;

  // linear input pixel under tap (0, 0) of output pixel m (may lie outside the image, or before its start)
  auto locate = [&](int m, int& h0, int& w0) -> int {
    const int n = fast_div(m, T.magic_pq, T.shift_pq);
    const int pq = m - n * T.PQ;
    const int p = fast_div(pq, T.magic_q, T.shift_q);
    h0 = p - pad;
    w0 = pq - p * T.Q - pad;
    return (n * H + h0) * W + w0;
  };
  int h0, w0;
  const int lo = __builtin_amdgcn_readfirstlane(locate(m0, h0, w0));

  // staging geometry (see conv_tile): the row of an instruction's block this lane fetches, and which chunk of it
  const int lr = lane / CH;
  const int swz = (KB == 256) ? ((4 * wave + lr) & 15) : ((4 * (wave & 1) + (lr >> 1)) & 7);
  const int chunk = (lane % CH) ^ swz;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem + (uint32_t)wave * 1024u;
  const uint32_t b_lds0 = __builtin_amdgcn_readfirstlane((all_blocks > 1 ? 2u : 1u) * p_bytes);
  const int pr0 = wave * RPI + lr;
  const uint32_t pv0 = (uint32_t)((lo + pr0) * (int)c_bytes + chunk * 16);
  const int p_left = p_rows - pr0;
  const uint32_t turn_bytes = (uint32_t)(4 * RPI) * c_bytes;
  auto issue_patch = [&](int j, uint32_t soff, uint32_t lds) {      // load instruction j of a channel block's patch
    const uint32_t v = j * 4 * RPI < p_left ? pv0 + (uint32_t)j * turn_bytes : kInvalidOffset;
    load_to_lds<POL::kActAux, 0>(rx, v, soff, __builtin_amdgcn_readfirstlane(lds + (uint32_t)j * 4096u));
  };
  uint32_t b_off[BW];
  const int b_row = n0 + wave * RPI + lr;
  const uint32_t b_first = (uint32_t)(b_row * T.Kg + chunk * VEC) * ES, b_turn = (uint32_t)(4 * RPI * ES) * (uint32_t)T.Kg;
#pragma unroll
  for (int i = 0; i < BW; ++i) b_off[i] = b_row + i * 4 * RPI < T.K ? b_first + (uint32_t)i * b_turn : kInvalidOffset;
  uint32_t b_soff = __builtin_amdgcn_readfirstlane((uint32_t)(block0 * KB));      // of the step to be staged next
  const uint32_t wrap_b = (uint32_t)KB - (uint32_t)(kTaps - 1) * c_bytes;
  const uint32_t b_base = lds0 + b_lds0;
  auto issue_filter = [&](auto I, uint32_t stage_off) {
    constexpr int i = decltype(I)::value;
    load_to_lds<0, i * 4096>(rw, b_off[i], b_soff, __builtin_amdgcn_readfirstlane(b_base + stage_off));
  };
  {
    const uint32_t soff = b_soff;
    for (int j = 0; j < p_loads; ++j) issue_patch(j, soff, lds0);
  }
  static_for<ST>([&](auto S) {
    static_for<BW>([&](auto I) { issue_filter(I, decltype(S)::value * kStage); });
    b_soff += c_bytes;
  });

  // MFMA operands: filters as in conv_tile; for a pixel its LDS address per tap, in the patch being read
  const int wm0 = (wave % WPX) * WM;
  const int wn0 = (wave / WPX) * WN;
  const int lrow = lane & (MF - 1);
  const int lk = lane / MF;
  const int rsw = (KB == 256) ? (lrow & 15) : ((lrow >> 1) & 7);
  const int rbase = lrow * KB + (lk ^ rsw) * 16;
  uint32_t a_tap[kTaps][BM];
  const uint32_t b_lds = (uint32_t)(rbase + wn0 * KB) + b_lds0;
#pragma unroll
  for (int i = 0; i < BM; ++i) {
    const int m = m0 + wm0 + i * MF + lrow;
    const int row0 = locate(m < T.M ? m : m0, h0, w0) - lo;
#pragma unroll
    for (int t = 0; t < kTaps; ++t) {
      const int r = t / 3, s = t % 3;
      const bool in = m < T.M && (uint32_t)(h0 + r) < (uint32_t)H && (uint32_t)(w0 + s) < (uint32_t)W;
      const int row = in ? row0 + r * W + s : p_rows;
      a_tap[t][i] = (uint32_t)(row * KB + lk * 16) ^ (KB == 256 ? ((uint32_t)row << 4) & 0xf0u : ((uint32_t)row << 3) & 0x70u);
    }
  }

  Acc acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j)
#pragma unroll
      for (int v = 0; v < (int)(sizeof(Acc) / 4); ++v) acc[i][j][v] = 0.f;
  struct Frags { u32x4 w[NSUB][BN], x[NSUB][BM]; };
  auto read_one = [&](auto I, auto N, uint32_t b_addr, Frags& f) {      // operand I of tap N, its filters at b_addr
    constexpr int u = decltype(I)::value / (BN + BM), q = decltype(I)::value % (BN + BM), n = decltype(N)::value;
    if constexpr (q < BN) f.w[u][q] = *(const u32x4*)(smem + (b_addr ^ (uint32_t)(u * SUBB)) + q * MF * KB);
    else f.x[u][q - BN] = *(const u32x4*)(smem + (a_tap[n][q - BN] ^ (uint32_t)(u * SUBB)));
  };
  constexpr int NR = NSUB * (BN + BM), NMMA = NSUB * BM * BN;
  auto mma_one = [&](auto I, const Frags& f) {
    constexpr int u = decltype(I)::value / (BM * BN), i = decltype(I)::value / BN % BM, j = decltype(I)::value % BN;
    acc[i][j] = MMA::run(f.w[u][j], f.x[u][i], acc[i][j]);
  };

  wait_loads_barrier<(ST - 1) * BW>();
  if (prof && tid == 0) prof[1] = __builtin_readcyclecounter();
  Frags f0, f1;
  static_for<NR>([&](auto I) { read_one(I, std::integral_constant<int, 0>{}, b_lds, f0); });
  uint32_t cur = 0;      // the stage the step being computed was read from
  // One channel block.  Step t computes tap t, reads the operands of the next one and issues the filters ST steps ahead
  // into the stage tap t was read from.  MORE blocks to come: the next one's patch is loaded in one go behind step 0's filters,
  // since loads return in order: filters issued behind it arrive no earlier, and the patch often comes from far away.
  uint32_t delta = p_bytes, next_lds = lds0 + p_bytes, p_soff = (uint32_t)((block0 + 1) * KB);
  auto block = [&](auto MORE) {
    constexpr bool more = decltype(MORE)::value;
    static_for<kTaps>([&](auto TT) {
      constexpr int t = decltype(TT)::value, n = (t + 1) % kTaps;
      constexpr bool read = more || t + 1 < kTaps, load = more || t + ST < kTaps;
      // loads younger than tap t + 1's filters: those of the taps up to t + ST - 1, and the patch loads (at least kPatchMin)
      constexpr int younger = (more ? ST - 2 : (kTaps - 2 - t < ST - 2 ? (kTaps - 2 - t > 0 ? kTaps - 2 - t : 0) : ST - 2)) * BW + (more && t >= 1 && t <= ST - 1 ? kPatchMin : 0);
      const Frags& fc = t % 2 == 0 ? f0 : f1;
      Frags& fn = t % 2 == 0 ? f1 : f0;
      const uint32_t nxt = cur + kStage < (uint32_t)(ST * kStage) ? cur + kStage : 0u, b_addr = b_lds + nxt;
      if constexpr (read) wait_loads_barrier<younger>();
      static_for<BW>([&](auto L) {
        constexpr int l = decltype(L)::value, b = l * NR / BW, e = (l + 1) * NR / BW, mb = l * NMMA / BW, me = (l + 1) * NMMA / BW;
        if constexpr (load) issue_filter(L, cur);
        if constexpr (read)
          static_for<e - b>([&](auto I) { read_one(std::integral_constant<int, b + decltype(I)::value>{}, std::integral_constant<int, n>{}, b_addr, fn); });
        static_for<me - mb>([&](auto I) { mma_one(std::integral_constant<int, mb + decltype(I)::value>{}, fc); });
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (more && t == 0) {
        static_for<kPatchMin>([&](auto J) {
          constexpr int j = decltype(J)::value;
          issue_patch(j < p_loads - 1 ? j : p_loads - 1, p_soff, next_lds);
        });
        for (int j = kPatchMin; j < p_loads; ++j) issue_patch(j, p_soff, next_lds);
      }
      if constexpr (load) b_soff += (t + ST) % kTaps == kTaps - 1 ? wrap_b : c_bytes;
      cur = nxt;
      if constexpr (more) {
#pragma unroll
        for (int i = 0; i < BM; ++i) a_tap[t][i] += delta;
      }
    });
    if constexpr (more) {
      f0 = f1;
      next_lds -= delta;
      delta = 0u - delta;
      p_soff += KB;
    }
  };
  for (int b = 1; b < blocks; ++b) block(std::true_type{});
  block(std::false_type{});

  if (prof && tid == 0) prof[2] = __builtin_readcyclecounter();
  if (T.split_k > 1 && !split_k_reduce<MT, NT, BM, BN, MF, POL>(T, it, acc, tid, smem, prof)) return;
  tile_epilogue<MT, NT, BM, BN, MF, DT, 1, kSmemBytes, POL>(T, acc, m0, T.M, n0, wm0, wn0, lrow, lk, tid, smem);
  if (prof && tid == 0) stamp_end(prof);
}

// ---- gather tile: channel counts that hold no whole 16-byte vector, and those where its walk is much the shorter one (form_on) -------
// The same implicit GEMM for any C, D steps of loads kept in flight in registers ahead of an LDS double buffer with rows
// padded by 16 bytes.  A vector of the reduction index is contiguous in memory as long as it stays inside one filter row,
// and is then one 16-byte load from an element-aligned address; only vectors that cross into the next filter row, into the
// padding or past the end are put together element by element, by the wavefronts that have any.
// Bound by the texture addresser either way: a 64x64 bf16 step of C = 1023 takes 1140 clocks (3530 with every element loaded
// by itself), of 5x5 with C = 239 1490 (3460), of 3x3 with C = 67, where a third of the steps cross a row, 1940 (2560).
template <int MT, int NT, int WPX, int WCH, int MF, int KB, int D, int DT, class POL = PlainActs>
__device__ __forceinline__ void conv_tile_gather(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr int ES = ElemOf<DT>::ES;
  constexpr int VEC = 16 / ES;          // elements per 16-byte vector
  constexpr int KT = KB / ES;           // elements of K per step
  constexpr int ROWB = KB + 16;         // LDS row pitch: the 16-byte pad spreads rows over all banks
  constexpr int CH = KB / 16;           // 16-byte chunks per row
  constexpr int RPP = kThreads / CH;    // rows staged per pass of the workgroup
  constexpr int WM = MT / WPX, WN = NT / WCH;
  constexpr int BM = WM / MF, BN = WN / MF;
  constexpr int A_IT = (MT + RPP - 1) / RPP, B_IT = (NT + RPP - 1) / RPP;
  constexpr int SUBB = (MF == 32) ? 32 : 64;   // row bytes one MFMA sub-step consumes
  constexpr int NSUB = KB / SUBB;
  static_assert(D % 2 == 0, "D must be even so that register slots and LDS buffers are both static");
  typedef Mma<DT, MF> MMA;
  typedef typename MMA::Acc Acc;
  static_assert(WPX * WCH == 4 && WM % MF == 0 && WN % MF == 0, "bad tile shape");
  static_assert(2 * (MT + NT) * ROWB <= kSmemBytes, "tile does not fit the LDS allocation");

  char* sA = smem;                          // [2][MT][ROWB]  patches
  char* sB = smem + 2 * MT * ROWB;          // [2][NT][ROWB]  filters

  const int tid = work_thread_id();
  if (prof && tid == 0) stamp_start(prof);
  const int chunk = tid % CH;    // which 16 bytes of the row slab this thread stages
  const int row0 = tid / CH;
  const int m0 = (int)it.tile_m * MT;
  const int n0 = (int)it.tile_n * NT;
  const int C = T.C, H = T.H, W = T.W, R = T.R, S = T.S, Kg = T.Kg;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(T.x, T.x_bytes);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(T.w, T.w_bytes);

  // K-step range of this work item; loads at or past klimit are suppressed
  const int ks_begin = (int)it.k_split_idx * T.k_steps_per_split;
  int ks_end = ks_begin + T.k_steps_per_split;
  if (ks_end > T.k_steps) ks_end = T.k_steps;
  const int nsteps = ks_end - ks_begin;
  const int klimit = (ks_end * KT < Kg) ? ks_end * KT : Kg;

  // per-thread patch rows
  int a_base[A_IT], a_h0[A_IT], a_w0[A_IT];
#pragma unroll
  for (int i = 0; i < A_IT; ++i) {
    const int row = row0 + i * RPP;
    const int m = m0 + row;
    const bool ok = (row < MT) && (m < T.M);
    const int mm = ok ? m : 0;
    const int n = fast_div(mm, T.magic_pq, T.shift_pq);
    const int pq = mm - n * T.PQ;
    const int p = fast_div(pq, T.magic_q, T.shift_q);
    const int q = pq - p * T.Q;
    a_h0[i] = ok ? p * T.stride - T.pad : -(1 << 24);   // a dead row fails every bounds check
    a_w0[i] = q * T.stride - T.pad;
    a_base[i] = ((n * H + a_h0[i]) * W + a_w0[i]) * C;
  }
  int b_off[B_IT];
  bool b_ok[B_IT];
#pragma unroll
  for (int i = 0; i < B_IT; ++i) {
    const int row = row0 + i * RPP;
    b_ok[i] = (row < NT) && (n0 + row < T.K);
    b_off[i] = b_ok[i] ? (n0 + row) * Kg : 0;
  }

  // elements of a filter row (s*C + c) that lie inside the image: [a_lo, a_hi)
  const int SC = S * C, WC = W * C;
  int a_lo[A_IT], a_hi[A_IT];
#pragma unroll
  for (int i = 0; i < A_IT; ++i) {
    const int s_lo = a_w0[i] < 0 ? -a_w0[i] : 0, s_hi = W - a_w0[i];
    a_lo[i] = (s_lo < S ? s_lo : S) * C;
    a_hi[i] = (s_hi < 0 ? 0 : s_hi < S ? s_hi : S) * C;
  }

  // position of the next vector this thread will fetch, in the reduction index k = (r*S + s)*C + c
  int k_elem = ks_begin * KT + chunk * VEC;

  u32x4 ra[D][A_IT], rb[D][B_IT];

  // Issue the global loads of the next K step into one register slot, then advance the K position.
  auto issue = [&](u32x4 (&qa)[A_IT], u32x4 (&qb)[B_IT]) {
    const int kr = fast_div(fast_div(k_elem, T.magic_c, T.shift_c), T.magic_s, T.shift_s);
    const int kk = k_elem - kr * SC, koff = kr * WC + kk;
    const bool whole_k = k_elem + VEC <= klimit, one_row = whole_k & (kk + VEC <= SC);
    bool a_part[A_IT], b_part = !whole_k & (k_elem < klimit), any = b_part;
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
      const bool in = one_row & ((unsigned)(a_h0[i] + kr) < (unsigned)H) & (kk >= a_lo[i]) & (kk + VEC <= a_hi[i]);
      // anything of it inside, though not all as one piece
      a_part[i] = !in & (k_elem < klimit) & (a_h0[i] + R > 0) & (!one_row | (((unsigned)(a_h0[i] + kr) < (unsigned)H) & (kk < a_hi[i]) & (kk + VEC > a_lo[i])));
      any |= a_part[i];
      qa[i] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(in ? (uint32_t)(a_base[i] + koff) * ES : kInvalidOffset), 0, POL::kActAux);
    }
#pragma unroll
    for (int i = 0; i < B_IT; ++i)
      qb[i] = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)((b_ok[i] & whole_k) ? (uint32_t)(b_off[i] + k_elem) * ES : kInvalidOffset), 0, 0);
    if (__builtin_expect(__ballot(any) != 0, 0)) {
      uint32_t ea[A_IT][VEC], eb[B_IT][VEC];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const int ke = k_elem + e;
        const bool kin = ke < klimit;
        const bool next = kk + e >= SC;                   // in a later filter row
        const int er = next ? fast_div(fast_div(ke, T.magic_c, T.shift_c), T.magic_s, T.shift_s) : kr;
        const int ek = ke - er * SC;
#pragma unroll
        for (int i = 0; i < A_IT; ++i) {
          const bool ok = a_part[i] & kin & ((unsigned)(a_h0[i] + er) < (unsigned)H) & (ek >= a_lo[i]) & (ek < a_hi[i]);
          const uint32_t off = ok ? (uint32_t)(a_base[i] + er * WC + ek) * ES : kInvalidOffset;
          if constexpr (ES == 4) ea[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rx, (int)off, 0, POL::kActAux);
          else ea[i][e] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rx, (int)off, 0, POL::kActAux);
        }
#pragma unroll
        for (int i = 0; i < B_IT; ++i) {
          const uint32_t off = (b_ok[i] & b_part & kin) ? (uint32_t)(b_off[i] + ke) * ES : kInvalidOffset;
          if constexpr (ES == 4) eb[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rw, (int)off, 0, 0);
          else eb[i][e] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rw, (int)off, 0, 0);
        }
      }
      // a vector is either whole or gathered; the other kind's loads were out of range and gave zeros
#pragma unroll
      for (int i = 0; i < A_IT; ++i) {
        if constexpr (ES == 4) qa[i] |= u32x4{ea[i][0], ea[i][1], ea[i][2], ea[i][3]};
        else qa[i] |= u32x4{ea[i][0] | (ea[i][1] << 16), ea[i][2] | (ea[i][3] << 16), ea[i][4] | (ea[i][5] << 16), ea[i][6] | (ea[i][7] << 16)};
      }
#pragma unroll
      for (int i = 0; i < B_IT; ++i) {
        if constexpr (ES == 4) qb[i] |= u32x4{eb[i][0], eb[i][1], eb[i][2], eb[i][3]};
        else qb[i] |= u32x4{eb[i][0] | (eb[i][1] << 16), eb[i][2] | (eb[i][3] << 16), eb[i][4] | (eb[i][5] << 16), eb[i][6] | (eb[i][7] << 16)};
      }
    }
    k_elem += KT;
  };
  auto store_lds = [&](const u32x4 (&qa)[A_IT], const u32x4 (&qb)[B_IT], int buf) {
#pragma unroll
    for (int i = 0; i < A_IT; ++i) {
      const int row = row0 + i * RPP;
      if (MT % RPP == 0 || row < MT) *(u32x4*)(sA + (buf * MT + row) * ROWB + chunk * 16) = qa[i];
    }
#pragma unroll
    for (int i = 0; i < B_IT; ++i) {
      const int row = row0 + i * RPP;
      if (NT % RPP == 0 || row < NT) *(u32x4*)(sB + (buf * NT + row) * ROWB + chunk * 16) = qb[i];
    }
  };

  // wavefront / lane geometry
  const int lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave % WPX) * WM;
  const int wn0 = (wave / WPX) * WN;
  const int lrow = lane & (MF - 1);
  const int lk = lane / MF;          // 0..1 for 32x32 blocks, 0..3 for 16x16 blocks

  Acc acc[BM][BN];
#pragma unroll
  for (int i = 0; i < BM; ++i)
#pragma unroll
    for (int j = 0; j < BN; ++j)
#pragma unroll
      for (int v = 0; v < (int)(sizeof(Acc) / 4); ++v) acc[i][j][v] = 0.f;

  auto compute = [&](int buf) {
    const char* pa = sA + (buf * MT + wm0 + lrow) * ROWB + lk * 16;
    const char* pb = sB + (buf * NT + wn0 + lrow) * ROWB + lk * 16;
#pragma unroll
    for (int sub = 0; sub < NSUB; ++sub) {
      u32x4 wf[BN], xf[BM];
#pragma unroll
      for (int j = 0; j < BN; ++j) wf[j] = *(const u32x4*)(pb + j * MF * ROWB + sub * SUBB);
#pragma unroll
      for (int i = 0; i < BM; ++i) xf[i] = *(const u32x4*)(pa + i * MF * ROWB + sub * SUBB);
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int j = 0; j < BN; ++j) acc[i][j] = MMA::run(wf[j], xf[i], acc[i][j]);
    }
  };

  if (nsteps > 0) {
    // Steps 0..D-1 go in flight at once; step s lives in register slot s % D.  Steps past the end of the
    // K range load nothing (every lane out of range), so no issue below needs a condition.
    static_for<D>([&](auto J) { issue(ra[decltype(J)::value], rb[decltype(J)::value]); });
    store_lds(ra[0], rb[0], 0);
    issue(ra[0], rb[0]);
    __syncthreads();
    if (prof && tid == 0) prof[1] = __builtin_readcyclecounter();
    // one K step: compute from LDS buffer j&1, meanwhile move step k+1 from its register slot to the
    // other buffer and put step k+1+D in flight in that slot
    auto step = [&](auto J) {
      constexpr int j = decltype(J)::value;
      constexpr int nslot = (j + 1) % D;
      compute(j & 1);
      store_lds(ra[nslot], rb[nslot], (j + 1) & 1);
      issue(ra[nslot], rb[nslot]);
      __syncthreads();
    };
    int k = 0;
    for (; k + D <= nsteps; k += D) static_for<D>(step);     // whole groups: no exits, exact wait counts
    // remainder (fewer than D steps), nested so that each step is reached only through the previous one
    const int rem = nsteps - k;
    static_nest<D - 1>(rem, step);
  }

  if (prof && tid == 0) prof[2] = __builtin_readcyclecounter();

  if (T.split_k > 1 && !split_k_reduce<MT, NT, BM, BN, MF, POL>(T, it, acc, tid, smem, prof)) return;

  // ---- epilogue: (+ residual) -> ReLU -> cast -> store ---------------------------------------------
  tile_epilogue<MT, NT, BM, BN, MF, DT, 1, kSmemBytes, POL>(T, acc, m0, T.M, n0, wm0, wn0, lrow, lk, tid, smem);
  if (prof && tid == 0) stamp_end(prof);
}

// The 128 bits that start kk 16-bit elements into the 256-bit value hi:lo (kk wave-uniform, 0..8).
__device__ __forceinline__ u32x4 window128(const u32x4& lo, const u32x4& hi, int kk) {
  const uint32_t b = (uint32_t)(kk & 1) * 16u;
  uint32_t w0, w1, w2, w3, w4;
  switch (kk >> 1) {
    case 0: w0 = lo[0]; w1 = lo[1]; w2 = lo[2]; w3 = lo[3]; w4 = hi[0]; break;
    case 1: w0 = lo[1]; w1 = lo[2]; w2 = lo[3]; w3 = hi[0]; w4 = hi[1]; break;
    case 2: w0 = lo[2]; w1 = lo[3]; w2 = hi[0]; w3 = hi[1]; w4 = hi[2]; break;
    case 3: w0 = lo[3]; w1 = hi[0]; w2 = hi[1]; w3 = hi[2]; w4 = hi[3]; break;
    default: w0 = hi[0]; w1 = hi[1]; w2 = hi[2]; w3 = hi[3]; w4 = 0u; break;
  }
  return u32x4{__builtin_amdgcn_alignbit(w1, w0, b), __builtin_amdgcn_alignbit(w2, w1, b),
               __builtin_amdgcn_alignbit(w3, w2, b), __builtin_amdgcn_alignbit(w4, w3, b)};
}

// ---- row tile for layers with very few input channels ---------------------------------------------
// For the 7x7 / stride-2 / 3-channel stem the im2col row of one (pixel, filter row r) is S*C = 21
// contiguous elements of the NHWC image, at an odd element offset, so neither 16-byte gathers nor the
// any-channel tile are efficient.  This kernel gives one workgroup up to kRowsPerTile consecutive
// output rows (a segment of up to 128 pixels of each) x 64 filters: the input rows they need are copied
// whole into LDS with 16-byte loads (rows outside the image and the left/right padding are zeros), the
// 64 filters are copied once into an LDS array [filter][r][32] padded with zeros, and the MFMA operands
// are assembled from LDS.  K is laid out as r*32 + (s*C + c).  Eligibility is decided by the planner:
// 16-bit types, 8 <= S*C <= 32, W*C*2 a multiple of 16, stride*C even, LDS footprint.
template <int DT, class POL = PlainActs>
__device__ __forceinline__ void conv_tile_rows(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr int MT = 128, NT = 64, MF = 32, WM = 64, WN = 32, BM = 2, BN = 1, KR = 32;
  const int RT = T.rows_per_tile;                    // output rows per work item (1..kRowsPerTile)
  constexpr int EPI_PASSES = 2;
  // epilogue transposition buffer: the larger of half a tile of fp32 values and a whole tile of 16-bit ones
  constexpr int kStageBytes = kRowStageBytes;
  static_assert(kStageBytes >= (MT / EPI_PASSES) * (NT + 4) * 4 && kStageBytes >= MT * (NT * 2 + 16), "row tile stage buffer");
  typedef Mma<DT, MF> MMA;
  typedef typename MMA::Acc Acc;
  constexpr bool HOLD = POL::kActAux == 0;           // (see rows_held)
  const int tid = work_thread_id();
  if (prof && tid == 0) stamp_start(prof);
  const int lane = tid & 63, wave = tid >> 6;
  const int wm0 = (wave & 1) * WM, wn0 = (wave >> 1) * WN;
  const int lrow = lane & 31, lk = lane >> 5;
  const int C = T.C, H = T.H, W = T.W, R = T.R, S = T.S, P = T.P, Q = T.Q, Kg = T.Kg;
  const int SC = S * C;
  const int qt = (Q + MT - 1) / MT;                 // pixel segments per output row
  const int pg = (P + RT - 1) / RT;                 // row groups per image
  const int npg = (int)it.tile_m / qt;
  const int q0 = ((int)it.tile_m - npg * qt) * MT;
  const int n = npg / pg;
  const int p0 = (npg - n * pg) * RT;
  const int nrows_out = (P - p0 < RT) ? (P - p0) : RT;
  const int n0 = (int)it.tile_n * NT;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(T.x, T.x_bytes);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(T.w, T.w_bytes);

  // LDS: [transposition buffer][NR image rows][filters].  Each image row is [pad*C zeros][W*C elements]
  // [zeros] starting on a 16-byte boundary, so that every pixel's patch (which starts stride*C elements
  // after its neighbour's) is 4-byte aligned.
  const int NR = R + T.stride * (RT - 1);                   // input rows held
  const int lpad = T.pad * C * 2;                           // bytes of left padding
  const int rowb = W * C * 2;                               // bytes of one image row (multiple of 16)
  const int pitch = T.row_pitch;                            // bytes of one LDS row (multiple of 16)
  char* sX = smem + kStageBytes;
  char* sW = sX + NR * pitch;                               // [NT][R][KR] elements
  const int h_first = p0 * T.stride - T.pad;

  // Both arrays are written as whole 16-byte vectors in linear order, each from one 16-byte load at a
  // 2-byte-aligned address; a round of 256 filter vectors covers 64 (filter, filter row) pairs with the
  // position inside the filter row fixed per thread.  An image-row vector that straddles an end of the
  // row data, and the last vector of a filter row, are loaded from the nearest position that lies wholly
  // inside the row and shifted into place (zeros move in), so no load touches bytes outside its own row.
  // All loads of the first round are put in flight before the first LDS write.
  const int nvp = pitch >> 4, total_rv = NR * nvp;
  const int sl = (lpad & 15) >> 1;                          // elements the row data sits past a vector boundary
  const int jl = lpad >> 4, jr = (lpad + rowb) >> 4;        // the two straddling vectors of a row (when sl != 0)
  const int nf = (T.K - n0 < NT) ? (T.K - n0) : NT;
  const int nvec = (SC + 7) >> 3;                           // vectors of a filter row that hold data
  const int kkw = 8 * nvec - SC;                            // elements the last of them is loaded early by
  const int npairs = NT * R;                                // (filter, filter row) pairs
  constexpr int RB = 5, RW = 7;                             // rounds per batch: image-row vectors, filter vectors
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  auto row_base = [&](int r) -> uint32_t { return (uint32_t)((n * H + h_first + r) * W) * (uint32_t)(C * 2); };
  auto row_load = [&](int v, bool& mine) -> u32x4 {
    const int r = fast_div(v, T.magic_nvp, T.shift_nvp), j = v - r * nvp;
    const int sj = 16 * j - lpad;                           // byte position of this vector in the row data
    const bool ok = (v < total_rv) & ((unsigned)(h_first + r) < (unsigned)H) & (sj >= 0) & (sj + 16 <= rowb);
    mine = (v < total_rv) & !((sl != 0) & ((j == jl) | (j == jr)));      // the straddlers are written below
    return __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok ? row_base(r) + (uint32_t)sj : kInvalidOffset), 0, POL::kActAux);
  };
  auto row_store = [&](int v, const u32x4& d, bool mine) {
    if (mine) *(u32x4*)(sX + v * 16) = d;
  };
  const int slot = tid & 3;                                 // 16-byte position inside a padded filter row
  const bool lastslot = slot == nvec - 1;
  const int e0 = lastslot ? SC - 8 : slot * 8;
  const uint32_t mlast = lastslot ? 0xffffffffu : 0u;
  auto w_load = [&](int cr) -> u32x4 {
    const int ch = fast_div(cr, T.magic_r, T.shift_r), r = cr - ch * R;
    const bool live = (slot < nvec) & (cr < npairs) & (ch < nf);
    const uint32_t off = live ? ((uint32_t)(n0 + ch) * (uint32_t)Kg + (uint32_t)(r * SC + e0)) * 2u : kInvalidOffset;
    return __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, 0, 0);
  };
  auto w_store = [&](int cr, u32x4 d) {
    if (kkw != 0) {
      const u32x4 ds = window128(d, zero4, kkw);
#pragma unroll
      for (int e = 0; e < 4; ++e) d[e] = (ds[e] & mlast) | (d[e] & ~mlast);
    }
    if (cr < npairs) *(u32x4*)(sW + (cr * 4 + slot) * 16) = d;
  };
  u32x4 drow[RB], dw[RW], dfix = zero4;
  bool rmine[RB];
  const int fr = tid >> 1, fside = tid & 1;                 // straddler (row, end) handled by this thread
#pragma unroll
  for (int u = 0; u < RB; ++u) drow[u] = row_load(u * kThreads + tid, rmine[u]);
  if (sl != 0) {
    const bool ok = (fr < NR) & ((unsigned)(h_first + fr) < (unsigned)H);
    dfix = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok ? row_base(fr) + (uint32_t)(fside ? rowb - 16 : 0) : kInvalidOffset), 0, POL::kActAux);
  }
#pragma unroll
  for (int u = 0; u < RW; ++u) dw[u] = w_load((tid >> 2) + 64 * u);
#pragma unroll
  for (int u = 0; u < RB; ++u) row_store(u * kThreads + tid, drow[u], rmine[u]);
  for (int v0 = RB * kThreads; v0 < total_rv; v0 += kThreads) {       // wider images: further rounds
    bool mine;
    const u32x4 d = row_load(v0 + tid, mine);
    row_store(v0 + tid, d, mine);
  }
  if (sl != 0) {
    // left end: the data moves up by sl elements; right end: down by 8 - sl; both are the window that starts
    // 8 - sl elements into (data, zeros) resp. (zeros, data)
    const uint32_t ms = fside ? 0xffffffffu : 0u;
    const u32x4 lo = {dfix[0] & ms, dfix[1] & ms, dfix[2] & ms, dfix[3] & ms};
    const u32x4 hi = {dfix[0] & ~ms, dfix[1] & ~ms, dfix[2] & ~ms, dfix[3] & ~ms};
    const u32x4 d = window128(lo, hi, 8 - sl);
    if (fr < NR) *(u32x4*)(sX + fr * pitch + (fside ? jr : jl) * 16) = d;
  }
#pragma unroll
  for (int u = 0; u < RW; ++u) w_store((tid >> 2) + 64 * u, dw[u]);
  for (int c0 = 64 * RW; c0 < npairs; c0 += 64 * RW) {     // taller filters
#pragma unroll
    for (int u = 0; u < RW; ++u) dw[u] = w_load(c0 + (tid >> 2) + 64 * u);
#pragma unroll
    for (int u = 0; u < RW; ++u) w_store(c0 + (tid >> 2) + 64 * u, dw[u]);
  }
  __syncthreads();
  if (prof && tid == 0) prof[1] = __builtin_readcyclecounter();

  // per-lane masks that clear the elements at or past S*C (they belong to the next pixel)
  uint32_t msk[2][4];
#pragma unroll
  for (int half = 0; half < 2; ++half)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int j = 16 * half + 8 * lk + 2 * d;
      msk[half][d] = (j < SC ? 0x0000ffffu : 0u) | (j + 1 < SC ? 0xffff0000u : 0u);
    }
  const int nh = (SC + 15) >> 4;     // 16-element halves of a filter row that hold data
  int qa[BM];
#pragma unroll
  for (int i = 0; i < BM; ++i) {
    int q = q0 + wm0 + i * MF + lrow;
    q = q < Q ? q : Q - 1;           // columns past the row end repeat the last pixel; they are never stored
    qa[i] = q * T.stride * C * 2 + lk * 16;
  }
  const char* wrow = sW + (wn0 + lrow) * R * (KR * 2) + lk * 16;
  const int q_end = (q0 + MT < Q) ? q0 + MT : Q;
  // operands of one (filter row, half): the filter vector and BM masked pixel vectors
  struct Ops { u32x4 xf[BM]; };
  auto fetch_w = [&](auto HALF, int r) -> u32x4 { return *(const u32x4*)(wrow + r * (KR * 2) + decltype(HALF)::value * 32); };
  auto fetch = [&](auto HALF, int rt, int r, Ops& o) {
    constexpr int half = decltype(HALF)::value;
    const char* xr = sX + (rt * T.stride + r) * pitch + half * 32;
#pragma unroll
    for (int i = 0; i < BM; ++i) {
      const uint32_t* src = (const uint32_t*)(xr + qa[i]);
      o.xf[i] = u32x4{src[0], src[1], src[2], src[3]};
    }
  };
  // masking is left to the point of use, so that the LDS reads stay in flight behind the other half's MFMAs
  auto mma = [&](auto HALF, auto NH, const u32x4& wf, const Ops& o, Acc (&acc)[BM][BN]) {
    constexpr int half = decltype(HALF)::value;
    constexpr bool LAST = half + 1 == decltype(NH)::value;       // (an earlier half is full)
#pragma unroll
    for (int i = 0; i < BM; ++i) {
      u32x4 xf = o.xf[i];
      if (LAST) xf = u32x4{xf[0] & msk[half][0], xf[1] & msk[half][1], xf[2] & msk[half][2], xf[3] & msk[half][3]};
      acc[i][0] = MMA::run(wf, xf, acc[i][0]);
    }
  };
  // One output row after another: row(rt, acc) adds up its pixels.
  auto each_row = [&](auto row) {
    for (int rt = 0; rt < nrows_out; ++rt) {
      Acc acc[BM][BN];
#pragma unroll
      for (int i = 0; i < BM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][0][v] = 0.f;
      row(rt, acc);
      const int mrow = (n * P + p0 + rt) * Q;
      tile_epilogue<MT, NT, BM, BN, MF, DT, EPI_PASSES, kStageBytes, POL, false>(T, acc, mrow + q0, mrow + q_end, n0, wm0, wn0, lrow, lk, tid, smem);
    }
  };
  // Seven filter rows of two halves, the usual stem: the filters stay in registers for all output rows of the item, and the
  // pixels of the next filter row are fetched from LDS while the MFMAs of the current one run.  What bounds it is still the
  // latency of those reads and of the epilogue's two barriers: an output row of 128 pixels x 64 filters beside a second
  // workgroup 6270 clocks (filters read again for every row, a loop over the filter rows) -> 4750, of which the MFMAs are 900; eight
  // stems of batch 8 60.8 us -> 51.6.  Not in a chain: its one kernel has no registers to spare for it (eight networks of
  // batch 1 346 us -> 351).
  auto rows_held = [&](auto RN, auto NH) {
    constexpr int rows = decltype(RN)::value, halves = decltype(NH)::value;
    u32x4 w[rows][halves];
    static_for<rows>([&](auto RR) {
      static_for<halves>([&](auto HALF) { w[decltype(RR)::value][decltype(HALF)::value] = fetch_w(HALF, decltype(RR)::value); });
    });
    each_row([&](int rt, Acc (&acc)[BM][BN]) {
      Ops o[2][halves];
      static_for<halves>([&](auto HALF) { fetch(HALF, rt, 0, o[0][decltype(HALF)::value]); });
      static_for<rows>([&](auto RR) {
        constexpr int r = decltype(RR)::value;
        if constexpr (r + 1 < rows) static_for<halves>([&](auto HALF) { fetch(HALF, rt, r + 1, o[(r + 1) & 1][decltype(HALF)::value]); });
        __builtin_amdgcn_sched_barrier(0);
        static_for<halves>([&](auto HALF) { mma(HALF, NH, w[r][decltype(HALF)::value], o[r & 1][decltype(HALF)::value], acc); });
        __builtin_amdgcn_sched_barrier(0);
      });
    });
  };
  // Any number of filter rows: operands of the next half step are fetched while the MFMAs of the current one run; the loop
  // exists once per number of halves so that its body is free of branches.
  auto rows_streamed = [&](auto NH) {
    constexpr int halves = decltype(NH)::value;
    each_row([&](int rt, Acc (&acc)[BM][BN]) {
      Ops o0, o1;
      u32x4 w0, w1;
      auto first = [&](int r) { w0 = fetch_w(std::integral_constant<int, 0>{}, r); fetch(std::integral_constant<int, 0>{}, rt, r, o0); };
      first(0);
      for (int r = 0; r < R; ++r) {
        if constexpr (halves > 1) { w1 = fetch_w(std::integral_constant<int, 1>{}, r); fetch(std::integral_constant<int, 1>{}, rt, r, o1); }
        mma(std::integral_constant<int, 0>{}, NH, w0, o0, acc);
        first((r + 1 < R) ? r + 1 : r);      // the last time filter row R - 1 again instead of a branch around the reads
        if constexpr (halves > 1) mma(std::integral_constant<int, 1>{}, NH, w1, o1, acc);
      }
    });
  };
  const std::integral_constant<int, 1> one{};
  const std::integral_constant<int, 2> two{};
  if (HOLD && R == 7 && nh > 1) {
    if constexpr (HOLD) rows_held(std::integral_constant<int, 7>{}, two);
  } else if (nh > 1) {
    rows_streamed(two);
  } else {
    rows_streamed(one);
  }
  if (prof && tid == 0) {
    prof[2] = __builtin_readcyclecounter();
    stamp_end(prof);
  }
}

// ---- max-pool of one output vector -----------------------------------------------------------------
// NHWC max-pool, one 16-byte vector of channels of one output pixel: idx counts (n, p, q, channel vector) with the
// channel vector fastest.  Padding never wins; the result is a copy of the winning input's bits.
// AUX: cache policy of the input loads (0: through the caches; kAuxDeviceCoherent: device-scope loads, for an input
// that other workgroups of the same launch wrote); x_bytes is the size of the input; it and the output's are below 2^31, so
// 32 bits are enough for everything (64-bit divisions are hundreds of instructions).
template <int DT, int AUX = 0>
__device__ __forceinline__ u32x4 maxpool_vector(const void* __restrict__ xv, uint32_t x_bytes, uint32_t idx, int H, int W, int C, int P,
                                                int Q, int win, int stride, int pad) {
  constexpr int ES = ElemOf<DT>::ES, VEC = 16 / ES;
  const uint32_t CV = (uint32_t)C / VEC, cv = idx % CV, pixel = idx / CV, pq = pixel / (uint32_t)Q;
  const int q = (int)(pixel - pq * (uint32_t)Q), n = (int)(pq / (uint32_t)P), p = (int)(pq - (uint32_t)n * (uint32_t)P);
  float best[VEC];
  uint32_t bits[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) { best[e] = 0.f; bits[e] = 0u; }
  bool any = false;
  // The taps are visited row by row as a plain loop would, but nine at a time: all nine loads are issued before the
  // first is looked at (taps outside the image or past the window get an out-of-range offset and are skipped), so a
  // 3x3 window costs one memory round trip, not nine.
  constexpr int B = 9;
  const __amdgpu_buffer_rsrc_t rx = make_rsrc(xv, x_bytes);
  const int taps = win * win;
  int r = 0, sx = 0;
  for (int t0 = 0; t0 < taps; t0 += B) {
    u32x4 raw[B];
    bool ok[B];
#pragma unroll
    for (int u = 0; u < B; ++u) {
      const int h = p * stride - pad + r, w = q * stride - pad + sx;
      ok[u] = (t0 + u < taps) & ((unsigned)h < (unsigned)H) & ((unsigned)w < (unsigned)W);
      const uint32_t xoff = ((uint32_t)((n * H + h) * W + w) * (uint32_t)C + cv * VEC) * ES;
      raw[u] = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ok[u] ? xoff : kInvalidOffset), 0, AUX);
      if (++sx == win) { sx = 0; ++r; }
    }
#pragma unroll
    for (int u = 0; u < B; ++u) {
      if (!ok[u]) continue;
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        uint32_t b;
        float v;
        if constexpr (ES == 4) {
          b = raw[u][e];
          v = __builtin_bit_cast(float, b);
        } else {
          b = (raw[u][e >> 1] >> (16 * (e & 1))) & 0xffffu;
          v = (DT == ST_DT_BF16) ? bf16_bits_to_f32((uint16_t)b) : f16_bits_to_f32((uint16_t)b);
        }
        if (!any || v > best[e]) { best[e] = v; bits[e] = b; }
      }
      any = true;
    }
  }
  if constexpr (ES == 4) return u32x4{bits[0], bits[1], bits[2], bits[3]};
  else return u32x4{bits[0] | (bits[1] << 16), bits[2] | (bits[3] << 16), bits[4] | (bits[5] << 16), bits[6] | (bits[7] << 16)};
}

// One max-pool work item: kThreads output vectors, stored write-through.
template <int DT, class POL>
__device__ __forceinline__ void pool_item(ConstOp& T, const st_work_item it) {
  const uint32_t idx = it.tile_m * (uint32_t)kThreads + (uint32_t)work_thread_id();
  if (idx >= (uint32_t)T.M) return;
  const u32x4 v = maxpool_vector<DT, POL::kActAux>(T.x, T.x_bytes, idx, T.H, T.W, T.C, T.P, T.Q, T.R, T.stride, T.pad);
  __builtin_amdgcn_raw_buffer_store_b128(v, make_rsrc(T.y, T.y_bytes), (int)(idx * 16u), 0, POL::kOutAux);
}

template <int CFG, int DT, class POL>
__device__ __forceinline__ void vector_tile(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr TileShape s = kTileShapes[CFG];
  conv_tile<s.MT, s.NT, s.WPX, s.WCH, s.MF, s.KB, s.D, DT, false, POL>(T, it, smem, prof);
}
template <int CFG, int DT, class POL>
__device__ __forceinline__ void patch_tile(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr TileShape s = kTileShapes[CFG];
  if constexpr (DT != ST_DT_F32) conv_tile_patch<s.MT, s.NT, s.WPX, s.WCH, s.MF, s.KB, kPatchStages[CFG], DT, POL>(T, it, smem, prof);
}
template <int CFG, int DT, class POL>
__device__ __forceinline__ void pieces_tile(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr TileShape s = kTileShapes[CFG];
  conv_tile<s.MT, s.NT, s.WPX, s.WCH, s.MF, s.KB, s.D, DT, true, POL>(T, it, smem, prof);
}
template <int CFG, int DT, class POL>
__device__ __forceinline__ void gather_tile(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr TileShape s = kTileShapes[CFG];
  conv_tile_gather<s.MT, s.NT, s.WPX, s.WCH, s.MF, 128, CFG == 1 ? 2 : 4, DT, POL>(T, it, smem, prof);
}

template <uint32_t HAS, int DT, class POL>
__device__ __forceinline__ void run_form(uint32_t form, ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr bool rows = (HAS & kHasRows) != 0u && DT != ST_DT_F32, gather = (HAS & kHasGather) != 0u, patch = DT != ST_DT_F32;
  switch (form) {
    case kFormVector + 0: vector_tile<0, DT, POL>(T, it, smem, prof); break;
    case kFormVector + 1: vector_tile<1, DT, POL>(T, it, smem, prof); break;
    case kFormVector + 2: vector_tile<2, DT, POL>(T, it, smem, prof); break;
    case kFormVector + 3: vector_tile<3, DT, POL>(T, it, smem, prof); break;
    case kFormVector + 4: vector_tile<4, DT, POL>(T, it, smem, prof); break;
    case kFormVector + 5: vector_tile<5, DT, POL>(T, it, smem, prof); break;
    case kFormPatch + 1: if constexpr (patch) patch_tile<1, DT, POL>(T, it, smem, prof); break;
    case kFormPatch + 2: if constexpr (patch) patch_tile<2, DT, POL>(T, it, smem, prof); break;
    case kFormPatch + 3: if constexpr (patch) patch_tile<3, DT, POL>(T, it, smem, prof); break;
    case kFormPatch + 4: if constexpr (patch) patch_tile<4, DT, POL>(T, it, smem, prof); break;
    case kFormGather + 1: if constexpr (gather) gather_tile<1, DT, POL>(T, it, smem, prof); break;
    case kFormGather + 3: if constexpr (gather) gather_tile<3, DT, POL>(T, it, smem, prof); break;
    case kFormPieces + 1: if constexpr (gather) pieces_tile<1, DT, POL>(T, it, smem, prof); break;
    case kFormPieces + 3: if constexpr (gather) pieces_tile<3, DT, POL>(T, it, smem, prof); break;
    case kFormPieces + 4: if constexpr (gather) pieces_tile<4, DT, POL>(T, it, smem, prof); break;
    case kFormPieces + 5: if constexpr (gather) pieces_tile<5, DT, POL>(T, it, smem, prof); break;
    case kFormRows: if constexpr (rows) conv_tile_rows<DT, POL>(T, it, smem, prof); break;
    case kFormPool:
      if constexpr ((HAS & kHasPools) != 0u) {
        if (prof && threadIdx.x == 0) stamp_start(prof);
        pool_item<DT, POL>(T, it);
        if (prof && threadIdx.x == 0) stamp_end(prof);
      }
      break;
    default: break;
  }
}

// One work item of a plan or chain: a tile of a convolution, or (chains only) a max-pool item.  it.reserved is its code word.
template <uint32_t HAS, class POL>
__device__ __forceinline__ void run_item(ConstOp& T, const st_work_item it, char* smem, uint64_t* prof) {
  constexpr uint32_t types = HAS & 7u;
  const uint32_t form = it.reserved & kFormMask;
  if constexpr (types == 1u << ST_DT_BF16) run_form<HAS, ST_DT_BF16, POL>(form, T, it, smem, prof);
  else if constexpr (types == 1u << ST_DT_F16) run_form<HAS, ST_DT_F16, POL>(form, T, it, smem, prof);
  else if constexpr (types == 1u << ST_DT_F32) run_form<HAS, ST_DT_F32, POL>(form, T, it, smem, prof);
  else {
    switch (it.reserved >> kFormTypeShift) {
      case ST_DT_BF16: run_form<HAS, ST_DT_BF16, POL>(form, T, it, smem, prof); break;
      case ST_DT_F16: run_form<HAS, ST_DT_F16, POL>(form, T, it, smem, prof); break;
      default: run_form<HAS, ST_DT_F32, POL>(form, T, it, smem, prof); break;
    }
  }
}

}  // namespace st
