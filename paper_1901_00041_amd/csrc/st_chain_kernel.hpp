// The fused space-time policy over a whole chain of dependent layers as ONE persistent launch (gfx950).
//
// Section 4 merges the ready kernels of disjoint DNN graphs into super-kernels; a launch per layer still pays, per
// layer, the launch gap, the ramp of a fresh grid and the drain of its slowest tile.  Here every tenant's whole
// sequence of layers is worked through by a fixed set of resident workgroups; an entry of sequence q and stage s may
// start once every work item of q's earlier stages is complete, so a tenant's next layer starts the moment its own
// previous layer is done, while other tenants' tiles fill the slots that its stragglers leave idle.  The entries lie
// either in columns per XCD (8 sequences or more: see st_chain_kernel) or, on request, in one queue in (stage, cost)
// order that the workgroups claim entry by entry with one atomic each.  (The default with fewer than 8 sequences is
// neither: a launch of st_conv_kernel per stage, in which the sequences are in lock-step.)
//
// Progress: an entry depends only on earlier stages.  One queue: entries are claimed strictly in stage order, so the
// lowest unfinished entry is always held by a running workgroup whose dependencies are complete; no co-residency of
// all workgroups is needed.  Columns: each is worked through in stage order, and every column in use needs its
// workgroup.  Every wait is bounded twice over: by a wall-clock limit and by a count of polls; when
// either expires the waiter raises the abort flag; a workgroup that sees it claims no further entry, and works through the
// rest of its column with waits of a few looks.  A workgroup also takes at most n_items + 1 entries.  So the kernel always exits,
// whatever the clock or the counters do.
//
// Memory: consumers read activations, residuals and partial tiles with device-scope loads, which never stop at a vector
// cache and take from an L2 what that L2 holds newer than memory, so no cache is ever invalidated.  Producers wait for
// their stores before they signal: with one queue they write through to memory (CoherentActs), with queues per XCD, where
// all of a sequence's readers share their L2, to that L2 (LocalActs).  Eight networks, us per pass written through and to the
// L2: batch 1 361 -> 353, batch 3 597 -> 596, batch 8 1142 -> 1137.  (The workgroup-scope invalidate does nothing for a workgroup that sits on one compute unit, and
// the device-scope one also empties the XCD's L2 of the filters: measured 1-2 us per work item.)  The signal is,
// with one queue for the chip, a device-scope atomic on the sequence's counter; with queues per XCD, where producer
// and consumer share one L2, a plain store of the run's number into the work item's own flag, which the consumer's
// polls then find in that L2 (0.25 us from store to sight, against 0.6 us and more through memory).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "st_chain_args.h"
#include "st_internal.h"
#include "st_tiles.hpp"

namespace st {

constexpr int kChainGraceLooks = 24;             // looks at a dependency (0.3 us each) before the abort flag and the clock are looked at
// Looks after which a wait of at most `limit` ticks of 10 ns ends whatever the clock says.  A look takes 0.2 us at the least (a load
// from the L2 and the pause), so one per 80 ns of the limit cannot end it early.
__device__ __forceinline__ uint32_t max_polls(uint32_t limit) { return (limit >> 3) + 64u; }

// Nothing counts as invariant inside the loop over work items, which has stores, atomics and barriers in it: what never
// changes while a launch runs is read through the constant address space.
typedef __attribute__((address_space(4))) const ChainPrefetch ConstPrefetch;

// Filters are read from memory exactly once per pass (376 MB for eight 53-layer networks: more than the memory-side cache
// holds) and do not depend on any earlier layer, and a small stage's tiles wait for them more than for anything else.  So
// workgroups that wait with nothing to do pull a stage's filters into their XCD's L2 while the stage before it runs: each
// of the kChainColumns workgroups with a shared column touches its share of the 128-byte lines of w.  The touches are
// spread out on purpose, one line per lane and round trip: in one burst they delay the running stage's own loads.
// Eight networks of batch 1, us per pass: no prefetch 411, 256 threads with four lines each in flight 394, with one line
// 388, 128 threads 378, 64 threads 380; batch 8: 1333, 1255, 1249, 1246, 1273.
constexpr uint32_t kPrefetchLanes = 128u;
__device__ __forceinline__ void prefetch_filters(ConstOp& T, uint32_t rank, int tid) {      // threads below kPrefetchLanes
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(T.w, T.w_bytes);
  const uint32_t w_bytes = T.w_bytes;
  for (uint32_t off = (rank * kPrefetchLanes + (uint32_t)tid) * 128u; off < w_bytes; off += (uint32_t)kChainColumns * kPrefetchLanes * 128u) {
    const uint32_t v = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rw, (int)off, 0, 0);
    asm volatile("" ::"v"(v));
  }
}

// The flags an entry waits for: [gate, gate + n_gate) and [tiles, tiles + n - n_gate), looked at as one list of n.
struct FlagList { uint32_t gate, n_gate, tiles, n; };

// Whether flags c0 .. n - 1 of the list all hold the run's number (one wavefront, uniform); c0 moves past those found set.  64
// flags at a time, or 256 while that many are left.
__device__ __forceinline__ bool flags_set(const uint32_t* item_flags, const FlagList& l, uint32_t run, uint32_t lane, uint32_t& c0) {
  auto flag = [&](uint32_t c) { return __hip_atomic_load(item_flags + (c < l.n_gate ? l.gate + c : l.tiles + (c - l.n_gate)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  while (c0 + 64u < l.n) {
    constexpr int G = 4;
    uint32_t v[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const uint32_t c = c0 + 64u * g + lane;
      v[g] = flag(c < l.n ? c : l.n - 1u);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
      if (__builtin_amdgcn_ballot_w64(v[g] != run) != 0ull) return false;
      c0 += 64u;
    }
  }
  if (c0 < l.n) {
    const uint32_t c = c0 + lane;
    const bool unset = (c < l.n) && flag(c) != run;
    if (__builtin_amdgcn_ballot_w64(unset) != 0ull) return false;
    c0 = l.n;
  }
  return true;
}

// Whether the pass has been abandoned (uniform in a wavefront).
__device__ __forceinline__ bool abandoned(const ChainArgs& a) {
  return __builtin_amdgcn_readfirstlane(__hip_atomic_load(&a.ctl[kChainCtlAbort * kChainCtlStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) != 0u;
}

// A wavefront gives the pass up: the flag that the pass's workgroups look at, the one that outlives it, and one off the count of
// completed items, since wavefront 0 of the workgroup may call the item complete all the same (it can see the last flag just then).
__device__ __forceinline__ void abandon(const ChainArgs& a) {
  __hip_atomic_store(&a.ctl[kChainCtlLost * kChainCtlStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(&a.ctl[kChainCtlAbort * kChainCtlStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_fetch_sub(&a.ctl[kChainCtlDone * kChainCtlStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether the stage before prefetch entry pf's has started, i.e. the stage before that one is complete.
__device__ __forceinline__ bool prefetch_due(const ChainArgs& a, uint32_t pf, uint32_t lane, uint32_t& c0) {
  ConstPrefetch& p = ((ConstPrefetch*)a.prefetch)[pf];
  return flags_set(a.item_flags, FlagList{p.gate_begin, p.gate_count, 0u, p.gate_count}, a.run_number, lane, c0);
}

// Next position of queue q for this workgroup (thread 0 only); past the end once the pass has been abandoned.
__device__ __forceinline__ uint32_t chain_claim(const ChainArgs& a, uint32_t q, uint32_t qb, uint32_t qe) {
  uint32_t idx = qb + __hip_atomic_fetch_add(&a.ctl[(kChainCtlHead + q) * kChainCtlStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (idx >= qe || __hip_atomic_load(&a.ctl[kChainCtlAbort * kChainCtlStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) idx = 0xffffffffu;
  return idx;
}

// With queues per XCD, an XCD's entries are dealt into 2 x kChainColumns COLUMNS, each a list of entries in stage
// order, and every workgroup works through ONE column that it draws when it starts (one atomic): nothing is claimed
// per entry, so no round trip to memory stands between a finished entry and the workgroup's next one.  Two
// workgroups fit a compute unit, and two tiles that share one run 20-45 % slower each than a tile that has it to
// itself; a stage of a sequence often has no more tiles than the XCD has compute units.  So the first workgroup to
// arrive on a compute unit draws one of the kChainColumns EXCLUSIVE columns and every later one a SHARED column, and
// the host deals a stage's entries (longest first) to the exclusive columns first, to the shared ones only beyond
// one per compute unit.  Every column that holds entries needs a workgroup: should fewer become resident on an XCD
// than it has columns in use, the entries of the columns nobody drew stay undone, their dependants' waits expire,
// and the pass is abandoned and reported.  (The one-queue form, whose entries are claimed one by one, completes with
// any number of resident workgroups.)
//
// COLUMNS: this form.  Otherwise one queue, claimed entry by entry (what goes with either, signals and stores, is then known
// when the kernel is compiled).
template <uint32_t HAS, bool COLUMNS>
__global__ __launch_bounds__(kThreads, 2) void st_chain_kernel(const ChainArgs a) {
  __shared__ __attribute__((aligned(16))) char smem[kSmemBytes];
  uint32_t* s_msg = (uint32_t*)smem;      // between work items only: read, then a barrier, before a tile or the next message
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {
    // the control block of the NEXT run (runs alternate between two blocks; the stream orders them), but for the slots that are
    // st_chain_aborted's to clear
    for (uint32_t i = (uint32_t)tid; i < a.ctl_slots; i += kThreads)
      if (i == (uint32_t)kChainCtlAbort || i >= (uint32_t)kChainCtlHead) __hip_atomic_store(&a.ctl_other[i * kChainCtlStride], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 64) __hip_atomic_fetch_add(&a.ctl[kChainCtlStarted * kChainCtlStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (uint32_t i = (uint32_t)tid; i < (uint32_t)kChainRankWords; i += kThreads)
      __hip_atomic_store(&a.ctl_other[a.ctl_slots * kChainCtlStride + i], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  // the entries of this workgroup: [qb, qe) of the work list; one queue: claimed one by one from all of it
  constexpr bool claiming = !COLUMNS, by_flags = COLUMNS;
  uint32_t qb = 0u, qe = a.q_end;
  uint32_t pf = 0u, pf_end = 0u, rank = 0u;     // filters still to prefetch (shared columns only), and this workgroup's share
  if (!claiming) {
    const uint32_t xcc = (uint32_t)__builtin_amdgcn_s_getreg(0x1814) & 15u;       // XCC_ID
    if (xcc >= a.n_queues) {
      // an XCD this launch was not planned for: its workgroups must not touch any entry (completion flags are only
      // valid inside one XCD); the pass is reported as abandoned
      if (tid == 0) abandon(a);
      return;
    }
    if (tid == 0) {
      // shader engine, shader array and compute unit of HW_ID: one of kChainRankWords / kNumXCDs keys per XCD
      const uint32_t cu = ((uint32_t)__builtin_amdgcn_s_getreg(0xF804) >> 8) & 255u;
      const uint32_t arrived = __hip_atomic_fetch_add(&a.ctl[a.ctl_slots * kChainCtlStride + xcc * 256u + cu], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint32_t cls = arrived != 0u ? 1u : 0u;
      const uint32_t drawn = __hip_atomic_fetch_add(&a.ctl[(kChainCtlHead + 2u * xcc + cls) * kChainCtlStride], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_msg[0] = drawn < (uint32_t)kChainColumns ? xcc * 2u * kChainColumns + cls * kChainColumns + drawn : 0xffffffffu;
    }
    __syncthreads();
    const uint32_t col = __builtin_amdgcn_readfirstlane(s_msg[0]);
    __syncthreads();
    if (col == 0xffffffffu) return;        // every column of this kind has its workgroup
    const __attribute__((address_space(4))) uint32_t* cb = (const __attribute__((address_space(4))) uint32_t*)(a.colbegin + col);
    qb = cb[0];
    qe = cb[1];
    const uint32_t in_xcd = col - xcc * 2u * kChainColumns;
    if (in_xcd >= (uint32_t)kChainColumns) {
      rank = in_xcd - (uint32_t)kChainColumns;
      pf = a.prefetch_begin[xcc];
      if (__builtin_amdgcn_readfirstlane((uint32_t)tid) < kPrefetchLanes) pf_end = a.prefetch_begin[xcc + 1u];
    }
  }
  uint32_t n_done = 0u;
  bool gave_up = false;                         // per wavefront
  uint32_t seen_key = 0xffffffffu, seen_need = 0u;      // the dependency (with flags: the gate) this workgroup last saw complete
  uint32_t seen_begin = 0u, seen_end = 0u;              // ... and the range of tiles
  {
    uint32_t next = 0xffffffffu;            // one queue, thread 0: the entry claimed ahead
    if (claiming && tid == 0) next = chain_claim(a, 0u, qb, qe);
    for (uint32_t round = 0; round <= qe - qb; ++round) {
      uint32_t idx = qb + round;
      if (claiming) {
        if (tid == 0) s_msg[0] = next;
        __syncthreads();
        idx = __builtin_amdgcn_readfirstlane(s_msg[0]);
        __syncthreads();
      }
      if (idx >= qe) break;
      ConstItem* ip = (ConstItem*)(a.items + idx);
      st_work_item it;
      it.tenant = ip->tenant;
      it.k_split_idx = ip->k_split_idx;
      it.tile_m = ip->tile_m;
      it.tile_n = ip->tile_n;
      it.reserved = ip->reserved;
      ConstOp& T = *(ConstOp*)(a.ops + it.tenant);
      uint64_t* prof = a.prof ? a.prof + (size_t)idx * kProfSlots : nullptr;
      uint64_t waited = 0;
      // one word of every 64-byte line of the op record, requested before the dependency wait and used after it, so
      // that the record sits in the scalar cache when the tile code reads its fields
      const uint32_t rec_touch = (uint32_t)(uintptr_t)T.x ^ (uint32_t)T.R ^ (uint32_t)T.tiles_m ^ T.x_bytes ^ T.chain_flag_base;
      // What this workgroup has seen complete need not be looked at again: the gate of its earlier entries of this stage, and
      // their tiles (the items of one pixel tile often follow each other in a column).
      const uint32_t key = by_flags ? T.chain_dep_begin : (uint32_t)T.chain_seq;
      const bool gate_seen = key == seen_key && T.chain_need <= seen_need;
      FlagList wanted{0u, 0u, 0u, 0u};
      if (by_flags) {
        const __attribute__((address_space(4))) ChainDep& d = ((const __attribute__((address_space(4))) ChainDep*)a.deps)[idx];
        const uint32_t begin = d.begin, count = d.count;
        wanted.gate = T.chain_dep_begin;
        wanted.n_gate = gate_seen ? 0u : T.chain_dep_count;
        wanted.tiles = begin;
        wanted.n = wanted.n_gate + (begin >= seen_begin && begin + count <= seen_end ? 0u : count);
      }
      if (T.chain_need != 0u && (by_flags ? wanted.n != 0u : !gate_seen)) {
        // Look at the dependency: with flags, at those of the gate and of the tiles the entry reads (ChainDep),
        // 64 at a time from the first that was not yet set (they were stored by workgroups of this XCD and sit, newer than
        // memory, in its L2, where a device-scope load finds them; such a load never stops at the vector cache); with a
        // counter, at the sequence's count of finished entries (bumped by device-scope atomics, carried out at the
        // memory side; a workgroup-scope load would stop at the vector cache and never see it move).
        const uint32_t run = a.run_number, need = T.chain_need;
        const uint32_t* ctr = a.ctl + (kChainCtlSeq + T.chain_seq) * kChainCtlStride;
        const uint32_t lane = (uint32_t)work_thread_id() & 63u;
        uint32_t c0 = 0u;                     // flags before c0 are known to be set
        auto satisfied = [&]() -> bool {      // uniform in a wavefront
          if (!by_flags) return (int32_t)(__builtin_amdgcn_readfirstlane(__hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) - need) >= 0;
          return flags_set(a.item_flags, wanted, run, lane, c0);
        };
        // Columns: every wavefront looks for itself, so that neither a message through LDS nor a barrier stands between the flag that ends
        // the wait and the tile (one wavefront looking for all: eight networks of batch 1 346 us, of batch 8 1107; each for
        // itself 335 and 1095; how long a wavefront pauses between looks, 64 or 128 clocks, changes neither).  In between, filters of coming stages may be due (pf).  A wavefront that gives up goes on as if
        // the wait had ended, so that the barriers of all four stay in step: every access is checked against the tensors' sizes,
        // and what is computed is lost with the pass, which the abort flag reports; a later wait of its that is not over at once ends
        // when the flag is next looked at, after a few looks (knowing that it gave up costs every wait: 325 us -> 333).
        // One queue: wavefront 0 looks for all; four looking at a counter at the memory side slow each other down (670 us -> 719).
        const uint64_t t0 = wall_clock64();
        uint32_t polls = 0u, p0 = 0u;
        if (COLUMNS || tid < 64) {
          while (!satisfied()) {
            if (pf < pf_end && prefetch_due(a, pf, lane, p0)) {
              prefetch_filters(*(ConstOp*)(a.ops + ((ConstPrefetch*)a.prefetch)[pf].op), rank, tid);
              ++pf;
              p0 = 0u;
              continue;
            }
            // the abort flag and the clock are looked at on every 16th poll (every few microseconds) after the first looks
            if ((++polls & 15u) != 0u || polls <= (uint32_t)kChainGraceLooks) { __builtin_amdgcn_s_sleep(1); continue; }
            if (__builtin_expect(abandoned(a) || wall_clock64() - t0 > (uint64_t)a.spin_limit || polls > max_polls(a.spin_limit), 0)) {
              if (lane == 0u) abandon(a);
              gave_up = true;
              break;
            }
            __builtin_amdgcn_s_sleep(1);
          }
        }
        if (!COLUMNS) __syncthreads();
        else asm volatile("" ::: "memory");   // no barrier, but the compiler may not move a load of the tile's before the looks either
        waited = wall_clock64() - t0;
        // No cache is invalidated here: everything an entry reads that this launch wrote (activations, residuals,
        // split-K partial tiles) is read with device-scope loads, and everything else did not change.
        if (T.chain_dep_count != 0u) {        // (an empty range has no beginning to be known by)
          seen_key = key;
          seen_need = T.chain_need;
        }
        if (wanted.n != wanted.n_gate) {
          seen_begin = wanted.tiles;
          seen_end = wanted.tiles + (wanted.n - wanted.n_gate);
        }
      }
      while (pf < pf_end && ((ConstPrefetch*)a.prefetch)[pf].flag_base <= T.chain_flag_base) ++pf;      // too late to prefetch these
      asm volatile("" ::"s"(rec_touch));
      run_item<HAS, std::conditional_t<COLUMNS, LocalActs, CoherentActs>>(T, it, smem, prof);
      // Completion.  With one queue outputs were stored write-through; channel counts that are not a multiple of 8 take an
      // epilogue with plain stores and need the release fence (write-back of the L2).
      if (!COLUMNS && (it.reserved & kFormMask) != kFormPool && (T.K & 7) != 0) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      __builtin_amdgcn_s_waitcnt(0);          // every store of this thread has been acknowledged
      __syncthreads();                        // ... of every thread; also: smem and s_msg are free again
      if (!gave_up) ++n_done;
      if (tid == 0 && !gave_up) {
        if (by_flags) {
          const uint32_t pos = ((uint32_t)it.tile_m * (uint32_t)T.tiles_n + (uint32_t)it.tile_n) * (uint32_t)T.split_k + (uint32_t)it.k_split_idx;
          __hip_atomic_store(a.item_flags + T.chain_flag_base + pos, a.run_number, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        } else {
          __hip_atomic_fetch_add(a.ctl + (kChainCtlSeq + T.chain_seq) * kChainCtlStride, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (prof) prof[7] = waited;
      }
      // One queue: the following entry is claimed only now.  The claim is a round trip to memory: issued before the
      // entry's work it sits in front of the first operand loads in the in-order memory counter; issued before the
      // completion signal (even as early as the end of the K loop: measured) it delays every dependant.
      if (claiming && tid == 0) next = chain_claim(a, 0u, qb, qe);
    }
  }
  // a shared column is often done long before the pass is: go on prefetching (a favour: nothing to report if it cannot)
  const uint64_t t0 = wall_clock64();
  const uint32_t lane = (uint32_t)work_thread_id() & 63u;
  uint32_t polls = 0u, p0 = 0u;
  while (pf < pf_end && !gave_up) {
    if (prefetch_due(a, pf, lane, p0)) {
      prefetch_filters(*(ConstOp*)(a.ops + ((ConstPrefetch*)a.prefetch)[pf].op), rank, tid);
      ++pf;
      p0 = 0u;
      continue;
    }
    __builtin_amdgcn_s_sleep(8);
    if ((++polls & 15u) == 0u)
      gave_up = wall_clock64() - t0 > (uint64_t)a.spin_limit || polls > max_polls(a.spin_limit) ||
                abandoned(a);
  }
  if (tid == 0 && n_done != 0u) __hip_atomic_fetch_add(&a.ctl[kChainCtlDone * kChainCtlStride], n_done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <uint32_t HAS, bool COLUMNS>
const void* chain_kernel() { return (const void*)st_chain_kernel<HAS, COLUMNS>; }

}  // namespace st
