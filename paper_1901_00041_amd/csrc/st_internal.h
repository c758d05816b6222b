// Internal types shared by the host planner and the device kernels (not part of the C ABI).
#pragma once
#include <stddef.h>
#include <stdint.h>

#include "st_conv.h"

namespace st {

constexpr int kThreads = 256;      // workgroup size of every conv kernel: 4 wavefronts of 64
constexpr int kNumCUs = 256;       // MI355X
constexpr int kNumXCDs = 8;        // workgroup b of a launch runs on XCD b mod 8
constexpr int kProfSlots = 8;      // 64-bit stamps per work item in a profiled launch

// Tile family.  MT = output pixels (rows of the im2col matrix), NT = filters per workgroup tile.
// The 4 wavefronts form a WPX x WCH grid; MF is the MFMA block edge (32 -> 32x32 blocks,
// 16 -> 16x16 blocks); KB = bytes of the reduction index staged per row per K step; D = K steps of operands
// resident in LDS (as many as fit kSmemBytes; the loads of D - 1 of them are in flight).
struct TileShape {
  int MT, NT, WPX, WCH, MF, KB, D;
};
constexpr int kNumTileCfgs = 7;
constexpr int kRowCfg = 6;         // the row tile for few-channel layers (conv_tile_rows): 128-pixel segments of
                                   // kRowsPerTile consecutive output rows x 64 filters, one filter row per K step
constexpr int kChainPoolCfg = 7;   // chain kernel only: TenantDev.cfg of a max-pool op (not a convolution tile shape)
constexpr int kRowsPerTile = 4;    // most output rows one row-tile work item may take (the planner picks 1, 2 or 4)
constexpr TileShape kTileShapes[kNumTileCfgs] = {
    {128, 128, 2, 2, 32, 128, 2},  // 0: wave tile 64x64
    {128, 64, 2, 2, 32, 128, 3},   // 1: wave tile 64x32
    {64, 128, 2, 2, 32, 128, 3},   // 2: wave tile 32x64
    {64, 64, 2, 2, 32, 128, 4},    // 3: wave tile 32x32
    {32, 64, 2, 2, 16, 256, 3},    // 4: wave tile 16x32
    {16, 64, 1, 4, 16, 256, 3},    // 5: wave tile 16x16
    {128, 64, 2, 2, 32, 64, 2},    // 6: row tile (few input channels), wave tile 64x32
};
constexpr int kSmemBytes = 81920;  // LDS per workgroup: half a compute unit's 160 KiB
constexpr int kRowStageBytes = 18432;   // row tile: LDS set aside for the epilogue's transposition buffer
// tile shapes that exist for any channel count through conv_tile_gather; the planner maps tenants whose channels are not
// a multiple of the 16-byte vector onto one of them
constexpr bool kGenericCfg[kNumTileCfgs] = {false, true, false, true, false, false, false};
// ... and those that exist for whole vectors and channels left over (kOrderPieces)
constexpr bool kPiecesCfg[kNumTileCfgs] = {false, true, false, true, true, true, false};

// What a workgroup runs, in the `reserved` word of the device's copy of a work item: a tile form (vector and any-channel forms
// of a shape, its form with the input patch resident, the row tile, a chain's max-pool) and the operands' type.  A workgroup
// then needs nothing but its work item to find its code, and the tenant's record is fetched once, by the tile that runs.
constexpr uint32_t kFormVector = 0, kFormPatch = 8, kFormGather = 16, kFormRows = 24, kFormPool = 25, kFormPieces = 32;     // + the tile shape for all but rows and pool
constexpr uint32_t kFormTypeShift = 8, kFormMask = (1u << kFormTypeShift) - 1u;
// What a kernel was compiled for: bit `type` for every operand type, and the forms beyond vector and patch tiles.  All tile
// code in one kernel costs every launch: a tile is reached over several far jumps through instructions that no other
// workgroup has fetched, and registers are allotted for the largest.  A launch takes the smallest kernel that has its forms
// (one kernel with nested switches over the record -> these, us per pass: four 3x3 layers of batch 1 7.47 -> 7.13, eight
// 256->256 at 14x14 8.33 -> 8.20, 20 fp32 layers 20.0 -> 19.4, eight 53-layer networks of batch 1 as a chain 369 -> 357, four of
// batch 4 as 49 launches 543 -> 535).
constexpr uint32_t kHasRows = 8u, kHasGather = 16u, kHasPools = 32u, kHasEverything = 63u;

constexpr int kOrderTaps = 0, kOrderChannels = 1, kOrderLinear = 2;   // see conv_tile
constexpr int kOrderPatch = 3;     // see conv_tile_patch
constexpr int kOrderPieces = 4;    // any channel count of more than a vector: whole vectors first, then the channels left over (conv_tile)
// filter steps resident in LDS when a tile shape keeps its input patch there (0: the shape has no such form; two patches and
// two 16 KiB steps of a 128x128 tile would leave no room for a third).  Filters from beyond the L2 need the fourth step
// where a step is short: eight tenants of 3x3 on 64x64 tiles 11.1 us with three, 9.1 with four.
constexpr int kPatchStages[kNumTileCfgs] = {0, 4, 3, 4, 3, 0, 0};
constexpr int kPatchTaps = 9;
constexpr int kPatchMin = 4;       // load instructions per wavefront and channel block: at least (some twice, if fewer would do)

// Device-side tenant record, read through scalar loads by every workgroup of that tenant.
struct TenantDev {
  // read by every tile, most of it at once (tile_fields_loaded): three 64-byte lines
  const void* x;
  const void* w;
  void* y;
  const void* res;
  int32_t C, H, W, K, R, S, stride, pad;
  int32_t Q, PQ, M, Kg;
  int32_t in_dtype, out_dtype, epilogue;
  int32_t cfg, split_k, k_steps, k_steps_per_split;
  int32_t vec_ok;        // 1: C is a multiple of the 16-byte vector width, 2: kOrderPieces (both conv_tile), 0: any channel count or row tile
  int32_t step_dk, step_dr;   // one K step in the reduction index (r*S + s)*C + c: KT elements = step_dr filter rows of
                              //    S*C elements and step_dk elements more; kOrderPieces: a tap's channels in whole vectors, and
                              //    the steps that all taps' whole vectors take (k_steps counts those of the channels left over, too)
  int32_t k_order;            // kOrder*: how conv_tile walks the reduction index
  uint32_t tap_rows;          // kOrderChannels: bit r*S for every filter row r
  int32_t patch_rows;         // kOrderPatch: most input pixels a tile's taps touch
  int32_t patch_loads;        // load instructions per wavefront and channel block
  int32_t patch_blocks;       // channel blocks per K slice
  int32_t tiles_n;
  int32_t shift_pq, shift_q;  // floor(n/d) = ((n * magic) >> 31) >> shift, for d = P*Q and d = Q (pixel index -> image, row, column)
  uint32_t magic_pq, magic_q;
  uint32_t x_bytes, w_bytes;  // buffer sizes for bounds-checked loads
  uint32_t y_bytes;           // size of y (and of the residual) in bytes
  int32_t shift_c, shift_s;   // the same division for d = C (kOrderPieces: step_dk) and d = S
  uint32_t magic_c, magic_s;
  int32_t P;
  // read by some
  float* ws;             // split-K partial tiles (nullptr when split_k == 1)
  uint32_t* counters;    // one arrival counter per output tile (split-K only), zero between runs
  int32_t shift_r, shift_nvp; // same for d = R and d = row_pitch/16 (row tile only)
  uint32_t magic_r, magic_nvp;
  int32_t rows_per_tile;      // row tile only: output rows per work item
  int32_t row_pitch;          // row tile only: bytes of one image row in LDS (padding included, multiple of 16)
  int32_t tiles_m;
  // chain kernel only (st_chain.hip); the per-plan kernel ignores them
  int32_t chain_seq;          // sequence whose completion counter this op's work items wait on and bump
  uint32_t chain_need;        // work items of that sequence that must be complete before this op's may start
  // one completion flag per work item (queue per XCD): work item (tile_m, tile_n, slice) of this op owns flag
  // chain_flag_base + (tile_m * tiles_n + tile_n) * split_k + slice; an entry of the op may start once the flags
  // [chain_dep_begin, chain_dep_begin + chain_dep_count) and those of its own ChainDep all hold the run's number
  uint32_t chain_flag_base, chain_dep_begin, chain_dep_count;
};
static_assert(offsetof(TenantDev, ws) == 192 && sizeof(TenantDev) == 256, "lines of the scalar cache");
static_assert(sizeof(TenantDev) % 8 == 0, "TenantDev must keep pointer alignment in arrays");

// The work item's code word for an op, and what its kernel must have been compiled for.
inline uint32_t tile_code(const TenantDev& T) {
  const uint32_t form = T.cfg == kChainPoolCfg ? kFormPool
                        : T.vec_ok == 2        ? kFormPieces + (uint32_t)T.cfg
                        : T.vec_ok             ? (T.k_order == kOrderPatch ? kFormPatch : kFormVector) + (uint32_t)T.cfg
                        : T.cfg == kRowCfg     ? kFormRows
                                               : kFormGather + (T.cfg == 1 ? 1u : 3u);
  return form | ((uint32_t)T.in_dtype << kFormTypeShift);
}
inline uint32_t kernel_needs(const TenantDev& T) {
  const uint32_t form = tile_code(T) & kFormMask;
  return (1u << T.in_dtype) | (form == kFormPool ? kHasPools : form == kFormRows ? kHasRows : form >= kFormGather ? kHasGather : 0u);
}

// Launchers.  All asynchronous; return the hipError_t as int.  `needs`: kernel_needs of every tenant in the list.
int launch_conv(uint32_t needs, const TenantDev* tenants_dev, const st_work_item* items_dev, int64_t n_items, void* stream,
                uint64_t* prof_dev);
// ... of one kernel (st_conv_kernel.hpp)
template <uint32_t HAS>
int launch_conv_kernel(const TenantDev* tenants_dev, const st_work_item* items_dev, int64_t n_items, void* stream, uint64_t* prof_dev);
// Persistent chain launch (st_chain.hip).  ctl / ctl_other: this run's and the next run's control block.  A block is
// ctl_slots slots of kChainCtlStride 32-bit words (256 bytes) with one live word each, so that the words hundreds of
// workgroups poll and bump sit in different cache lines and memory channels: slot kChainCtlAbort the abort flag,
// kChainCtlLost whether any run on the block was abandoned, kChainCtlDone the completed work items of all runs on it and
// kChainCtlStarted the number of these runs (a run clears the other block for the next one, all but these three, which only
// st_chain_aborted clears), kChainCtlHead the head of the one queue, or with queues per XCD
// kChainCtlHead + 2x + k the number of exclusive (k = 0) / shared (k = 1) columns of XCD x drawn so far,
// kChainCtlSeq + s the completion counter of sequence s; kChainRankWords dense words follow the slots (how many
// workgroups have arrived on each compute unit).  n_queues is 1 (entries [0, n_items) claimed one by one) or
// kNumXCDs (colbegin_dev: kNumXCDs * 2 * kChainColumns + 1 column boundaries in device memory; XCD x's exclusive
// columns are x * 2 * kChainColumns + [0, kChainColumns), its shared ones follow).  item_flags / run_number: the
// per-item completion flags and this run's number (queues per XCD only; else nullptr / anything).
// A run that is captured into a graph has a block and a number of its own (kChainCapturedRun, which no other run gets);
// launch_chain_reset goes ahead of it and clears what the run before would have, and every flag.
constexpr int kChainCtlBlocks = 4;
constexpr uint32_t kChainCapturedRun = 0xffffffffu;
constexpr int kChainCtlStride = 64;
constexpr int kChainCtlLost = 0, kChainCtlAbort = 1, kChainCtlDone = 2, kChainCtlStarted = 3, kChainCtlHead = 4, kChainCtlSeq = 4 + 2 * kNumXCDs;
constexpr int kChainRankWords = kNumXCDs * 256;   // arrival counts per (XCD, compute unit key), dense, after the slots
constexpr int kChainColumns = kNumCUs / kNumXCDs; // exclusive columns per XCD (one per compute unit), and as many shared
constexpr uint32_t kChainFlagLocalFlags = 4u;     // completion travels through per-item flags in the XCD's own L2
// Filters to pull into an XCD's L2 ahead of their stage: op's w, once the flags [gate_begin, gate_begin + gate_count) are
// set (those of the stage two before; none for the first two stages); flag_base is the op's own.
// What an entry waits for besides the range in its op's record: the flags [begin, begin + count).  An op that reads exactly what
// one op of the previous stage writes has the stage before that in its record (everything earlier is then complete) and
// here, per entry, the previous stage's tiles that the entry reads; any other op has the whole previous stage in its record.
struct ChainDep { uint32_t begin, count; };
struct ChainPrefetch { uint32_t op, flag_base, gate_begin, gate_count; };
int chain_max_workgroups(int* out_workgroups, int* out_xcds);
int launch_chain(uint32_t needs, const TenantDev* ops_dev, const st_work_item* items_dev, uint32_t n_items, const uint32_t* colbegin_dev, const ChainDep* deps_dev, uint32_t n_queues, const ChainPrefetch* prefetch_dev,
                 const uint32_t* prefetch_begin, uint32_t* ctl, uint32_t* ctl_other, uint32_t ctl_slots, uint32_t* item_flags, uint32_t run_number,
                 uint32_t spin_limit_ticks, uint32_t flags, int grid, void* stream, uint64_t* prof_dev);
int launch_chain_reset(uint32_t* ctl, uint32_t ctl_slots, uint32_t* item_flags, uint32_t n_flags, void* stream);
int launch_empty(void* stream);
// Allocation-free path: device address of the current GPU's fixed scratch array (looked up on first use per device),
// host bytes -> device through kernel arguments (sizes rounded up to 16 bytes; dst 16-byte aligned), and a zero fill.
constexpr int64_t kNoallocScratchBytes = (int64_t)32 << 20;
int noalloc_scratch(void** out_ptr);
int launch_poke(const void* host_src, int64_t bytes, void* dst_dev, void* stream);
// the four tensor pointers of n records -> device table, through kernel arguments
int launch_bind(const TenantDev* host, int n, TenantDev* table_dev, void* stream);
int launch_zero(void* dst_dev, int64_t bytes, void* stream);
int launch_copy(const void* src, void* dst, int64_t bytes, void* stream);
int launch_maxpool(const void* x, void* y, int N, int H, int W, int C, int P, int Q, int win, int stride,
                   int pad, int dtype, void* stream);

}  // namespace st
