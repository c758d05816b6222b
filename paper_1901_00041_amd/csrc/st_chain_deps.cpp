// What the entries of a chain laid out per XCD wait for, and the order and columns they are dealt in (host only).
//
// An op's entries may start once everything of the sequence's earlier stages that they touch is complete.  Most layers of a
// network read exactly what the one before wrote, and a tile reads a few rows of it: such an entry waits for the tiles of the
// previous stage that write those rows (its LOCAL range) and for all of the stage before that one (the GATE), so two
// neighbouring stages overlap and a stage whose tiles do not fill the compute units evenly does not leave them idle.
// Why two: an entry of stage t runs beside entries of stage t-1 only, so only those two stages' tensors need be compared for
// overwrites, and everything older is complete.  That needs "a stage complete" to imply "the stage before it complete",
// which holds if some op of the stage waits for all of it or the local ranges of its entries together cover it
// (require_coverage in st_chain.cpp).
// Eight 53-layer networks, us per pass, whole stages -> tiles (and outputs left in the L2, see st_chain_kernel.hpp): batch 1
// 357 -> 347, batch 3 661 -> 590, batch 8 1147 -> 1129.  A stage of batch 8 has few enough tiles that what bounds it is the time
// from one stage's tile to the next one's, and the 56x56 stages are bound by memory.
#include <algorithm>
#include <vector>

#include "st_chain_deps.h"

namespace st {

namespace {

struct Bytes { uintptr_t begin, end; };
Bytes bytes_of(const void* p, uint64_t n) { return {(uintptr_t)p, (uintptr_t)p + (p ? n : 0)}; }
bool overlap(Bytes a, Bytes b) { return a.begin < b.end && b.begin < a.end; }

// (Pixels, vectors and tiles of an op are fewer than 2^31.)
// Output pixels [a, b) (linear over image, row, column) of one tile.
void output_pixels(const TenantDev& T, uint32_t tile_m, uint32_t* a, uint32_t* b) {
  if (T.cfg == kChainPoolCfg) {
    const uint32_t cv = T.C / (16 / elem_size(T.in_dtype)), end = std::min<uint32_t>(T.M, (tile_m + 1) * kThreads);
    *a = tile_m * kThreads / cv;
    *b = (end + cv - 1) / cv;
  } else if (T.cfg == kRowCfg) {
    const uint32_t qt = cdiv(T.Q, kTileShapes[kRowCfg].MT), pg = cdiv(T.P, T.rows_per_tile), g = tile_m / qt, n = g / pg, p = g % pg * T.rows_per_tile;
    *a = (n * T.P + p) * T.Q;
    *b = (n * T.P + std::min<uint32_t>(T.P, p + T.rows_per_tile)) * T.Q;
  } else {
    const uint32_t mt = kTileShapes[T.cfg].MT;
    *a = tile_m * mt;
    *b = std::min<uint32_t>(T.M, (tile_m + 1) * mt);
  }
}

// Input pixels [lo, hi) that hold everything output pixels [a, b) read: whole rows, unless the layer is a 1x1 of stride 1.
void input_pixels(const TenantDev& T, uint32_t a, uint32_t b, uint32_t* lo, uint32_t* hi) {
  if (T.R == 1 && T.S == 1 && T.stride == 1 && T.pad == 0) { *lo = a; *hi = b; return; }
  const uint32_t n0 = a / T.PQ, p0 = a % T.PQ / T.Q, n1 = (b - 1) / T.PQ, p1 = (b - 1) % T.PQ / T.Q;
  const uint32_t h0 = (uint32_t)std::min<int32_t>(T.H - 1, std::max<int32_t>(0, (int32_t)(p0 * T.stride) - T.pad));
  const uint32_t h1 = (uint32_t)std::min<int32_t>(T.H - 1, std::max<int32_t>(0, (int32_t)(p1 * T.stride) - T.pad + T.R - 1));
  *lo = (n0 * T.H + h0) * T.W;
  *hi = (n1 * T.H + h1 + 1) * T.W;
}

// Tiles (first, last) of an op that write its output pixels [lo, hi).
void tiles_writing(const TenantDev& P, uint32_t lo, uint32_t hi, uint32_t* first, uint32_t* last) {
  if (P.cfg == kChainPoolCfg) {
    const uint32_t cv = P.C / (16 / elem_size(P.in_dtype));
    *first = lo * cv / kThreads;
    *last = (hi * cv - 1) / kThreads;
  } else if (P.cfg == kRowCfg) {
    const uint32_t qt = cdiv(P.Q, kTileShapes[kRowCfg].MT), pg = cdiv(P.P, P.rows_per_tile);
    auto group = [&](uint32_t m) { return m / P.PQ * pg + m % P.PQ / P.Q / P.rows_per_tile; };
    *first = group(lo) * qt;
    *last = group(hi - 1) * qt + qt - 1;
  } else {
    *first = lo / kTileShapes[P.cfg].MT;
    *last = (hi - 1) / kTileShapes[P.cfg].MT;
  }
}

}  // namespace

// Whether an entry of T may run while entries of P (another stage, same sequence) do, but for P's output that T reads as x.
bool chain_ops_disjoint(const TenantDev& T, const TenantDev& P) {
  const Bytes ty = bytes_of(T.y, T.y_bytes), py = bytes_of(P.y, P.y_bytes);
  const bool t_res = (T.epilogue & ST_EPI_RESIDUAL) != 0u, p_res = (P.epilogue & ST_EPI_RESIDUAL) != 0u;
  if (overlap(ty, bytes_of(P.x, P.x_bytes)) || overlap(ty, bytes_of(P.w, P.w_bytes)) || overlap(ty, py)) return false;
  if (p_res && overlap(ty, bytes_of(P.res, P.y_bytes))) return false;
  if (overlap(py, bytes_of(T.w, T.w_bytes)) || (t_res && overlap(py, bytes_of(T.res, T.y_bytes)))) return false;
  // both sum partial tiles in the sequence's one workspace
  return T.split_k <= 1 || P.split_k <= 1;
}
bool chain_reads(const TenantDev& T, const TenantDev& P) { return overlap(bytes_of(T.x, T.x_bytes), bytes_of(P.y, P.y_bytes)); }
// Whether T's input is P's output, whole and with the same pixels and channels.
bool chain_reads_exactly(const TenantDev& T, const TenantDev& P) {
  if (T.x != P.y || T.x_bytes != P.y_bytes || T.in_dtype != P.out_dtype || T.C != P.K) return false;
  return T.H == P.P && T.W == P.Q;       // equal bytes: as many images
}

ChainDep chain_local_range(const TenantDev& T, const TenantDev& P, uint32_t tile_m) {
  uint32_t a, b, lo, hi, first, last;
  output_pixels(T, tile_m, &a, &b);
  input_pixels(T, a, b, &lo, &hi);
  tiles_writing(P, lo, hi, &first, &last);
  last = std::min<uint32_t>(last, P.tiles_m - 1);
  const uint32_t per = (uint32_t)P.tiles_n * P.split_k;
  return {P.chain_flag_base + first * per, (last - first + 1) * per};
}

ChainDealer::ChainDealer(bool shared_too) : shared_too_(shared_too) {
  for (auto& tree : first_)
    for (size_t n = kKind - 1; n >= 1; --n) tree[n] = n < kKind / 2 ? tree[2 * n] : (uint8_t)(2 * n - kKind);
}

void ChainDealer::place(size_t column, double ready, double cost) {
  free_[column] = finish(column, ready, cost);
  const size_t kind = column / kKind, base = kind * kKind;
  uint8_t* tree = first_[kind];
  for (size_t n = (column - base + kKind) / 2; n >= 1; n /= 2) {
    const size_t l = 2 * n < kKind ? tree[2 * n] : 2 * n - kKind, r = 2 * n < kKind ? tree[2 * n + 1] : 2 * n + 1 - kKind;
    tree[n] = (uint8_t)(free_[base + r] < free_[base + l] ? r : l);
  }
}

}  // namespace st
