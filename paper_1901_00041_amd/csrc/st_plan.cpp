// Host side of the library: descriptor validation, derived sizes, tile / split-K selection, work-list
// construction, device tables, the three issue policies and the C ABI (declared in st_conv.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <thread>
#include <vector>

#include "st_host.h"
#include "st_internal.h"

using namespace st;

// ---------------------------------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------------------------------
static thread_local char g_err[512] = "";

st_status st::fail(st_status s, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return s;
}
st_status st::hip_fail(hipError_t e, const char* what) {
  (void)hipGetLastError();      // reported here: the runtime must not report it again to whoever asks next on this thread
  return fail(e == hipErrorOutOfMemory ? ST_ERR_OUT_OF_MEMORY : ST_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

static st_status validate(const st_conv_desc& d, int t) {
  if (d.N <= 0 || d.C <= 0 || d.H <= 0 || d.W <= 0 || d.K <= 0 || d.R <= 0 || d.S <= 0)
    return fail(ST_ERR_INVALID_ARG, "tenant %d: every size must be positive", t);
  if (d.stride <= 0 || d.pad < 0) return fail(ST_ERR_INVALID_ARG, "tenant %d: stride must be > 0 and pad >= 0", t);
  if (d.reserved != 0) return fail(ST_ERR_INVALID_ARG, "tenant %d: reserved field must be 0", t);
  if (d.in_dtype != ST_DT_F32 && d.in_dtype != ST_DT_BF16 && d.in_dtype != ST_DT_F16)
    return fail(ST_ERR_UNSUPPORTED, "tenant %d: unknown in_dtype %d", t, d.in_dtype);
  if (d.out_dtype != ST_DT_F32 && d.out_dtype != d.in_dtype)
    return fail(ST_ERR_UNSUPPORTED, "tenant %d: out_dtype must be f32 or equal to in_dtype", t);
  if (d.layout == ST_LAYOUT_NCHW_KCRS)
    return fail(ST_ERR_UNSUPPORTED, "tenant %d: layout NCHW/KCRS is not implemented (tensors must be NHWC / KRSC)", t);
  if (d.layout != ST_LAYOUT_NHWC_KRSC) return fail(ST_ERR_UNSUPPORTED, "tenant %d: unknown layout %d", t, d.layout);
  if (d.epilogue & ~(uint32_t)(ST_EPI_RELU | ST_EPI_RESIDUAL))
    return fail(ST_ERR_UNSUPPORTED, "tenant %d: unknown epilogue bits 0x%x", t, d.epilogue);
  if ((int64_t)d.H + 2 * (int64_t)d.pad < d.R || (int64_t)d.W + 2 * (int64_t)d.pad < d.S)
    return fail(ST_ERR_INVALID_ARG, "tenant %d: filter larger than the padded image (empty output)", t);
  if (!d.x || !d.w || !d.y) return fail(ST_ERR_INVALID_ARG, "tenant %d: x, w and y must be non-NULL", t);
  if ((d.epilogue & ST_EPI_RESIDUAL) && !d.residual)
    return fail(ST_ERR_INVALID_ARG, "tenant %d: ST_EPI_RESIDUAL without a residual pointer", t);
  if ((const void*)d.y == d.x || (const void*)d.y == d.w)
    return fail(ST_ERR_INVALID_ARG, "tenant %d: y must not alias x or w", t);
  const int64_t lim = (int64_t)1 << 31;
  const int64_t P = ((int64_t)d.H + 2 * d.pad - d.R) / d.stride + 1, Q = ((int64_t)d.W + 2 * d.pad - d.S) / d.stride + 1;
  const int64_t nx = (int64_t)d.N * d.C * d.H * d.W, nw = (int64_t)d.K * d.C * d.R * d.S, ny = (int64_t)d.N * P * Q * d.K;
  const int64_t es = elem_size(d.in_dtype);
  if (nx * es >= lim || nw * es >= lim || ny * elem_size(d.out_dtype) >= lim || d.pad >= (1 << 20) || d.stride >= (1 << 20) ||
      d.C >= (1 << 20) || d.S >= (1 << 20))
    return fail(ST_ERR_UNSUPPORTED, "tenant %d: x, w and y must each stay below 2^31 bytes", t);
  return ST_OK;
}


// Multiplier and shift with floor(n/d) == ((n*m) >> 31) >> L for every 0 <= n < 2^31 and 1 <= d < 2^31
// (m = floor(2^(31+L)/d) + 1 fits 32 bits because d > 2^(L-1); m*d - 2^(31+L) <= d, so the error of n*m/2^(31+L)
// against n/d stays below n/2^31 < 1 and cannot carry past the next integer).
static void magic_for(int d, uint32_t* m, int32_t* L) {
  int l = 0;
  while (((int64_t)1 << l) < (int64_t)d) ++l;
  *L = l;
  *m = (uint32_t)((((uint64_t)1) << (31 + l)) / (uint64_t)d + 1);
}

// ---------------------------------------------------------------------------------------------------
// tile shape and split-K selection
// ---------------------------------------------------------------------------------------------------
// Cost of one work item in shader clocks, from in-kernel time stamps on an MI355X (st_conv_run_profiled):
//   first operands staged | one K step | epilogue | split-K hand-off (write-through, counter, read back).
// A workgroup that has its compute unit to itself and two that share one behave differently (the shared step is bound by
// the compute unit's 64 bytes per clock from the L2, the lone one by latency and instruction issue), and fp32 MFMAs take
// eight times as long as 16-bit ones, so there are four tables; two more for 16-bit 3x3 layers whose input patch stays
// in LDS (a shape without that form costs there what it costs in the first table); and two for 16-bit layers whose channels are no
// multiple of the step (kOrderTaps), whose rows straddle cache lines and whose lanes keep a position each: a shared step
// of 64x64 takes 850 clocks (16 to 240 channels, 3x3 and 5x5) where one of 64 or 128 channels takes 430.  fp32 layers of that order are bound by their MFMAs and
// cost what the others do.
// The launch is modelled as list scheduling of the items on workgroup slots: its duration is about max(longest item, sum
// of item times / slots).  The planner picks, per tenant, the (tile, split) option that minimises that maximum over
// the whole launch: once for kSlots slots of shared compute units and, if the caller names no number of slots, once for
// one workgroup on each.  (So a plan with target_items, which every stack and chain has, is priced by the shared tables
// throughout; and the order of the fused list goes by the shared tables without the patch form, whatever was planned.)
// The epilogues' prices are of the time when they took half as many vector instructions again, and are too high by now: 128x128 alone
// 3900, now 1840 to 3320 (ReLU, residual); 64x64 alone 1500, now 1190 to 1670.
struct ItemCosts { double first[kNumTileCfgs], step[kNumTileCfgs], epi[kNumTileCfgs]; };
enum { kCosts16 = 0, kCosts32 = 1, kCostsPatch = 2, kCostsTaps = 3 };
// [kCosts*][alone on the compute unit]
static const ItemCosts kCosts[4][2] = {
    {{{4800, 4500, 4500, 3800, 4200, 3250, 3000}, {1250, 740, 740, 430, 650, 560, 310}, {4700, 2500, 2600, 1800, 1400, 1230, 2300}},
     {{2700, 2500, 2500, 2300, 2600, 2200, 3000}, {820, 470, 470, 305, 450, 375, 310}, {3900, 2070, 2080, 1500, 1240, 1120, 2300}}},
    {{{5200, 5500, 5500, 4300, 4300, 3250, 0}, {7200, 3600, 3600, 1850, 1850, 1060, 0}, {8000, 4500, 4000, 3000, 1800, 1330, 0}},
     {{3500, 3000, 3000, 2500, 2700, 2300, 0}, {4350, 2260, 2240, 1200, 1300, 740, 0}, {4300, 2200, 2200, 1670, 1430, 1180, 0}}},
    {{{4800, 2300, 2400, 2000, 2300, 3250, 0}, {1250, 620, 680, 380, 590, 560, 0}, {4700, 2400, 2500, 1700, 1400, 1230, 0}},
     {{2700, 1500, 1550, 1300, 1600, 2200, 0}, {820, 465, 445, 310, 410, 375, 0}, {3900, 2060, 2030, 1500, 1240, 1120, 0}}},
    {{{1200, 2250, 2300, 2650, 2400, 1850, 0}, {2210, 1300, 1370, 850, 1060, 840, 0}, {4700, 2500, 2600, 1800, 1400, 1230, 0}},
     {{2050, 3350, 3000, 3550, 2950, 2300, 0}, {1490, 745, 785, 475, 605, 475, 0}, {3900, 2070, 2080, 1500, 1240, 1120, 0}}}};
static double row_stage_cost(int rows_per_tile) { return 4300.0 + 300.0 * rows_per_tile; }      // row tile: copying image rows and filters into LDS
// any channel count (conv_tile_gather) [fp32 operands]: bound by the texture addresser, which takes unaligned vectors apart
static const double kGatherStepCost[2][kNumTileCfgs] = {{0, 2600.0, 0, 1550.0, 0, 0, 0}, {0, 3600.0, 0, 2000.0, 0, 0, 0}};
static const double kGatherPartCost[kNumTileCfgs] = {0, 4000.0, 0, 1900.0, 0, 0, 0};   // more if the step crosses a filter row
static const double kGatherFirstCost = 7000.0;
static const double kSplitCost = 3600.0, kSplitPerElem = 0.6;               // hand-off, grows with the tile
static const double kSplitRoundCost = 2000.0, kSplitRoundPerElem = 0.25;    // per further batch of slices read back
static const int kSlots = 400;                  // two workgroups resident per compute unit (512), derated: the launch's
                                                // tail and the dispatch ramp leave some of them empty
static const int kSplitChoices[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};

// One K step of conv_tile_gather; the share of steps that cross a filter row grows as filter rows get shorter.
static double gather_step_cost(const st_conv_desc& d, int cfg) {
  const double kt = 128.0 / elem_size(d.in_dtype), crossing = d.R == 1 ? 0.0 : std::min(1.0, kt / ((double)d.S * d.C));
  return kGatherStepCost[d.in_dtype == ST_DT_F32 ? 1 : 0][cfg] + crossing * kGatherPartCost[cfg];
}

enum Form { kGathered = 0, kVectors = 1, kPieces = 2 };       // (TenantDev.vec_ok)

// Pieces: until the first operands are staged | a step of whole vectors | a step of channels left over | more for every tap in it;
// [16-bit types and an even channel count, 16-bit types and an odd one (vectors at odd multiples of two bytes), fp32][alone on the
// compute unit][tile shape].  Least relative squares over the stamps of 1x1, 3x3 and 5x5 layers of 5 to 243 channels, 24 layers or so
// to a table: the items are within 15 % of it, 2 to 7 % in the root mean square.  120 random launches of 3 to 40 layers off every round
// number, with all three epilogues: 0.97 (one launch of 17.7 us; the next 1.00) to 2.7 times as fast as with gathered tiles for all of
// them, 1.37 in the geometric mean; where pieces went by the vector tiles' prices, and epilogues by one price each, 0.76 to 1.7, 1.22.
struct PieceCosts { double first[kNumTileCfgs], step[kNumTileCfgs], left[kNumTileCfgs], tap[kNumTileCfgs]; };
static const PieceCosts kPieceCosts[3][2] = {
    {{{0, 3000, 0, 2400, 1850, 1700, 0}, {0, 1490, 0, 970, 1220, 1030, 0}, {0, 690, 0, 560, 1340, 1180, 0}, {0, 34, 0, 27, 0, 0, 0}},
     {{0, 3000, 0, 2350, 2450, 2000, 0}, {0, 850, 0, 510, 690, 590, 0}, {0, 1010, 0, 950, 990, 920, 0}, {0, 36, 0, 27, 26, 18, 0}}},
    {{{0, 1750, 0, 1500, 1400, 1400, 0}, {0, 1790, 0, 1200, 1720, 1470, 0}, {0, 1580, 0, 1100, 1340, 1200, 0}, {0, 400, 0, 250, 180, 140, 0}},
     {{0, 2050, 0, 1600, 2250, 1700, 0}, {0, 1100, 0, 720, 1120, 950, 0}, {0, 1800, 0, 1410, 810, 920, 0}, {0, 150, 0, 100, 115, 80, 0}}},
    {{{0, 3900, 0, 2200, 1600, 1950, 0}, {0, 4000, 0, 2200, 2380, 1440, 0}, {0, 3440, 0, 1930, 3180, 1820, 0}, {0, 185, 0, 130, 17, 21, 0}},
     {{0, 2900, 0, 2050, 2200, 1900, 0}, {0, 2600, 0, 1410, 1540, 975, 0}, {0, 2550, 0, 1800, 2030, 1370, 0}, {0, 82, 0, 25, 20, 12, 0}}}};
static const PieceCosts& piece_costs(const st_conv_desc& d, bool alone) {
  return kPieceCosts[d.in_dtype == ST_DT_F32 ? 2 : d.C % 2][alone ? 1 : 0];
}

// Epilogues whose rows are no whole vectors, by elements, of a tile full of filters, [with a residual][filter count off four][fp32
// output][alone on the compute unit][tile shape]: stamps of 3x3 layers of 64 and 67 channels with 241 to 252 filters, every type.
static const double kElementEpi[2][2][2][2][kNumTileCfgs] = {
    {{{{11000, 3500, 3500, 1900, 1400, 850, 0}, {7000, 2800, 2800, 1900, 1350, 850, 0}}, {{12000, 4300, 4400, 2200, 1250, 750, 0}, {6500, 2800, 2900, 1700, 1200, 750, 0}}},
     {{{41000, 12400, 12200, 6450, 2170, 1080, 0}, {21000, 9800, 9500, 4400, 1650, 1000, 0}}, {{45000, 15500, 16000, 8000, 2700, 1150, 0}, {23000, 10700, 10700, 4800, 1600, 925, 0}}}},
    {{{{36000, 14300, 17500, 6750, 3030, 1710, 0}, {20500, 10300, 10500, 5400, 2830, 1650, 0}}, {{46500, 18600, 22200, 8700, 3500, 2100, 0}, {24000, 10500, 11500, 5500, 2800, 1620, 0}}},
     {{{60000, 26500, 30000, 12400, 4150, 2000, 0}, {32000, 16500, 16800, 8600, 3660, 1860, 0}}, {{79000, 32500, 39000, 15200, 5400, 2450, 0}, {43000, 18200, 20000, 9500, 4000, 1880, 0}}}}};
// A residual of whole vectors that no K step hides (every form for any channel count), more than the same epilogue without.
static const double kOpenResidualEpi[kNumTileCfgs] = {0, 700, 0, 350, 400, 400, 0};

// The K steps of a layer on a tile shape: those of the reduction index, or in pieces those of all taps' whole vectors (`vectors`
// channels of each tap), then those of the channels left over, a vector per tap.
struct KSteps { int main, left, vectors; };
static KSteps k_steps_of(const st_conv_desc& d, int form, int cfg) {
  const int es = elem_size(d.in_dtype), vec = 16 / es, c = form == kPieces ? d.C / vec * vec : d.C;
  const int64_t taps = (int64_t)d.R * d.S;
  return {cdiv(taps * c * es, kTileShapes[cfg].KB), form == kPieces ? cdiv(taps * 16, kTileShapes[cfg].KB) : 0, c};
}

static const ItemCosts& item_costs(const st_conv_desc& d, int cfg, bool patch, bool alone) {
  const bool taps = cfg != kRowCfg && d.C % (kTileShapes[cfg].KB / 2) != 0;
  return kCosts[d.in_dtype == ST_DT_F32 ? kCosts32 : patch ? kCostsPatch : taps ? kCostsTaps : kCosts16][alone ? 1 : 0];
}

// Clocks that steps [begin, end) of a layer take.
static double steps_cost(const st_conv_desc& d, int form, int cfg, const ItemCosts& c, bool alone, const KSteps& k, int begin, int end) {
  if (form == kGathered) return (end - begin) * gather_step_cost(d, cfg);
  if (form == kVectors) return (end - begin) * c.step[cfg];
  const PieceCosts& p = piece_costs(d, alone);
  const int main = std::min(end, k.main) - std::min(begin, k.main);
  return main * p.step[cfg] + (end - begin - main) * (p.left[cfg] + p.tap[cfg] * d.R * d.S / k.left);
}

// Clocks from the last MFMA to the end of the item.  any_filters: the launch's kernel stores whole vectors for any filter count
// (kHasEverything; see tile_epilogue).
static double epilogue_cost(const st_conv_desc& d, int form, int cfg, const ItemCosts& c, bool alone, bool any_filters) {
  const bool residual = (d.epilogue & ST_EPI_RESIDUAL) != 0u;
  if (d.K % 8 == 0) return c.epi[cfg] + (residual && form != kVectors ? kOpenResidualEpi[cfg] : 0.0);
  if (!residual && any_filters) return c.epi[cfg];
  const double full = std::min(1.0, (double)d.K / kTileShapes[cfg].NT);
  return std::max(c.epi[cfg], full * kElementEpi[residual][d.K % 4 != 0][d.out_dtype == ST_DT_F32][alone ? 1 : 0][cfg]);
}

struct Option {
  int form;
  int cfg, split, steps_per_split, rows_per_tile;
  int64_t items;
  double item_time, area;
};

// Bytes of one image row in the row tile's LDS array: left padding, the row, right padding, rounded up to
// whole 16-byte vectors, plus the 64 bytes the operand read of the last pixel may run past its patch.
static int row_tile_pitch(const st_conv_desc& d) {
  const int64_t lpad = (int64_t)d.pad * d.C * 2;
  const int64_t pitch = ((lpad + (int64_t)d.W * d.C * 2 + lpad + 15) & ~(int64_t)15) + 64;
  return (int)std::min<int64_t>(pitch, 1 << 24);
}

// Whether a layer's operands can be fetched as 16-byte vectors: the channel count is a multiple of the vector, and an
// element position inside a padded image row (conv_tile counts in those) fits 31 bits.
static bool vector_ok(const st_conv_desc& d) {
  return d.C % (16 / elem_size(d.in_dtype)) == 0 && ((int64_t)d.W + 2 * (int64_t)d.pad) * d.C < ((int64_t)1 << 31);
}
// Whether operands can be fetched as the whole vectors of every tap and, by elements, the channels left over.
static bool pieces_ok(const st_conv_desc& d) {
  const int vec = 16 / elem_size(d.in_dtype);
  return d.C % vec != 0 && d.C > vec && ((int64_t)d.W + 2 * (int64_t)d.pad) * d.C < ((int64_t)1 << 31);
}

// Which form a layer takes on a tile shape (-1: it has none there).  Nothing but the layer and the shape decides: a layer's fp32 sums
// then run in one order whatever company it is planned in.  Where a shape has both forms for any channel count, the one of whole
// vectors and channels left over is the faster one at every channel count for 16-bit types (64x64 and 128x64 tiles, 1x1 to 5x5,
// 9 to 243 channels, alone and beside a second workgroup: 1.3 to 4.1 times) and for fp32 but where its vector of left-over
// channels per tap makes the reduction more than half as long again.  fp32, 64x64 beside a second workgroup, clocks of an item gathered
// and in pieces: five channels 3x3 13500 14750, 5x5 22300 25400; seven 3x3 14000 14800, 5x5 28400 25500; nine 17100 17400, 37300
// 31500; 13 to 122 channels 1.05 to 1.3 times as fast in pieces, alone on the unit up to 1.5.
static int form_on(const st_conv_desc& d, int cfg) {
  if (cfg == kRowCfg) return -1;
  if (vector_ok(d)) return kVectors;
  if (pieces_ok(d) && kPiecesCfg[cfg]) {
    const int vec = 16 / elem_size(d.in_dtype), padded = d.C / vec * vec + vec;
    if (!kGenericCfg[cfg] || d.in_dtype != ST_DT_F32 || 2 * padded <= 3 * d.C) return kPieces;
  }
  return kGenericCfg[cfg] ? kGathered : -1;
}

// Whether a tile shape can keep the layer's input patch in LDS (see conv_tile_patch), and the patch's size: 16-bit types,
// 3x3, stride 1, no more output columns and rows than input ones (then the input pixels under a tile's pixels ascend),
// channels a multiple of the step, and LDS room for the patch (twice when there is more than one channel block) beside
// the filter stages.
static bool patch_geometry(const st_conv_desc& d, int cfg, int32_t* rows, int32_t* loads) {
  if (d.in_dtype == ST_DT_F32 || kPatchStages[cfg] == 0 || d.stride != 1 || d.R != 3 || d.S != 3 || d.pad > 1) return false;
  const int64_t kb = kTileShapes[cfg].KB, mt = kTileShapes[cfg].MT, blocks = (int64_t)d.C * 2 / kb;
  const int64_t P = (int64_t)d.H + 2 * d.pad - 2, Q = (int64_t)d.W + 2 * d.pad - 2;
  if ((int64_t)d.C * 2 % kb != 0) return false;
  // from a tile's first pixel to its last: one input pixel per pixel, W - Q more per row begun, (H - P) * W more per image
  const int64_t span = (mt - 1) + (mt - 1 + Q - 1) / Q * (d.W - Q) + (mt - 1 + P * Q - 1) / (P * Q) * (d.H - P) * d.W;
  const int64_t n = span + 2 * (int64_t)d.W + 3;
  const int64_t per_turn = 4 * 64 / (kb / 16);                       // rows the four wavefronts load with one instruction each
  const int64_t turns = (n + 1 + per_turn - 1) / per_turn;           // the row after the last is the zero row
  const int64_t lds = turns * per_turn * kb * (blocks > 1 ? 2 : 1) + (int64_t)kPatchStages[cfg] * kTileShapes[cfg].NT * kb;
  if (lds > kSmemBytes) return false;
  *rows = (int32_t)n;
  *loads = (int32_t)turns;
  return true;
}

// Row tile eligibility (see conv_tile_rows): 16-bit types, 8 <= S*C <= 32, image rows a multiple of 16 bytes,
// stride*C even, LDS footprint within the allocation.
static bool row_tile_ok(const st_conv_desc& d) {
  if (d.in_dtype == ST_DT_F32) return false;
  if (d.C % 8 == 0) return false;                       // the vector kernels are better
  if (d.S * d.C > 32 || d.S * d.C < 8) return false;    // a filter row is one K step of 32, loaded as 16-byte vectors
  if ((d.W * d.C * 2) % 16 != 0) return false;
  if ((d.stride * d.C * 2) % 4 != 0) return false;       // pixel patches must stay 4-byte aligned in LDS
  const int pitch = row_tile_pitch(d);
  if (d.R + d.stride * (kRowsPerTile - 1) > kThreads / 2) return false;   // one thread per row end
  const int Q = (d.W + 2 * d.pad - d.S) / d.stride + 1;
  const int reach = (Q - 1) * d.stride * d.C * 2 + 64;             // furthest byte a pixel operand read touches
  if (reach > pitch) return false;
  const int64_t stage = kRowStageBytes;                                                       // epilogue buffer
  const int64_t rows = d.R + d.stride * (kRowsPerTile - 1);
  return stage + rows * pitch + (int64_t)kTileShapes[kRowCfg].NT * d.R * 64 <= kSmemBytes;
}

// XCD-aware placement.  The hardware hands workgroup b of a launch to XCD b mod 8, and each XCD has an L2 of
// its own, so what one XCD's work items read is fetched into that L2 once, and every operand slice is fetched once
// per XCD that has an item reading it.  A tenant's tiles are cut into xcd_blocks_m x xcd_blocks_n blocks (contiguous
// ranges of pixel tiles x contiguous ranges of filter tiles, at most 8 blocks); block g = bm * xcd_blocks_n + bn
// prefers XCD g, all K slices of a tile with it.  The XCDs together then fetch the activations xcd_blocks_n times and
// the filters xcd_blocks_m times.  The items of a run are dealt out position by position: position q (XCD
// (phase + q) mod 8) takes the next item that prefers this XCD, or, when none is left, the next item of the XCD with
// the most items left (lowest XCD on ties).
static int xcd_block_of(const st_work_item& it, const st_tenant_info& ti) {
  const int64_t bm = (int64_t)it.tile_m * ti.xcd_blocks_m / ti.tiles_m;
  const int64_t bn = (int64_t)it.tile_n * ti.xcd_blocks_n / ti.tiles_n;
  return (int)(bm * ti.xcd_blocks_n + bn);
}

// Fills n positions from the XCDs' own lists: position q (XCD (phase + q) mod 8) takes the next item of its XCD, or, when
// none is left, of the XCD with the most items left (lowest XCD on ties).
static void deal(const std::vector<st_work_item> (&bucket)[kNumXCDs], st_work_item* out, int64_t n, int phase) {
  size_t head[kNumXCDs] = {};
  for (int64_t q = 0; q < n; ++q) {
    int x = (int)((phase + q) % kNumXCDs);
    if (head[x] == bucket[x].size()) {
      size_t best = 0;
      for (int c = 0; c < kNumXCDs; ++c)
        if (bucket[c].size() - head[c] > best) { best = bucket[c].size() - head[c]; x = c; }
    }
    out[q] = bucket[x][head[x]++];
  }
}

static void xcd_arrange(st_work_item* items, int64_t n, int phase, const st_tenant_info& ti) {
  if (ti.xcd_blocks_m * ti.xcd_blocks_n <= 1 || n < 2) return;
  std::vector<st_work_item> bucket[kNumXCDs];
  for (int64_t i = 0; i < n; ++i) bucket[xcd_block_of(items[i], ti) % kNumXCDs].push_back(items[i]);
  deal(bucket, items, n, phase);
}

// The block grid of a tenant: among the grids a x b with a, b in {1, 2, 4, 8}, a * b <= blocks, a <= tiles_m, b <= tiles_n,
// the one with the most blocks, then the fewest bytes fetched over all XCDs (b times the activations plus a times the
// filters), then the smallest a.
static void xcd_block_choice(const st_conv_desc& d, const st_tenant_info& ti, int blocks, int* out_a, int* out_b) {
  const int64_t es = elem_size(d.in_dtype);
  const int64_t w_bytes = ti.Ngemm * ti.Kgemm * es, x_bytes = (int64_t)d.N * d.C * d.H * d.W * es;
  int best_a = 1, best_b = 1;
  int64_t best_cost = x_bytes + w_bytes;
  for (int a = 1; a <= blocks; a *= 2)
    for (int b = 1; a * b <= blocks; b *= 2) {
      if (a > ti.tiles_m || b > ti.tiles_n) continue;
      const int64_t cost = b * x_bytes + a * w_bytes;
      if (a * b > best_a * best_b || (a * b == best_a * best_b && cost < best_cost)) {
        best_a = a; best_b = b; best_cost = cost;
      }
    }
  *out_a = best_a;
  *out_b = best_b;
}

// Placement of a stretch of the fused list that holds several tenants' items of about the same cost.  Cutting every
// tenant into 8 blocks would have every XCD fetch some of every tenant (for 120 tenants of 8 tiles each, 157 MB
// instead of 43 MB, and the fills of the L2s, at about 7 TB/s, then bound the launch); here a tenant is cut into as
// few blocks as fit an XCD's share of the stretch, and the blocks are dealt to the XCDs, largest first, each to the XCD
// with the fewest items.  Positions then take their own XCD's items in order; where the shares are uneven, the XCD with
// the most items left gives one away, as in xcd_arrange.  [begin, end) are the stretch's runs of one tenant's items each.
struct ItemRun { int tenant; int64_t begin, end; };

static void xcd_arrange_tenants(st_work_item* items, const std::vector<ItemRun>& runs, const std::vector<st_conv_desc>& descs,
                                const std::vector<st_tenant_info>& info) {
  const int64_t first = runs.front().begin, total = runs.back().end - first;
  const int64_t share = (total + kNumXCDs - 1) / kNumXCDs;
  struct Block { size_t run; int index; int64_t count; };
  std::vector<Block> blocks;
  std::vector<int> grid_a(runs.size()), grid_b(runs.size()), block_base(runs.size());
  auto block_of = [&](size_t r, const st_work_item& it) {
    const st_tenant_info& ti = info[runs[r].tenant];
    return (int)((int64_t)it.tile_m * grid_a[r] / ti.tiles_m) * grid_b[r] + (int)((int64_t)it.tile_n * grid_b[r] / ti.tiles_n);
  };
  for (size_t r = 0; r < runs.size(); ++r) {
    int nb = 1;
    while (nb < kNumXCDs && (runs[r].end - runs[r].begin) > share * nb) nb *= 2;
    xcd_block_choice(descs[runs[r].tenant], info[runs[r].tenant], nb, &grid_a[r], &grid_b[r]);
    block_base[r] = (int)blocks.size();
    for (int g = 0; g < grid_a[r] * grid_b[r]; ++g) blocks.push_back({r, g, 0});
    for (int64_t i = runs[r].begin; i < runs[r].end; ++i) ++blocks[block_base[r] + block_of(r, items[i])].count;
  }
  std::vector<size_t> order(blocks.size());
  for (size_t i = 0; i < order.size(); ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) { return blocks[a].count > blocks[b].count; });
  int64_t load[kNumXCDs] = {};
  std::vector<int> xcd(blocks.size());
  for (size_t i : order) {
    const int x = (int)(std::min_element(load, load + kNumXCDs) - load);
    xcd[i] = x;
    load[x] += blocks[i].count;
  }
  std::vector<st_work_item> bucket[kNumXCDs];
  for (size_t r = 0; r < runs.size(); ++r)
    for (int64_t i = runs[r].begin; i < runs[r].end; ++i) bucket[xcd[block_base[r] + block_of(r, items[i])]].push_back(items[i]);
  deal(bucket, items + first, total, (int)(first % kNumXCDs));
}

static Option make_row_option(const st_conv_desc& d, int rows_per_tile, bool alone) {
  Option o;
  o.form = kGathered;
  o.rows_per_tile = rows_per_tile;
  const int P = (d.H + 2 * d.pad - d.R) / d.stride + 1, Q = (d.W + 2 * d.pad - d.S) / d.stride + 1;
  o.cfg = kRowCfg;
  o.split = 1;
  o.steps_per_split = d.R;
  o.items = (int64_t)d.N * cdiv(P, rows_per_tile) * cdiv(Q, kTileShapes[kRowCfg].MT) * cdiv(d.K, kTileShapes[kRowCfg].NT);
  const ItemCosts& c = kCosts[0][alone ? 1 : 0];
  o.item_time = c.first[kRowCfg] + row_stage_cost(rows_per_tile) + rows_per_tile * (d.R * c.step[kRowCfg] + c.epi[kRowCfg]);
  o.area = o.item_time * (double)o.items;
  return o;
}

static Option make_option(const st_conv_desc& d, int64_t M, int64_t Ng, int form, bool alone, bool any_filters, int cfg, int split) {
  Option o;
  o.form = form;
  o.rows_per_tile = 0;
  const KSteps k = k_steps_of(d, form, cfg);
  const int k_steps = k.main + k.left;
  split = std::max(1, std::min(split, std::min(k_steps, 65535)));
  const int per = cdiv(k_steps, split);
  split = cdiv(k_steps, per);          // no empty slice
  o.cfg = cfg;
  o.split = split;
  o.steps_per_split = per;
  o.items = (int64_t)cdiv(M, kTileShapes[cfg].MT) * cdiv(Ng, kTileShapes[cfg].NT) * split;
  int32_t rows, loads;
  const bool patch = per % kPatchTaps == 0 && patch_geometry(d, cfg, &rows, &loads);
  const ItemCosts& c = item_costs(d, cfg, patch, alone);
  const double elems = (double)kTileShapes[cfg].MT * kTileShapes[cfg].NT;
  const int batch = elems > 4096 ? 4 : 8;      // slices read back at a time
  // the longest slice: the first one, or where channels left over are dearer the last whole one or the last one
  double steps_time = 0.0;
  for (int i : {0, split - 2, split - 1})
    if (i >= 0) steps_time = std::max(steps_time, steps_cost(d, form, cfg, c, alone, k, i * per, std::min(k_steps, (i + 1) * per)));
  const double around = (form == kGathered ? kGatherFirstCost : form == kPieces ? piece_costs(d, alone).first[cfg] : c.first[cfg]) +
                        epilogue_cost(d, form, cfg, c, alone, any_filters) +
                        (split > 1 ? kSplitCost + kSplitPerElem * elems + (kSplitRoundCost + kSplitRoundPerElem * elems) * ((split - 1) / batch) : 0.0);
  o.item_time = around + steps_time;
  o.area = o.item_time * (double)o.items;
  if (form == kPieces) o.area = (double)o.items * (around + steps_cost(d, form, cfg, c, alone, k, 0, k_steps) / split);    // slices may differ a lot
  return o;
}

static std::vector<Option> tenant_options(const st_conv_desc& d, int64_t M, int64_t Ng, bool alone, bool any_filters,
                                          const st_plan_opts& o) {
  std::vector<Option> out;
  const bool row_ok = row_tile_ok(d);
  if (row_ok && (o.tile_cfg == 0 || o.tile_cfg - 1 == kRowCfg) && o.split_k <= 1) {
    for (int rt = 1; rt <= kRowsPerTile; rt *= 2)
      if (o.rows_per_tile == 0 || o.rows_per_tile == rt) out.push_back(make_row_option(d, rt, alone));
    if (o.tile_cfg - 1 == kRowCfg) return out;
  }
  int forced = o.tile_cfg - 1;
  if (o.tile_cfg > 0) {
    if (forced == kRowCfg) forced = 1;                                              // row tile requested but not eligible
    if (form_on(d, forced) < 0) forced = (kTileShapes[forced].MT >= 128) ? 1 : 3;   // the nearest shape this layer has
  }
  for (int c = 0; c < kNumTileCfgs; ++c) {
    const int form = form_on(d, c);
    if (form < 0 || (o.tile_cfg > 0 && c != forced)) continue;
    if (o.split_k >= 1) {
      out.push_back(make_option(d, M, Ng, form, alone, any_filters, c, o.split_k));
      continue;
    }
    int last_split = 0;
    for (int sp : kSplitChoices) {
      Option op = make_option(d, M, Ng, form, alone, any_filters, c, sp);
      if (op.split == last_split) continue;             // clamped to the same factor as before
      if (op.split > 1 && op.steps_per_split < 2) continue;
      last_split = op.split;
      out.push_back(op);
    }
  }
  return out;
}

// For a bound `limit` on the item time, each tenant takes its cheapest (smallest area) option that meets
// the bound, or its fastest option if none does; returns the modelled launch duration.
static void evaluate_parts(const std::vector<std::vector<Option>>& opts, double limit, std::vector<int>* pick,
                           double* out_longest, double* out_area) {
  double area = 0.0, longest = 0.0;
  pick->assign(opts.size(), 0);
  for (size_t t = 0; t < opts.size(); ++t) {
    int best = -1, fastest = 0;
    for (size_t i = 0; i < opts[t].size(); ++i) {
      const Option& op = opts[t][i];
      if (op.item_time < opts[t][fastest].item_time) fastest = (int)i;
      if (op.item_time <= limit && (best < 0 || op.area < opts[t][best].area)) best = (int)i;
    }
    if (best < 0) best = fastest;
    (*pick)[t] = best;
    area += opts[t][best].area;
    longest = std::max(longest, opts[t][best].item_time);
  }
  *out_longest = longest;
  *out_area = area;
}

static double evaluate(const std::vector<std::vector<Option>>& opts, double limit, int slots, std::vector<int>* pick) {
  double longest = 0.0, area = 0.0;
  evaluate_parts(opts, limit, pick, &longest, &area);
  return std::max(longest, area / slots);
}

// Minimise the modelled duration over the candidate bounds (the item times of all options).  As the bound grows
// every tenant's chosen item time can only grow and its area only shrink, so the duration is the maximum of a
// non-decreasing and a non-increasing function of the bound: bisect for the crossing and compare its two sides.
// ST_PLAN_EXHAUSTIVE=1 in the environment evaluates every candidate instead (the tests compare the two).
static void choose_all(const std::vector<std::vector<Option>>& opts, int slots, std::vector<int>* pick) {
  std::vector<double> limits;
  for (const auto& v : opts)
    for (const Option& op : v) limits.push_back(op.item_time);
  std::sort(limits.begin(), limits.end());
  limits.erase(std::unique(limits.begin(), limits.end()), limits.end());
  if (limits.empty()) { pick->assign(opts.size(), 0); return; }
  std::vector<int> cur;
  const char* ex = std::getenv("ST_PLAN_EXHAUSTIVE");
  if (ex && ex[0] == '1') {
    double best = -1.0;
    for (double lim : limits) {
      const double d = evaluate(opts, lim, slots, &cur);
      if (best < 0 || d < best) { best = d; *pick = cur; }
    }
    return;
  }
  // first candidate whose longest item is at least its area share
  auto longest_wins = [&](size_t i) {
    double longest = 0.0, area = 0.0;
    evaluate_parts(opts, limits[i], &cur, &longest, &area);
    return longest >= area / slots;
  };
  size_t lo = 0, hi = limits.size();     // invariant: candidates below lo are area-bound, hi and above longest-bound
  while (lo < hi) {
    const size_t mid = (lo + hi) / 2;
    if (longest_wins(mid)) hi = mid; else lo = mid + 1;
  }
  size_t best_i = lo < limits.size() ? lo : limits.size() - 1;
  double best = evaluate(opts, limits[best_i], slots, pick);
  // the area-bound side, and any equal durations further left (the smallest bound wins ties)
  for (size_t i = best_i; i-- > 0;) {
    const double d = evaluate(opts, limits[i], slots, &cur);
    if (d > best) break;
    best = d;
    *pick = cur;
  }
}

// For a launch that is to give every item a compute unit of its own: the smallest bound on the item time that at most
// `cus` items can meet, every tenant taking its option of fewest items within the bound.  Returns the longest item's time,
// or a negative number if no bound does.
static double choose_alone(const std::vector<std::vector<Option>>& opts, int cus, std::vector<int>* pick) {
  std::vector<double> limits;
  for (const auto& v : opts)
    for (const Option& op : v) limits.push_back(op.item_time);
  std::sort(limits.begin(), limits.end());
  auto fits = [&](double limit) {
    int64_t items = 0;
    pick->assign(opts.size(), 0);
    for (size_t t = 0; t < opts.size(); ++t) {
      int best = -1;
      for (size_t i = 0; i < opts[t].size(); ++i) {
        const Option& op = opts[t][i];
        if (op.item_time > limit) continue;
        if (best < 0 || op.items < opts[t][best].items || (op.items == opts[t][best].items && op.item_time < opts[t][best].item_time)) best = (int)i;
      }
      if (best < 0) return false;
      (*pick)[t] = best;
      items += opts[t][best].items;
    }
    return items <= cus;
  };
  size_t lo = 0, hi = limits.size();
  while (lo < hi) {
    const size_t mid = (lo + hi) / 2;
    if (fits(limits[mid])) hi = mid; else lo = mid + 1;
  }
  if (lo == limits.size() || !fits(limits[lo])) return -1.0;
  return limits[lo];
}

// The option for all tenants of a launch of one layer shape, where every work item takes as long as any other: slots are then
// filled in whole rounds, and what is left over for the last one has compute units of its own if there are enough.  shared, lone:
// the tenant's options priced for two workgroups on a compute unit and for one (item by item the same).  `pick`, the choice of the
// model that knows no rounds, stays unless another is a good part shorter; us per launch with it and with the other:
// 3x3 128->128 at 16x16 in fp32, 20 tenants 640 items 20.15, 480 19.57; 48 tenants 384 items 40.1, 768 35.5; 90 tenants, where the
// other is 2 % shorter by the model, 720 items 62.8, 1440 65.8.
static int choose_alike(const std::vector<Option>& shared, const std::vector<Option>& lone, int tenants, int pick) {
  auto duration = [&](size_t i) {
    const int64_t items = shared[i].items * tenants, rounds = items / (2 * kNumCUs), rest = items % (2 * kNumCUs);
    return (double)rounds * shared[i].item_time + (rest == 0 ? 0.0 : rest <= kNumCUs ? lone[i].item_time : shared[i].item_time);
  };
  int best = pick;
  for (size_t i = 0; i < shared.size(); ++i)
    if (duration(i) < duration((size_t)best) && duration(i) < 0.93 * duration((size_t)pick)) best = (int)i;
  return best;
}

// The model's duration of a launch with the given choice per tenant.
static double modelled(const std::vector<std::vector<Option>>& opts, const std::vector<int>& pick, int slots) {
  double longest = 0.0, area = 0.0;
  for (size_t t = 0; t < opts.size(); ++t) {
    longest = std::max(longest, opts[t][pick[t]].item_time);
    area += opts[t][pick[t]].area;
  }
  return std::max(longest, area / slots);
}

// Its duration as list scheduling has it, item by item on slots that are never shared out: a few items more than slots take a second round.
static double scheduled(const std::vector<std::vector<Option>>& opts, const std::vector<int>& pick, int slots) {
  std::vector<std::pair<double, int64_t>> runs;        // length and number of a tenant's items
  double end = 0.0;
  for (size_t t = 0; t < opts.size(); ++t) {
    const Option& op = opts[t][pick[t]];
    runs.push_back({op.area / (double)op.items, op.items});
    end = std::max(end, op.item_time);
  }
  std::sort(runs.begin(), runs.end(), [](const auto& a, const auto& b) { return a.first > b.first; });
  std::map<double, int64_t> idle{{0.0, slots}};        // slots by the time from which they are idle
  for (auto [length, items] : runs)
    while (items > 0) {
      const auto first = idle.begin();
      const int64_t n = std::min(items, first->second);
      const double done = first->first + length;
      if (n == first->second) idle.erase(first); else first->second -= n;
      idle[done] += n;
      items -= n;
      end = std::max(end, done);
    }
  return end;
}

// Where the model's sum of item times hides such a second round, the choices that other bounds on the item time lead to; `pick` stays
// unless one of them is a good part shorter.  For launches with stems or with layers whose channels are no multiple of the step, whose
// items fill a round unevenly: 13 of 265 such launches are planned differently, 0.91 (24.0 us -> 26.5) to 1.25 times as fast (17.4 -> 13.9), 1.075 in
// the geometric mean; eight layers with a stem of batch four, 604 items -> 420, 17.2 -> 13.3.
static void choose_rounds(const std::vector<std::vector<Option>>& opts, int slots, std::vector<int>* pick) {
  double best = scheduled(opts, *pick, slots), bound = 0.0;
  if (best < 1.07 * modelled(opts, *pick, slots)) return;
  for (size_t t = 0; t < opts.size(); ++t) bound = std::max(bound, opts[t][(*pick)[t]].item_time);
  best *= 0.93;
  std::vector<int> other;
  for (double f : {0.55, 0.62, 0.7, 0.78, 0.86, 0.93, 1.08, 1.17, 1.27, 1.4, 1.6, 1.8}) {
    double longest, area;
    evaluate_parts(opts, f * bound, &other, &longest, &area);
    const double d = scheduled(opts, other, slots);
    if (d < best) {
      best = d;
      *pick = other;
    }
  }
}

// What such a launch takes beyond its modelled duration with two workgroups on a compute unit: beside an unlike neighbour a tenth of the
// items takes more than half as long again as modelled, while on a unit of their own most are within 15 %.  106 launches with a plan of either kind,
// the one chosen against the other: 1.6 % longer in the geometric mean and 20 % at worst without this; 0.5 % and 8 % with it (with 1.2: 1.2 % and 34 %).
static const double kUnevenShared = 1.1;

static void destroy_device(st_plan* p) {
  if (p->d_arena) (void)hipFree(p->d_arena);
  p->d_arena = nullptr;
  if (p->ev_fork) (void)hipEventDestroy(p->ev_fork);
  for (hipEvent_t e : p->ev_join)
    if (e) (void)hipEventDestroy(e);
  p->d_tenants = nullptr;
  p->d_items_fused = p->d_items_tenant = nullptr;
  p->d_workspace = nullptr;
  p->ev_fork = nullptr;
  p->ev_join.clear();
}

// Device side of a plan: ONE allocation holding [tenant table][fused list][tenant-major list][split-K counters]
// [split-K partial tiles], filled by one copy (the counters travel as zeros); the partial tiles need no
// initialisation.  Events for the space-only fork/join are created on first use.
static st_status upload(st_plan* p) {
  const size_t n = p->tenants.size();
  if (n == 0) return ST_OK;
  size_t ws_floats = 0, counters = 0;
  for (size_t t = 0; t < n; ++t) {
    const st_tenant_info& ti = p->info[t];
    if (ti.split_k > 1) {
      ws_floats += (size_t)ti.tiles_m * ti.tiles_n * ti.split_k * ti.MT * ti.NT;
      counters += (size_t)ti.tiles_m * ti.tiles_n;
    }
  }
  p->workspace_bytes = (int64_t)(ws_floats * 4 + counters * 4);
  p->ws_floats = (int64_t)ws_floats;
  p->n_counters = (int64_t)counters;
  if (p->host_only) return ST_OK;
  auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
  const size_t ib = p->items_fused.size() * sizeof(st_work_item);
  const size_t off_fused = up(n * sizeof(TenantDev));
  const size_t off_tenant = off_fused + up(ib);
  const size_t off_counters = off_tenant + up(ib);
  const size_t off_ws = off_counters + up(counters * 4);
  const size_t total = off_ws + ws_floats * 4;
  ST_HIP(hipMalloc((void**)&p->d_arena, total));
  p->d_tenants = (TenantDev*)p->d_arena;
  p->d_items_fused = (st_work_item*)(p->d_arena + off_fused);
  p->d_items_tenant = (st_work_item*)(p->d_arena + off_tenant);
  p->d_workspace = p->d_arena + off_counters;
  size_t wf = 0, ct = 0;
  for (size_t t = 0; t < n; ++t) {
    const st_tenant_info& ti = p->info[t];
    if (ti.split_k > 1) {
      p->tenants[t].ws = (float*)(p->d_arena + off_ws) + wf;
      p->tenants[t].counters = (uint32_t*)(p->d_arena + off_counters) + ct;
      wf += (size_t)ti.tiles_m * ti.tiles_n * ti.split_k * ti.MT * ti.NT;
      ct += (size_t)ti.tiles_m * ti.tiles_n;
    }
  }
  std::vector<char> host;
  try {
    host.assign(off_ws, 0);
  } catch (const std::bad_alloc&) {
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  std::memcpy(host.data(), p->tenants.data(), n * sizeof(TenantDev));
  coded_items(p->tenants, p->items_fused, (st_work_item*)(host.data() + off_fused));
  coded_items(p->tenants, p->items_tenant, (st_work_item*)(host.data() + off_tenant));
  ST_HIP(hipMemcpy(p->d_arena, host.data(), off_ws, hipMemcpyHostToDevice));
  return ST_OK;
}

// Fork/join events of the space-only policy, made when that policy first runs on the plan.
static st_status ensure_events(const st_plan* cp) {
  st_plan* p = const_cast<st_plan*>(cp);
  if (p->ev_fork) return ST_OK;
  ST_HIP(hipEventCreateWithFlags(&p->ev_fork, hipEventDisableTiming));
  p->ev_join.assign(p->tenants.size(), nullptr);
  for (size_t t = 0; t < p->tenants.size(); ++t) ST_HIP(hipEventCreateWithFlags(&p->ev_join[t], hipEventDisableTiming));
  return ST_OK;
}

extern "C" st_status st_conv_plan(const st_conv_desc* descs, int32_t n_tenants, const st_plan_opts* opts,
                                  st_plan** out_plan) {
  if (!out_plan) return fail(ST_ERR_INVALID_ARG, "out_plan is NULL");
  *out_plan = nullptr;
  if (n_tenants < 0) return fail(ST_ERR_INVALID_ARG, "n_tenants is negative");
  if (n_tenants > 0 && !descs) return fail(ST_ERR_INVALID_ARG, "descs is NULL");
  if (n_tenants > 65535) return fail(ST_ERR_UNSUPPORTED, "at most 65535 tenants per plan");
  st_plan_opts o;
  std::memset(&o, 0, sizeof(o));
  if (opts) o = *opts;
  if (o.tile_cfg < 0 || o.tile_cfg > kNumTileCfgs) return fail(ST_ERR_INVALID_ARG, "opts.tile_cfg out of range");
  if (o.split_k < 0 || o.order < 0 || o.order > 2 || o.target_items < 0 ||
      !(o.rows_per_tile == 0 || o.rows_per_tile == 1 || o.rows_per_tile == 2 || o.rows_per_tile == 4) ||
      o.chain_queues < 0 || o.chain_queues > 2 || o.reserved != 0)
    return fail(ST_ERR_INVALID_ARG, "opts: negative or unknown value");
  for (int t = 0; t < n_tenants; ++t) {
    st_status s = validate(descs[t], t);
    if (s != ST_OK) return s;
  }
  st_plan* p = new (std::nothrow) st_plan();
  if (!p) return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  try {
    p->host_only = o.host_only != 0;
    p->descs.assign(descs, descs + n_tenants);
    p->info.resize(n_tenants);
    p->tenants.resize(n_tenants);
    // derived sizes
    for (int t = 0; t < n_tenants; ++t) {
      const st_conv_desc& d = descs[t];
      st_tenant_info& ti = p->info[t];
      std::memset(&ti, 0, sizeof(ti));
      ti.P = (d.H + 2 * d.pad - d.R) / d.stride + 1;
      ti.Q = (d.W + 2 * d.pad - d.S) / d.stride + 1;
      ti.M = (int64_t)d.N * ti.P * ti.Q;
      ti.Ngemm = d.K;
      ti.Kgemm = (int64_t)d.C * d.R * d.S;
      ti.flops = 2 * ti.M * ti.Ngemm * ti.Kgemm;
      ti.bytes = ((int64_t)d.N * d.C * d.H * d.W + ti.Ngemm * ti.Kgemm) * elem_size(d.in_dtype) +
                 ti.M * ti.Ngemm * elem_size(d.out_dtype);
      p->flops += ti.flops;
      p->bytes += ti.bytes;
    }
    // tile shape and split-K per tenant, chosen jointly from the cost model
    bool any_filters = false;       // several types, or a form for any channel count (launch_conv)
    for (int t = 0; t < n_tenants; ++t) any_filters |= descs[t].in_dtype != descs[0].in_dtype || (!vector_ok(descs[t]) && !row_tile_ok(descs[t]));
    auto all_options = [&](bool alone) {
      std::vector<std::vector<Option>> options(n_tenants);
      for (int t = 0; t < n_tenants; ++t) {
        const st_tenant_info& ti = p->info[t];
        options[t] = tenant_options(descs[t], ti.M, ti.Ngemm, alone, any_filters, o);
      }
      return options;
    };
    std::vector<std::vector<Option>> options = all_options(false);
    std::vector<int> pick;
    choose_all(options, o.target_items > 0 ? o.target_items : kSlots, &pick);
    bool alike = n_tenants > 1;
    for (int t = 1; t < n_tenants; ++t) {
      const st_conv_desc &a = descs[0], &b = descs[t];
      alike = alike && a.N == b.N && a.C == b.C && a.H == b.H && a.W == b.W && a.K == b.K && a.R == b.R && a.S == b.S && a.stride == b.stride && a.pad == b.pad &&
              a.in_dtype == b.in_dtype && a.out_dtype == b.out_dtype;
    }
    // stems, and layers whose channels are no multiple of the step
    bool uneven = false;
    for (int t = 0; t < n_tenants; ++t) uneven |= (int64_t)descs[t].C * elem_size(descs[t].in_dtype) % 128 != 0;
    if (o.target_items == 0) {
      // A launch of no more work items than compute units puts every workgroup on a compute unit of its own.  Plan for
      // that too, and take it if the model says it is the shorter launch (one 3x3 layer of each of a ResNet's four stages,
      // batch 1: 207 items 6.7 us, the shared plan's 399 7.5; eight 3x3 layers 256->256 at 14x14: 224 tiles of 64x64 8.1 us,
      // 416 of 32x64 8.25).
      const bool rounds = !alike && uneven;
      if (rounds) choose_rounds(options, 2 * kNumCUs, &pick);
      std::vector<std::vector<Option>> lone = all_options(true);
      std::vector<int> alone;
      const double longest = choose_alone(lone, kNumCUs, &alone);
      if (longest >= 0.0 && longest < (rounds ? kUnevenShared * scheduled(options, pick, 2 * kNumCUs) : modelled(options, pick, 2 * kNumCUs))) {
        options.swap(lone);
        pick = alone;
      } else if (alike) {
        pick.assign((size_t)n_tenants, choose_alike(options[0], lone[0], n_tenants, pick[0]));
      }
    }
    std::vector<int> form;
    int64_t fused_total = 0;
    for (int t = 0; t < n_tenants; ++t) {
      st_tenant_info& ti = p->info[t];
      const Option& op = options[t][pick[t]];
      p->item_time.push_back(op.item_time);
      form.push_back(op.form);
      ti.tile_cfg = op.cfg;
      const KSteps k = k_steps_of(descs[t], op.form, op.cfg);
      ti.k_steps = k.main + k.left;
      ti.MT = kTileShapes[op.cfg].MT;
      ti.NT = kTileShapes[op.cfg].NT;
      ti.tiles_m = cdiv(ti.M, ti.MT);
      ti.row_tiled = (op.cfg == kRowCfg) ? 1 : 0;
      if (ti.row_tiled) {
        ti.k_steps = descs[t].R;
        ti.tiles_m = descs[t].N * cdiv(ti.P, op.rows_per_tile) * cdiv(ti.Q, ti.MT);
        ti.rows_per_tile = op.rows_per_tile;
      }
      ti.tiles_n = cdiv(ti.Ngemm, ti.NT);
      ti.split_k = op.split;
      ti.k_steps_per_split = op.steps_per_split;
      ti.item_begin = fused_total;
      ti.item_count = (int64_t)ti.tiles_m * ti.tiles_n * op.split;
      xcd_block_choice(descs[t], ti, kNumXCDs, &ti.xcd_blocks_m, &ti.xcd_blocks_n);
      fused_total += ti.item_count;
    }
    if (fused_total >= ((int64_t)1 << 31)) {
      delete p;
      return fail(ST_ERR_UNSUPPORTED, "more than 2^31 work items");
    }
    // tenant-major work list: tenant, pixel tile, filter tile, K slice
    p->items_tenant.reserve((size_t)fused_total);
    for (int t = 0; t < n_tenants; ++t) {
      const st_tenant_info& ti = p->info[t];
      for (int tm = 0; tm < ti.tiles_m; ++tm)
        for (int tn = 0; tn < ti.tiles_n; ++tn)
          for (int s = 0; s < ti.split_k; ++s) {
            st_work_item it;
            it.tenant = (uint16_t)t;
            it.k_split_idx = (uint16_t)s;
            it.tile_m = (uint32_t)tm;
            it.tile_n = (uint32_t)tn;
            it.reserved = 0;
            p->items_tenant.push_back(it);
          }
    }
    // fused order: longest work item first, so that short items fill the tail of the launch
    p->items_fused = p->items_tenant;
    // each tenant's launch of its own (the baselines) starts at its first item: XCD = position in the range, mod 8
    for (int t = 0; t < n_tenants; ++t) {
      const st_tenant_info& ti = p->info[t];
      xcd_arrange(p->items_tenant.data() + ti.item_begin, ti.item_count, 0, ti);
    }
    if (o.order == 1) p->items_fused = p->items_tenant;
    if (o.order == 2) {
      // equal progress: position by position, the tenant that is furthest behind its share of the launch goes
      // next (the one minimising (emitted + 1) / count; lowest tenant on ties), taking its items in their
      // tenant-major order
      std::vector<int64_t> emitted((size_t)n_tenants, 0);
      for (size_t q = 0; q < p->items_fused.size(); ++q) {
        int best = -1;
        for (int t = 0; t < n_tenants; ++t) {
          const int64_t c = p->info[t].item_count;
          if (emitted[t] >= c) continue;
          // (emitted[t] + 1) / c < (emitted[best] + 1) / c_best, in integers
          if (best < 0 || (emitted[t] + 1) * p->info[best].item_count < (emitted[best] + 1) * c) best = t;
        }
        p->items_fused[q] = p->items_tenant[(size_t)(p->info[best].item_begin + emitted[best])];
        ++emitted[best];
      }
    }
    if (o.order == 0) {
      // A tenant's items differ by their K slice only (the last one is shorter; in pieces the steps of the channels left over, which
      // lie at the end, are longer), so sorting the items by cost (stably, from the nested tenant-major order) is sorting
      // runs of slices that cost the same, few per tenant.
      // What every tile spends until its first operands is left out, but not what a row tile copies beyond that: without it, items of
      // two rows and 10 us counted less than others of 6 us and started last (13 tenants, one of them a stem, 13.6 us -> 12.4; 30 tenants
      // with three 43.5 -> 40.3; 120 launches with stems 0.95 to 1.10 times as fast, 1.006 in the geometric mean).
      constexpr double kUsualFirst = 4000.0;
      struct Run { int tenant, begin, end; int64_t cost, count; };      // K slices [begin, end) of every tile
      std::vector<Run> runs;
      runs.reserve((size_t)n_tenants * 2);
      for (int t = 0; t < n_tenants; ++t) {
        const st_tenant_info& ti = p->info[t];
        const ItemCosts& c = item_costs(descs[t], ti.tile_cfg, false, false);
        const KSteps k = k_steps_of(descs[t], form[t], ti.tile_cfg);
        const int64_t tiles = ti.item_count / ti.split_k;
        auto cost = [&](int slice) {
          const int begin = slice * ti.k_steps_per_split, end = std::min(ti.k_steps, begin + ti.k_steps_per_split);
          if (ti.row_tiled)
            return (int64_t)(c.first[kRowCfg] + row_stage_cost(ti.rows_per_tile) - kUsualFirst + ti.rows_per_tile * ((end - begin) * c.step[kRowCfg] + c.epi[kRowCfg]));
          return (int64_t)(steps_cost(descs[t], form[t], ti.tile_cfg, c, false, k, begin, end) + epilogue_cost(descs[t], form[t], ti.tile_cfg, c, false, any_filters));
        };
        for (int i = 0; i < ti.split_k; ++i) {
          const int64_t mine = cost(i);
          if (i > 0 && runs.back().cost == mine) {
            ++runs.back().end;
            runs.back().count += tiles;
          } else {
            runs.push_back({t, i, i + 1, mine, tiles});
          }
        }
      }
      std::stable_sort(runs.begin(), runs.end(), [](const Run& a, const Run& b) { return a.cost > b.cost; });
      p->items_fused.clear();
      for (const Run& r : runs) {
        const st_tenant_info& ti = p->info[r.tenant];
        for (int tm = 0; tm < ti.tiles_m; ++tm)
          for (int tn = 0; tn < ti.tiles_n; ++tn)
            for (int s = r.begin; s < r.end; ++s) {
              st_work_item it;
              it.tenant = (uint16_t)r.tenant;
              it.k_split_idx = (uint16_t)s;
              it.tile_m = (uint32_t)tm;
              it.tile_n = (uint32_t)tn;
              it.reserved = 0;
              p->items_fused.push_back(it);
            }
      }
      // Placement: a stretch of at least 8 runs whose items cost about the same (within a fifth) is shared out tenant by
      // tenant; otherwise every run is cut into 8 blocks, each kept on one XCD.
      size_t r0 = 0;
      int64_t at = 0;
      while (r0 < runs.size()) {
        size_t r1 = r0;
        std::vector<ItemRun> stretch;
        for (int64_t b = at; r1 < runs.size() && runs[r1].cost * 5 >= runs[r0].cost * 4; ++r1) {
          stretch.push_back({runs[r1].tenant, b, b + runs[r1].count});
          b += runs[r1].count;
        }
        if (stretch.size() >= (size_t)kNumXCDs) {
          xcd_arrange_tenants(p->items_fused.data(), stretch, p->descs, p->info);
        } else {
          for (const ItemRun& r : stretch)
            xcd_arrange(p->items_fused.data() + r.begin, r.end - r.begin, (int)(r.begin % kNumXCDs), p->info[r.tenant]);
        }
        at = stretch.back().end;
        r0 = r1;
      }
    }
    // device records
    for (int t = 0; t < n_tenants; ++t) {
      const st_conv_desc& d = descs[t];
      const st_tenant_info& ti = p->info[t];
      TenantDev& T = p->tenants[t];
      std::memset(&T, 0, sizeof(T));
      T.x = d.x; T.w = d.w; T.y = d.y; T.res = d.residual;
      T.C = d.C; T.H = d.H; T.W = d.W; T.K = d.K; T.R = d.R; T.S = d.S; T.stride = d.stride; T.pad = d.pad;
      T.P = ti.P; T.Q = ti.Q; T.PQ = ti.P * ti.Q; T.M = (int32_t)ti.M; T.Kg = (int32_t)ti.Kgemm;
      T.in_dtype = d.in_dtype; T.out_dtype = d.out_dtype; T.epilogue = (int32_t)d.epilogue;
      T.cfg = ti.tile_cfg; T.split_k = ti.split_k; T.k_steps = ti.k_steps; T.k_steps_per_split = ti.k_steps_per_split;
      T.tiles_m = ti.tiles_m; T.tiles_n = ti.tiles_n;
      T.vec_ok = form[t];
      const int kt = kTileShapes[ti.tile_cfg].KB / elem_size(d.in_dtype);
      T.step_dr = (int32_t)(kt / ((int64_t)d.S * d.C));
      T.step_dk = (int32_t)(kt % ((int64_t)d.S * d.C));
      T.k_order = d.C % kt != 0 || (int64_t)d.R * d.S > 32 ? kOrderTaps : (d.R == 1 && d.S == 1 && d.pad == 0) ? kOrderLinear : kOrderChannels;
      for (int r = 0; T.k_order == kOrderChannels && r < d.R; ++r) T.tap_rows |= 1u << (r * d.S);
      if (patch_geometry(d, ti.tile_cfg, &T.patch_rows, &T.patch_loads) && ti.k_steps_per_split % kPatchTaps == 0) {
        T.k_order = kOrderPatch;
        T.patch_blocks = ti.k_steps_per_split / kPatchTaps;
      }
      magic_for(d.C, &T.magic_c, &T.shift_c);
      magic_for(d.S, &T.magic_s, &T.shift_s);
      T.row_pitch = row_tile_pitch(d);
      magic_for(T.row_pitch / 16, &T.magic_nvp, &T.shift_nvp);
      if (form[t] == kPieces) {
        const KSteps k = k_steps_of(d, kPieces, ti.tile_cfg);
        T.k_order = kOrderPieces;
        T.step_dk = k.vectors;
        T.step_dr = k.main;
        magic_for(k.vectors, &T.magic_c, &T.shift_c);
      }
      magic_for(d.R, &T.magic_r, &T.shift_r);
      magic_for(T.PQ, &T.magic_pq, &T.shift_pq);
      magic_for(T.Q, &T.magic_q, &T.shift_q);
      T.x_bytes = (uint32_t)((int64_t)d.N * d.C * d.H * d.W * elem_size(d.in_dtype));
      T.w_bytes = (uint32_t)(ti.Ngemm * ti.Kgemm * elem_size(d.in_dtype));
      T.y_bytes = (uint32_t)(ti.M * ti.Ngemm * elem_size(d.out_dtype));
      T.rows_per_tile = ti.rows_per_tile;
      p->kernel_needs |= kernel_needs(T);
    }
  } catch (const std::bad_alloc&) {
    delete p;
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  st_status s = upload(p);
  if (s != ST_OK) {
    destroy_device(p);
    delete p;
    return s;
  }
  *out_plan = p;
  return ST_OK;
}

static st_status check_runnable(const st_plan* plan) {
  if (!plan) return fail(ST_ERR_INVALID_ARG, "plan is NULL");
  if (plan->host_only) return fail(ST_ERR_UNSUPPORTED, "plan was built host-only and cannot run");
  return ST_OK;
}

extern "C" st_status st_conv_run(const st_plan* plan, void* hip_stream) {
  st_status s = check_runnable(plan);
  if (s != ST_OK) return s;
  if (plan->items_fused.empty()) return ST_OK;
  ST_HIP((hipError_t)launch_conv(plan->kernel_needs, plan->d_tenants, plan->d_items_fused, (int64_t)plan->items_fused.size(), hip_stream, nullptr));
  return ST_OK;
}

// The fused launch for callers that cannot allocate device memory.  Scratch layout: [tenant table][work list]
// [split-K counters][split-K partial tiles], each part on a 256-byte boundary.
extern "C" int64_t st_conv_noalloc_max_bytes(void) { return kNoallocScratchBytes; }

extern "C" st_status st_conv_run_noalloc(const st_plan* plan, void* hip_stream) {
  if (!plan) return fail(ST_ERR_INVALID_ARG, "plan is NULL");
  const size_t n = plan->tenants.size();
  if (n == 0 || plan->items_fused.empty()) return ST_OK;
  auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
  const size_t ib = plan->items_fused.size() * sizeof(st_work_item);
  const size_t off_items = up(n * sizeof(TenantDev));
  const size_t off_counters = off_items + up(ib);
  const size_t off_ws = off_counters + up((size_t)plan->n_counters * 4);
  const size_t total = off_ws + (size_t)plan->ws_floats * 4;
  if ((int64_t)total > kNoallocScratchBytes)
    return fail(ST_ERR_UNSUPPORTED, "st_conv_run_noalloc: the plan needs %lld bytes of tables and split-K workspace, the fixed scratch "
                "array holds %lld", (long long)total, (long long)kNoallocScratchBytes);
  void* base = nullptr;
  ST_HIP((hipError_t)noalloc_scratch(&base));
  char* dev = (char*)base;
  std::vector<char> host;
  try {
    host.assign(off_counters, 0);
  } catch (const std::bad_alloc&) {
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  TenantDev* table = (TenantDev*)host.data();
  std::memcpy(table, plan->tenants.data(), n * sizeof(TenantDev));
  size_t wf = 0, ct = 0;
  for (size_t t = 0; t < n; ++t) {
    const st_tenant_info& ti = plan->info[t];
    table[t].ws = nullptr;
    table[t].counters = nullptr;
    if (ti.split_k > 1) {
      table[t].ws = (float*)(dev + off_ws) + wf;
      table[t].counters = (uint32_t*)(dev + off_counters) + ct;
      wf += (size_t)ti.tiles_m * ti.tiles_n * ti.split_k * ti.MT * ti.NT;
      ct += (size_t)ti.tiles_m * ti.tiles_n;
    }
  }
  coded_items(plan->tenants, plan->items_fused, (st_work_item*)(host.data() + off_items));
  ST_HIP((hipError_t)launch_poke(host.data(), (int64_t)off_counters, dev, hip_stream));
  // the array keeps the last call's contents: the arrival counters must start at zero (the partial tiles need not)
  if (plan->n_counters > 0) ST_HIP((hipError_t)launch_zero(dev + off_counters, (int64_t)up((size_t)plan->n_counters * 4), hip_stream));
  ST_HIP((hipError_t)launch_conv(plan->kernel_needs, (const TenantDev*)dev, (const st_work_item*)(dev + off_items), (int64_t)plan->items_fused.size(),
                                 hip_stream, nullptr));
  return ST_OK;
}

extern "C" st_status st_conv_run_profiled(const st_plan* plan, void* hip_stream, uint64_t* stamps, int64_t capacity) {
  st_status s = check_runnable(plan);
  if (s != ST_OK) return s;
  const int64_t n = (int64_t)plan->items_fused.size();
  if (!stamps || capacity < n * kProfSlots) return fail(ST_ERR_INVALID_ARG, "stamps buffer too small: need %lld entries", (long long)(n * kProfSlots));
  if (n == 0) return ST_OK;
  uint64_t* d = nullptr;
  ST_HIP(hipMalloc((void**)&d, (size_t)n * kProfSlots * 8));
  hipError_t e = hipMemsetAsync(d, 0, (size_t)n * kProfSlots * 8, (hipStream_t)hip_stream);   // ordered before the launch
  if (e == hipSuccess) e = (hipError_t)launch_conv(plan->kernel_needs, plan->d_tenants, plan->d_items_fused, n, hip_stream, d);
  if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)hip_stream);
  if (e == hipSuccess) e = hipMemcpy(stamps, d, (size_t)n * kProfSlots * 8, hipMemcpyDeviceToHost);
  (void)hipFree(d);
  if (e != hipSuccess) return hip_fail(e, "st_conv_run_profiled");
  return ST_OK;
}

extern "C" st_status st_conv_run_tenant_times(const st_plan* plan, void* hip_stream, int64_t* first_start_ns,
                                              int64_t* last_end_ns, int32_t n_tenants) {
  st_status s = check_runnable(plan);
  if (s != ST_OK) return s;
  if (!first_start_ns || !last_end_ns) return fail(ST_ERR_INVALID_ARG, "NULL output");
  if (n_tenants != (int32_t)plan->tenants.size()) return fail(ST_ERR_INVALID_ARG, "n_tenants differs from the plan's");
  const size_t n = plan->items_fused.size();
  std::vector<uint64_t> stamps;
  try {
    stamps.resize(n * kProfSlots);
  } catch (const std::bad_alloc&) {
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  s = st_conv_run_profiled(plan, hip_stream, stamps.data(), (int64_t)stamps.size());
  if (s != ST_OK) return s;
  uint64_t t0 = ~(uint64_t)0;
  for (size_t i = 0; i < n; ++i) t0 = std::min(t0, stamps[i * kProfSlots + 4]);
  for (int t = 0; t < n_tenants; ++t) { first_start_ns[t] = -1; last_end_ns[t] = -1; }
  for (size_t i = 0; i < n; ++i) {
    const int t = plan->items_fused[i].tenant;
    const int64_t b = (int64_t)(stamps[i * kProfSlots + 4] - t0) * 10, e = (int64_t)(stamps[i * kProfSlots + 6] - t0) * 10;
    if (first_start_ns[t] < 0 || b < first_start_ns[t]) first_start_ns[t] = b;
    if (e > last_end_ns[t]) last_end_ns[t] = e;
  }
  return ST_OK;
}

extern "C" st_status st_conv_run_time_only(const st_plan* plan, void* hip_stream) {
  st_status s = check_runnable(plan);
  if (s != ST_OK) return s;
  for (size_t t = 0; t < plan->info.size(); ++t) {
    const st_tenant_info& ti = plan->info[t];
    ST_HIP((hipError_t)launch_conv(plan->kernel_needs, plan->d_tenants, plan->d_items_tenant + ti.item_begin, ti.item_count, hip_stream, nullptr));
  }
  return ST_OK;
}

extern "C" st_status st_conv_run_space_only(const st_plan* plan, void* const* hip_streams, int32_t n_streams) {
  st_status s = check_runnable(plan);
  if (s != ST_OK) return s;
  if (!hip_streams || n_streams <= 0) return fail(ST_ERR_INVALID_ARG, "need at least one stream");
  const size_t n = plan->info.size();
  if (n == 0) return ST_OK;
  hipStream_t anchor = (hipStream_t)hip_streams[0];
  const size_t used = std::min<size_t>(n, (size_t)n_streams);
  if (used > 1) {
    s = ensure_events(plan);
    if (s != ST_OK) return s;
    ST_HIP(hipEventRecord(plan->ev_fork, anchor));
    for (size_t i = 1; i < used; ++i) ST_HIP(hipStreamWaitEvent((hipStream_t)hip_streams[i], plan->ev_fork, 0));
  }
  for (size_t t = 0; t < n; ++t) {
    const st_tenant_info& ti = plan->info[t];
    ST_HIP((hipError_t)launch_conv(plan->kernel_needs, plan->d_tenants, plan->d_items_tenant + ti.item_begin, ti.item_count,
                                   hip_streams[t % (size_t)n_streams], nullptr));
  }
  for (size_t i = 1; i < used; ++i) {
    ST_HIP(hipEventRecord(plan->ev_join[i], (hipStream_t)hip_streams[i]));
    ST_HIP(hipStreamWaitEvent(anchor, plan->ev_join[i], 0));
  }
  return ST_OK;
}

// Baselines with per-tenant plans: each plan (normally one tenant, planned alone so that its tiles suit a
// launch that has the whole GPU to itself) is issued as its own fused launch.
extern "C" st_status st_conv_run_plans_time_only(const st_plan* const* plans, int32_t n_plans, void* hip_stream) {
  if (n_plans < 0 || (n_plans > 0 && !plans)) return fail(ST_ERR_INVALID_ARG, "plans is NULL or n_plans negative");
  for (int32_t i = 0; i < n_plans; ++i) {
    st_status s = st_conv_run(plans[i], hip_stream);
    if (s != ST_OK) return s;
  }
  return ST_OK;
}

extern "C" st_status st_conv_run_plans_space_only(const st_plan* const* plans, int32_t n_plans, void* const* hip_streams,
                                                  int32_t n_streams) {
  if (n_plans < 0 || (n_plans > 0 && !plans)) return fail(ST_ERR_INVALID_ARG, "plans is NULL or n_plans negative");
  if (!hip_streams || n_streams <= 0) return fail(ST_ERR_INVALID_ARG, "need at least one stream");
  if (n_plans == 0) return ST_OK;
  for (int32_t i = 0; i < n_plans; ++i) {
    st_status s = check_runnable(plans[i]);
    if (s != ST_OK) return s;
  }
  hipStream_t anchor = (hipStream_t)hip_streams[0];
  const int32_t used = std::min(n_plans, n_streams);
  // fork: plans[0]'s event marks the work already queued on the anchor stream
  const st_plan* first = nullptr;
  for (int32_t i = 0; i < n_plans && !first; ++i)
    if (!plans[i]->tenants.empty()) first = plans[i];
  if (used > 1 && first) {
    st_status s = ensure_events(first);
    if (s != ST_OK) return s;
    ST_HIP(hipEventRecord(first->ev_fork, anchor));
    for (int32_t i = 1; i < used; ++i) ST_HIP(hipStreamWaitEvent((hipStream_t)hip_streams[i], first->ev_fork, 0));
  }
  for (int32_t i = 0; i < n_plans; ++i) {
    st_status s = st_conv_run(plans[i], hip_streams[i % n_streams]);
    if (s != ST_OK) return s;
  }
  // join: the last plan issued on each non-anchor stream lends its event
  for (int32_t sidx = 1; sidx < used; ++sidx) {
    const st_plan* last = nullptr;
    for (int32_t i = sidx; i < n_plans; i += n_streams)
      if (!plans[i]->tenants.empty()) last = plans[i];
    if (!last) continue;
    st_status s = ensure_events(last);
    if (s != ST_OK) return s;
    ST_HIP(hipEventRecord(last->ev_join[0], (hipStream_t)hip_streams[sidx]));
    ST_HIP(hipStreamWaitEvent(anchor, last->ev_join[0], 0));
  }
  return ST_OK;
}

// Issue `total` fused launches from several host threads: launch L runs plans[L mod n_plans] on stream
// streams[stream_of(L)]; thread t issues the launches whose stream index is t mod n_threads, in sequence order, so
// the order on every stream is that of a serial loop.  A launch costs the host about 2.3 us, more than a small
// fused launch needs on the device once several are in flight.
// A plan with a split-K workspace must not run on two streams at once (its partial tiles and arrival counters are
// shared by all its runs).  stream_of(i) is the stream index that launch i of one round of the sequence goes to,
// period = launches after which the (plan, stream) pattern repeats.
template <class StreamOf>
static st_status check_workspace_streams(const st_plan* const* plans, int32_t n_plans, int64_t period, StreamOf stream_of,
                                         const char* where) {
  for (int32_t i = 0; i < n_plans; ++i) {
    if (!plans[i] || plans[i]->workspace_bytes == 0) continue;
    long first = -1;
    for (int64_t L = 0; L < period; ++L) {
      if (plans[L % n_plans] != plans[i]) continue;
      const long si = (long)stream_of(L);
      if (first < 0) first = si;
      else if (si != first)
        return fail(ST_ERR_INVALID_ARG, "%s: plan %d owns a split-K workspace and would be queued on more than one stream", where, i);
    }
  }
  return ST_OK;
}

template <class StreamOf>
static st_status issue_threaded(const st_plan* const* plans, int32_t n_plans, const std::vector<hipStream_t>& streams,
                                int64_t total, int n_threads, StreamOf stream_of, const char* where) {
  for (int32_t i = 0; i < n_plans; ++i) {
    st_status s = check_runnable(plans[i]);
    if (s != ST_OK) return s;
  }
  int device = 0;
  ST_HIP(hipGetDevice(&device));
  std::vector<int> status((size_t)n_threads, (int)hipSuccess);
  auto work = [&](int t) {
    if (hipSetDevice(device) != hipSuccess) { status[(size_t)t] = (int)hipErrorInvalidDevice; return; }
    for (int64_t L = 0; L < total; ++L) {
      const size_t si = stream_of(L);
      if ((int)(si % (size_t)n_threads) != t) continue;
      const st_plan* plan = plans[L % n_plans];
      const int e = launch_conv(plan->kernel_needs, plan->d_tenants, plan->d_items_fused, (int64_t)plan->items_fused.size(), (void*)streams[si], nullptr);
      if (e != (int)hipSuccess) { status[(size_t)t] = e; return; }
    }
  };
  std::vector<std::thread> workers;
  int started = 1;                       // share 0 is the calling thread's
  try {
    for (; started < n_threads; ++started) workers.emplace_back(work, started);
  } catch (...) {
    // no more threads to be had: the calling thread takes the shares that have no thread of their own
  }
  work(0);
  for (int t = started; t < n_threads; ++t) work(t);
  for (std::thread& w : workers) w.join();
  for (int e : status)
    if (e != (int)hipSuccess) return hip_fail((hipError_t)e, where);
  return ST_OK;
}

static int issue_threads(size_t n_streams) {
  int n = (int)std::min<size_t>(n_streams, 4);
  if (const char* env = std::getenv("ST_PIPELINE_THREADS")) n = std::max(1, std::min(atoi(env), (int)n_streams));
  return n;
}

extern "C" st_status st_conv_run_plans_on_streams_many(const st_plan* const* plans, int32_t n_plans, void* const* hip_streams,
                                                       int32_t n_streams, int32_t rounds) {
  if (n_plans < 0 || rounds < 0 || (n_plans > 0 && !plans)) return fail(ST_ERR_INVALID_ARG, "plans is NULL or a count is negative");
  if (!hip_streams || n_streams <= 0) return fail(ST_ERR_INVALID_ARG, "need at least one stream");
  const int64_t total = (int64_t)rounds * n_plans;
  const size_t used = (size_t)std::min(n_plans, n_streams);
  for (int32_t i = 0; i < n_plans; ++i)
    if (!plans[i]) return fail(ST_ERR_INVALID_ARG, "plans[%d] is NULL", i);
  {
    st_status s = check_workspace_streams(plans, n_plans, n_plans, [=](int64_t L) { return (size_t)(L % n_streams); },
                                          "st_conv_run_plans_on_streams_many");
    if (s != ST_OK) return s;
  }
  const int n_threads = issue_threads(used);
  if (total < 64 || n_threads < 2) {
    for (int32_t r = 0; r < rounds; ++r) {
      st_status s = st_conv_run_plans_on_streams(plans, n_plans, hip_streams, n_streams);
      if (s != ST_OK) return s;
    }
    return ST_OK;
  }
  std::vector<hipStream_t> streams((hipStream_t*)hip_streams, (hipStream_t*)hip_streams + n_streams);
  return issue_threaded(plans, n_plans, streams, total, n_threads,
                        [=](int64_t L) { return (size_t)((L % n_plans) % n_streams); }, "st_conv_run_plans_on_streams_many (worker thread)");
}

extern "C" st_status st_conv_run_plans_on_streams(const st_plan* const* plans, int32_t n_plans, void* const* hip_streams,
                                                  int32_t n_streams) {
  if (n_plans < 0 || (n_plans > 0 && !plans)) return fail(ST_ERR_INVALID_ARG, "plans is NULL or n_plans negative");
  if (!hip_streams || n_streams <= 0) return fail(ST_ERR_INVALID_ARG, "need at least one stream");
  for (int32_t i = 0; i < n_plans; ++i)
    if (!plans[i]) return fail(ST_ERR_INVALID_ARG, "plans[%d] is NULL", i);
  {
    st_status s = check_workspace_streams(plans, n_plans, n_plans, [=](int64_t L) { return (size_t)(L % n_streams); },
                                          "st_conv_run_plans_on_streams");
    if (s != ST_OK) return s;
  }
  for (int32_t i = 0; i < n_plans; ++i) {
    st_status s = st_conv_run(plans[i], hip_streams[i % n_streams]);
    if (s != ST_OK) return s;
  }
  return ST_OK;
}

extern "C" st_status st_conv_plan_rebind(st_plan* plan, int32_t tenant, const void* x, const void* w, void* y,
                                         const void* residual) {
  if (!plan) return fail(ST_ERR_INVALID_ARG, "plan is NULL");
  if (tenant < 0 || (size_t)tenant >= plan->tenants.size()) return fail(ST_ERR_INVALID_ARG, "tenant index out of range");
  TenantDev T = plan->tenants[tenant];
  if (x) T.x = x;
  if (w) T.w = w;
  if (y) T.y = y;
  if (residual) T.res = residual;
  if (T.y == T.x || T.y == T.w) return fail(ST_ERR_INVALID_ARG, "y must not alias x or w");
  if (!plan->host_only)
    ST_HIP(hipMemcpy(plan->d_tenants + tenant, &T, sizeof(T), hipMemcpyHostToDevice));
  plan->tenants[tenant] = T;
  st_conv_desc& d = plan->descs[tenant];
  d.x = T.x; d.w = T.w; d.y = T.y; d.residual = T.res;
  return ST_OK;
}

extern "C" st_status st_conv_plan_rebind_all(st_plan* plan, const st_conv_desc* descs, int32_t n_tenants, void* hip_stream) {
  if (!plan) return fail(ST_ERR_INVALID_ARG, "plan is NULL");
  if (n_tenants != (int32_t)plan->tenants.size()) return fail(ST_ERR_INVALID_ARG, "n_tenants differs from the plan's");
  if (n_tenants > 0 && !descs) return fail(ST_ERR_INVALID_ARG, "descs is NULL");
  bool changed = false;
  for (int t = 0; t < n_tenants; ++t) {
    const st_conv_desc& d = descs[t];
    const TenantDev& T = plan->tenants[t];
    if (!d.x || !d.w || !d.y) return fail(ST_ERR_INVALID_ARG, "tenant %d: x, w and y must be non-NULL", t);
    if (d.y == d.x || d.y == d.w) return fail(ST_ERR_INVALID_ARG, "tenant %d: y must not alias x or w", t);
    if ((T.epilogue & ST_EPI_RESIDUAL) && !d.residual)
      return fail(ST_ERR_INVALID_ARG, "tenant %d: the plan adds a residual but none is given", t);
    changed |= d.x != T.x || d.w != T.w || d.y != T.y || ((T.epilogue & ST_EPI_RESIDUAL) && d.residual != T.res);
  }
  if (!changed) return ST_OK;
  // The new table is assembled in a copy; the plan's host mirrors are replaced only once the upload is queued, so a
  // failed call leaves the plan describing what the device table still holds.
  std::vector<TenantDev> next;
  try {
    next = plan->tenants;
  } catch (const std::bad_alloc&) {
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  for (int t = 0; t < n_tenants; ++t) {
    const st_conv_desc& d = descs[t];
    TenantDev& T = next[t];
    T.x = d.x; T.w = d.w; T.y = d.y;
    if (T.epilogue & ST_EPI_RESIDUAL) T.res = d.residual;
  }
  if (!plan->host_only) ST_HIP((hipError_t)launch_bind(next.data(), n_tenants, plan->d_tenants, hip_stream));
  plan->tenants.swap(next);
  for (int t = 0; t < n_tenants; ++t) {
    const TenantDev& T = plan->tenants[t];
    st_conv_desc& mine = plan->descs[t];
    mine.x = T.x; mine.w = T.w; mine.y = T.y; mine.residual = T.res;
  }
  return ST_OK;
}

// ---------------------------------------------------------------------------------------------------
// plan cache: the ready set of tenants changes from step to step; plans are keyed by everything in the
// descriptors except the pointers
// ---------------------------------------------------------------------------------------------------
struct st_plan_cache {
  struct Entry {
    std::vector<int32_t> key;
    st_plan* plan = nullptr;
    uint64_t last_use = 0;
  };
  std::vector<Entry> entries;
  st_plan_opts opts;
  int capacity = 0;
  uint64_t clock = 0;
  int64_t hits = 0, misses = 0, evictions = 0;
};

static void cache_key(const st_conv_desc* descs, int32_t n, std::vector<int32_t>* key) {
  key->clear();
  key->reserve((size_t)n * 14 + 1);
  key->push_back(n);
  for (int t = 0; t < n; ++t) {
    const st_conv_desc& d = descs[t];
    const int32_t f[14] = {d.N, d.C, d.H, d.W, d.K, d.R, d.S, d.stride, d.pad, d.in_dtype, d.out_dtype, d.layout,
                           (int32_t)d.epilogue, d.residual ? 1 : 0};
    key->insert(key->end(), f, f + 14);
  }
}

extern "C" st_status st_plan_cache_create(int32_t capacity, const st_plan_opts* opts, st_plan_cache** out_cache) {
  if (!out_cache) return fail(ST_ERR_INVALID_ARG, "out_cache is NULL");
  *out_cache = nullptr;
  if (capacity < 1) return fail(ST_ERR_INVALID_ARG, "capacity must be at least 1");
  st_plan_cache* c = new (std::nothrow) st_plan_cache();
  if (!c) return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  std::memset(&c->opts, 0, sizeof(c->opts));
  if (opts) c->opts = *opts;
  c->capacity = capacity;
  *out_cache = c;
  return ST_OK;
}

extern "C" st_status st_plan_cache_get(st_plan_cache* cache, const st_conv_desc* descs, int32_t n_tenants, void* hip_stream,
                                       st_plan** out_plan, int32_t* out_hit) {
  if (!cache || !out_plan) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  *out_plan = nullptr;
  if (n_tenants < 0 || (n_tenants > 0 && !descs)) return fail(ST_ERR_INVALID_ARG, "descs is NULL or n_tenants negative");
  std::vector<int32_t> key;
  try {
    cache_key(descs, n_tenants, &key);
  } catch (const std::bad_alloc&) {
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  ++cache->clock;
  for (st_plan_cache::Entry& e : cache->entries) {
    if (e.key == key) {
      st_status s = st_conv_plan_rebind_all(e.plan, descs, n_tenants, hip_stream);
      if (s != ST_OK) return s;
      e.last_use = cache->clock;
      ++cache->hits;
      if (out_hit) *out_hit = 1;
      *out_plan = e.plan;
      return ST_OK;
    }
  }
  st_plan* plan = nullptr;
  st_status s = st_conv_plan(descs, n_tenants, &cache->opts, &plan);
  if (s != ST_OK) return s;
  ++cache->misses;
  if ((int)cache->entries.size() >= cache->capacity) {
    size_t victim = 0;
    for (size_t i = 1; i < cache->entries.size(); ++i)
      if (cache->entries[i].last_use < cache->entries[victim].last_use) victim = i;
    st_conv_plan_destroy(cache->entries[victim].plan);
    cache->entries.erase(cache->entries.begin() + (long)victim);
    ++cache->evictions;
  }
  try {
    st_plan_cache::Entry e;
    e.key.swap(key);
    e.plan = plan;
    e.last_use = cache->clock;
    cache->entries.push_back(std::move(e));
  } catch (const std::bad_alloc&) {
    st_conv_plan_destroy(plan);
    return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  if (out_hit) *out_hit = 0;
  *out_plan = plan;
  return ST_OK;
}

extern "C" st_status st_plan_cache_get_stats(const st_plan_cache* cache, st_plan_cache_stats* out) {
  if (!cache || !out) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  out->hits = cache->hits;
  out->misses = cache->misses;
  out->evictions = cache->evictions;
  out->size = (int32_t)cache->entries.size();
  out->capacity = cache->capacity;
  return ST_OK;
}

extern "C" void st_plan_cache_destroy(st_plan_cache* cache) {
  if (!cache) return;
  for (st_plan_cache::Entry& e : cache->entries) st_conv_plan_destroy(e.plan);
  delete cache;
}

// ---------------------------------------------------------------------------------------------------
// pipeline: several independent batches in flight
// ---------------------------------------------------------------------------------------------------
struct st_pipeline {
  std::vector<hipStream_t> streams;
  size_t next = 0;
};

extern "C" st_status st_pipeline_create(int32_t depth, st_pipeline** out_pipeline) {
  if (!out_pipeline) return fail(ST_ERR_INVALID_ARG, "out_pipeline is NULL");
  *out_pipeline = nullptr;
  if (depth < 1 || depth > 64) return fail(ST_ERR_INVALID_ARG, "depth must be between 1 and 64");
  st_pipeline* p = new (std::nothrow) st_pipeline();
  if (!p) return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  for (int32_t i = 0; i < depth; ++i) {
    hipStream_t s = nullptr;
    const hipError_t e = hipStreamCreateWithFlags(&s, hipStreamNonBlocking);     // default priority
    if (e != hipSuccess) {
      for (hipStream_t t : p->streams) (void)hipStreamDestroy(t);
      delete p;
      return hip_fail(e, "st_pipeline_create");
    }
    p->streams.push_back(s);
  }
  *out_pipeline = p;
  return ST_OK;
}

extern "C" int32_t st_pipeline_slots(int32_t depth) {
  // One launch in flight fills the planner's default; two share the chip as 256 slots each, four and more as 128 each
  // (smaller shares lose to the fixed cost per work item, larger ones to launches that queue behind one another).  us per
  // batch with 64, 128, 192, 256, 320, 400 slots, two in flight: one 3x3 layer of each of a ResNet's four stages 4.3, 3.8,
  // 4.0, 4.0, 4.0, 4.4, eight 3x3 layers 256->256 at 14x14 6.4, 6.1, 5.2, 5.5, 5.5, 6.5; four: 4.5, 4.1, 4.4, 4.3, 4.4, 5.1 and
  // 6.7, 6.5, 6.1, 6.1, 6.1, 7.1 (sixteen unlike tenants do not care).
  if (depth <= 1) return 0;
  return depth == 2 ? 256 : 128;
}

extern "C" st_status st_pipeline_next(st_pipeline* pipeline, void** out_stream) {
  if (!pipeline || !out_stream) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  *out_stream = (void*)pipeline->streams[pipeline->next];
  pipeline->next = (pipeline->next + 1) % pipeline->streams.size();
  return ST_OK;
}

extern "C" st_status st_pipeline_run(st_pipeline* pipeline, const st_plan* plan) {
  if (!pipeline) return fail(ST_ERR_INVALID_ARG, "pipeline is NULL");
  void* stream = nullptr;
  st_status s = st_pipeline_next(pipeline, &stream);
  if (s != ST_OK) return s;
  return st_conv_run(plan, stream);
}

extern "C" st_status st_pipeline_run_many(st_pipeline* pipeline, const st_plan* const* plans, int32_t n_plans, int32_t rounds) {
  if (!pipeline) return fail(ST_ERR_INVALID_ARG, "pipeline is NULL");
  if (n_plans < 0 || rounds < 0 || (n_plans > 0 && !plans)) return fail(ST_ERR_INVALID_ARG, "plans is NULL or a count is negative");
  const int64_t total = (int64_t)rounds * n_plans;
  const size_t depth = pipeline->streams.size();
  for (int32_t i = 0; i < n_plans; ++i)
    if (!plans[i]) return fail(ST_ERR_INVALID_ARG, "plans[%d] is NULL", i);
  if (n_plans > 0 && rounds > 0) {
    // launch L goes to stream (next + L) mod depth; over `rounds` rounds the pattern repeats after lcm(n_plans, depth)
    int64_t a = n_plans, b = (int64_t)depth;
    while (b) { const int64_t r = a % b; a = b; b = r; }
    const int64_t period = std::min<int64_t>(total, (int64_t)n_plans / a * (int64_t)depth);
    const size_t first0 = pipeline->next;
    st_status s = check_workspace_streams(plans, n_plans, period, [=](int64_t L) { return (first0 + (size_t)L) % depth; },
                                          "st_pipeline_run_many");
    if (s != ST_OK) return s;
  }
  const int n_threads = issue_threads(depth);
  if (total < 64 || n_threads < 2) {
    for (int32_t r = 0; r < rounds; ++r)
      for (int32_t i = 0; i < n_plans; ++i) {
        st_status s = st_pipeline_run(pipeline, plans[i]);
        if (s != ST_OK) return s;
      }
    return ST_OK;
  }
  // launch L of the sequence goes to stream (next + L) mod depth, as in the serial loop
  const size_t first = pipeline->next;
  st_status s = issue_threaded(plans, n_plans, pipeline->streams, total, n_threads,
                               [=](int64_t L) { return (first + (size_t)L) % depth; }, "st_pipeline_run_many (worker thread)");
  pipeline->next = (first + (size_t)total) % depth;
  return s;
}

extern "C" st_status st_pipeline_sync(st_pipeline* pipeline) {
  if (!pipeline) return fail(ST_ERR_INVALID_ARG, "pipeline is NULL");
  for (hipStream_t s : pipeline->streams) ST_HIP(hipStreamSynchronize(s));
  return ST_OK;
}

extern "C" void st_pipeline_destroy(st_pipeline* pipeline) {
  if (!pipeline) return;
  for (hipStream_t s : pipeline->streams) {
    (void)hipStreamSynchronize(s);
    (void)hipStreamDestroy(s);
  }
  delete pipeline;
}

extern "C" st_status st_conv_plan_info(const st_plan* plan, st_plan_info* out) {
  if (!plan || !out) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  out->n_tenants = (int32_t)plan->info.size();
  out->host_only = plan->host_only ? 1 : 0;
  out->n_items = (int64_t)plan->items_fused.size();
  out->flops = plan->flops;
  out->bytes = plan->bytes;
  out->workspace_bytes = plan->workspace_bytes;
  return ST_OK;
}

extern "C" st_status st_conv_plan_tenant_info(const st_plan* plan, int32_t tenant, st_tenant_info* out) {
  if (!plan || !out) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  if (tenant < 0 || (size_t)tenant >= plan->info.size()) return fail(ST_ERR_INVALID_ARG, "tenant index out of range");
  *out = plan->info[tenant];
  return ST_OK;
}

extern "C" st_status st_conv_plan_tenant_form(const st_plan* plan, int32_t tenant, int32_t* out_form) {
  if (!plan || !out_form) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  if (tenant < 0 || tenant >= (int32_t)plan->tenants.size()) return fail(ST_ERR_INVALID_ARG, "tenant index out of range");
  const uint32_t form = tile_code(plan->tenants[tenant]) & kFormMask;
  *out_form = form == kFormRows ? ST_FORM_ROWS : form >= kFormPieces ? ST_FORM_PIECES : form >= kFormGather ? ST_FORM_GATHERED : form >= kFormPatch ? ST_FORM_PATCH : ST_FORM_VECTORS;
  return ST_OK;
}

extern "C" st_status st_conv_plan_worklist(const st_plan* plan, int32_t which, const st_work_item** items,
                                           int64_t* n_items) {
  if (!plan || !items || !n_items) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  if (which != 0 && which != 1) return fail(ST_ERR_INVALID_ARG, "which must be 0 or 1");
  const std::vector<st_work_item>& v = which == 0 ? plan->items_fused : plan->items_tenant;
  *items = v.data();
  *n_items = (int64_t)v.size();
  return ST_OK;
}

extern "C" void st_conv_plan_destroy(st_plan* plan) {
  if (!plan) return;
  destroy_device(plan);
  delete plan;
}

extern "C" st_status st_tile_shape(int32_t index, int32_t* MT, int32_t* NT, int32_t* k_step_bytes) {
  if (index < 0 || index >= kNumTileCfgs || !MT || !NT || !k_step_bytes)
    return fail(ST_ERR_INVALID_ARG, "tile index out of range or NULL output");
  *MT = kTileShapes[index].MT;
  *NT = kTileShapes[index].NT;
  *k_step_bytes = kTileShapes[index].KB;
  return ST_OK;
}
extern "C" int32_t st_tile_count(void) { return kNumTileCfgs; }

extern "C" st_status st_maxpool_nhwc(const void* x, void* y, int32_t N, int32_t H, int32_t W, int32_t C, int32_t win,
                                     int32_t stride, int32_t pad, int32_t dtype, void* hip_stream) {
  if (!x || !y) return fail(ST_ERR_INVALID_ARG, "x and y must be non-NULL");
  if (N <= 0 || H <= 0 || W <= 0 || C <= 0 || win <= 0 || stride <= 0 || pad < 0)
    return fail(ST_ERR_INVALID_ARG, "sizes must be positive");
  if (pad >= win) return fail(ST_ERR_INVALID_ARG, "pad must be smaller than the window");
  if (H + 2 * pad < win || W + 2 * pad < win) return fail(ST_ERR_INVALID_ARG, "window larger than the padded image");
  if (dtype != ST_DT_F32 && dtype != ST_DT_BF16 && dtype != ST_DT_F16) return fail(ST_ERR_UNSUPPORTED, "unknown dtype");
  const int P = (H + 2 * pad - win) / stride + 1, Q = (W + 2 * pad - win) / stride + 1;
  if ((int64_t)N * H * W * C >= ((int64_t)1 << 31)) return fail(ST_ERR_UNSUPPORTED, "tensor too large");
  ST_HIP((hipError_t)launch_maxpool(x, y, N, H, W, C, P, Q, win, stride, pad, dtype, hip_stream));
  return ST_OK;
}

extern "C" st_status st_launch_empty(void* hip_stream) {
  ST_HIP((hipError_t)launch_empty(hip_stream));
  return ST_OK;
}

extern "C" st_status st_launch_copy(const void* src, void* dst, int64_t bytes, void* hip_stream) {
  if (!src || !dst || bytes < 0 || (bytes & 15)) return fail(ST_ERR_INVALID_ARG, "need non-NULL pointers and a multiple of 16 bytes");
  ST_HIP((hipError_t)launch_copy(src, dst, bytes, hip_stream));
  return ST_OK;
}

extern "C" const char* st_status_string(st_status s) {
  switch (s) {
    case ST_OK: return "ST_OK";
    case ST_ERR_INVALID_ARG: return "ST_ERR_INVALID_ARG";
    case ST_ERR_UNSUPPORTED: return "ST_ERR_UNSUPPORTED";
    case ST_ERR_OUT_OF_MEMORY: return "ST_ERR_OUT_OF_MEMORY";
    case ST_ERR_DEVICE: return "ST_ERR_DEVICE";
  }
  return "ST_ERR_UNKNOWN";
}
extern "C" const char* st_last_error_message(void) { return g_err; }
