// Host side of the chain (st_chain_*): validation, per-stage planning through st_conv_plan, the queue, the dependency
// thresholds, the device arena and the launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <new>
#include <vector>

#include "st_chain_deps.h"
#include "st_host.h"
#include "st_internal.h"

using namespace st;

struct st_chain {
  std::vector<st_chain_op> ops;
  std::vector<st_chain_op_info> info;        // per op, caller's order
  std::vector<TenantDev> table;              // per op, caller's order (host mirror of the device table)
  std::vector<st_work_item> items;           // the queue; item.tenant = op index
  int n_sequences = 0, n_stages = 0;
  bool host_only = false;
  uint32_t kernel_needs = 0;
  std::vector<uint32_t> stage_needs;         // one queue: of every stage's launch
  int64_t flops = 0, bytes = 0, workspace_bytes = 0;
  uint32_t ctl_slots = 0;                    // slots of one control block (kChainCtlStride words each)
  uint32_t spin_limit_ticks = 10000000u;     // 100 ms of the 100 MHz constant clock
  uint32_t flags = 0;
  int n_queues = 1;                          // 1, or kNumXCDs
  bool stage_launches = false;               // one launch per stage instead of the persistent one (one queue, unless asked for it)
  std::vector<int64_t> stage_begin;          // one queue: stage s (in order) is items[stage_begin[s] .. stage_begin[s + 1])
  // one queue: all of items.  Queues per XCD: column j of XCD x is items[colbegin[x * 2 * kChainColumns + j] ..
  // colbegin[.. + j + 1]), the kChainColumns exclusive columns first, then the shared ones
  std::vector<uint32_t> colbegin;
  uint32_t* d_colbegin = nullptr;
  std::vector<ChainPrefetch> prefetch;       // queues per XCD: XCD x's filters in stage order, [prefetch_begin[x], prefetch_begin[x + 1])
  uint32_t prefetch_begin[kNumXCDs + 1] = {};
  ChainPrefetch* d_prefetch = nullptr;
  std::vector<st_chain_dep> deps;            // queues per XCD: beside every entry of items
  ChainDep* d_deps = nullptr;
  int workgroups = 0;                        // planned size of the persistent launch (what it would be, with a launch per stage)
  int launch_workgroups = 0;                 // 0 = workgroups; else a smaller size asked for by the caller
  unsigned run_parity = 0;                   // control block the next run uses
  uint32_t run_number = 0;                   // number of the most recent run that was not captured (per-item completion flags hold it)
  // device
  char* d_arena = nullptr;
  TenantDev* d_ops = nullptr;
  st_work_item* d_items = nullptr;
  // Control blocks: [0] and [1] for ordinary runs in turn, [2] for captured ones; [3] nobody reads (what a captured run clears
  // in place of the next run's).
  uint32_t* d_ctl[kChainCtlBlocks] = {};
  char* d_counters = nullptr;                // split-K arrival counters of all sequences
  size_t counters_bytes = 0;
  uint32_t* d_item_flags = nullptr;          // one completion flag per work item (queue per XCD only)
  size_t item_flags_bytes = 0;
};

static st_status validate_pool(const st_conv_desc& d, int i) {
  if (d.N <= 0 || d.C <= 0 || d.H <= 0 || d.W <= 0 || d.R <= 0 || d.stride <= 0 || d.pad < 0)
    return fail(ST_ERR_INVALID_ARG, "op %d (max-pool): sizes must be positive, pad >= 0", i);
  if (d.R != d.S || d.K != d.C) return fail(ST_ERR_INVALID_ARG, "op %d (max-pool): needs R == S (the window) and K == C", i);
  if (d.pad >= d.R) return fail(ST_ERR_INVALID_ARG, "op %d (max-pool): pad must be smaller than the window", i);
  if (d.H + 2 * (int64_t)d.pad < d.R || d.W + 2 * (int64_t)d.pad < d.R)
    return fail(ST_ERR_INVALID_ARG, "op %d (max-pool): window larger than the padded image", i);
  if (d.in_dtype != ST_DT_F32 && d.in_dtype != ST_DT_BF16 && d.in_dtype != ST_DT_F16)
    return fail(ST_ERR_UNSUPPORTED, "op %d (max-pool): unknown dtype", i);
  if (d.out_dtype != d.in_dtype) return fail(ST_ERR_UNSUPPORTED, "op %d (max-pool): out_dtype must equal in_dtype", i);
  if (d.layout != ST_LAYOUT_NHWC_KRSC) return fail(ST_ERR_UNSUPPORTED, "op %d (max-pool): tensors must be NHWC", i);
  if (d.C % (16 / elem_size(d.in_dtype)) != 0)
    return fail(ST_ERR_UNSUPPORTED, "op %d (max-pool): C must be a multiple of %d", i, 16 / elem_size(d.in_dtype));
  if (!d.x || !d.y || d.x == d.y) return fail(ST_ERR_INVALID_ARG, "op %d (max-pool): x and y must be non-NULL and distinct", i);
  if (d.epilogue != 0 || d.reserved != 0) return fail(ST_ERR_INVALID_ARG, "op %d (max-pool): epilogue and reserved must be 0", i);
  const int64_t P = (d.H + 2 * (int64_t)d.pad - d.R) / d.stride + 1, Q = (d.W + 2 * (int64_t)d.pad - d.R) / d.stride + 1;
  const int64_t es = elem_size(d.in_dtype);
  if ((int64_t)d.N * d.H * d.W * d.C * es >= ((int64_t)1 << 31) || (int64_t)d.N * P * Q * d.C * es >= ((int64_t)1 << 31))
    return fail(ST_ERR_UNSUPPORTED, "op %d (max-pool): tensors must stay below 2^31 bytes", i);
  return ST_OK;
}

static constexpr double kPoolItemClocks = 8000.0;      // a max-pool work item, 3.4 us in place
static constexpr double kBoundaryClocks = 3000.0;      // last store of a tile to the first load of one that waited for it

static uint32_t flag_of(const TenantDev& T, const st_work_item& it) {
  return T.chain_flag_base + (it.tile_m * (uint32_t)T.tiles_n + it.tile_n) * (uint32_t)T.split_k + it.k_split_idx;
}

// Ops that wait tile by tile rely on "a stage complete" meaning "the stage before it complete" (st_chain_deps.cpp): a
// sequence's ops of a stage keep their local ranges (by tile index; none: the op waits for all of the previous stage) if one
// of them waits for the whole previous stage anyway or the ranges together hold every flag of it.
typedef std::vector<std::vector<ChainDep>> LocalRanges;
static void require_coverage(const std::vector<int>& stage_ops, const st_chain_op* ops, const std::vector<int64_t>& prev_begin,
                             const std::vector<int64_t>& prev_count, LocalRanges* local) {
  std::map<int, std::vector<int>> by_seq;
  for (int i : stage_ops) by_seq[ops[i].sequence].push_back(i);
  for (const auto& kv : by_seq) {
    const int q = kv.first;
    if (std::any_of(kv.second.begin(), kv.second.end(), [&](int i) { return (*local)[i].empty(); })) continue;
    std::vector<int> steps((size_t)prev_count[q] + 1, 0);       // +1 where a range begins, -1 behind its end
    for (int i : kv.second)
      for (const ChainDep& d : (*local)[i]) {
        ++steps[(size_t)(d.begin - prev_begin[q])];
        --steps[(size_t)(d.begin - prev_begin[q]) + d.count];
      }
    bool all = true;
    int depth = 0;
    for (int64_t k = 0; k < prev_count[q]; ++k) {
      depth += steps[(size_t)k];
      all = all && depth > 0;
    }
    if (!all)
      for (int i : kv.second) (*local)[i].clear();
  }
}

static void prev_ops_next(const std::vector<int>& stage_ops, const st_chain_op* ops, int q, int64_t items, std::vector<int>* prev) {
  if (items == 0) return;
  prev->clear();
  for (int i : stage_ops)
    if (ops[i].sequence == q) prev->push_back(i);
}

// Deals one XCD's entries of a stage (of the ops mine) to its columns.  A stage that starts when the one before has ended:
// longest entries first, to the columns in turn, exclusive ones first and shared ones only beyond one per compute unit, so that
// a stage of no more entries than compute units never shares one.  A stage whose entries wait tile by tile: in the order of
// their place in the output, each to the column where the model has it end first, so that what the next stage reads comes
// in order and a compute unit that the stage before left idle goes on at once.
static void deal(const std::vector<TenantDev>& table, const std::vector<int>& mine, const LocalRanges& local, const std::vector<double>& cost,
                 const std::vector<st_work_item>& longest_first, std::vector<double>* flag_end, ChainDealer* dealer, std::vector<st_work_item>* columns) {
  const bool by_tile = std::all_of(mine.begin(), mine.end(), [&](int i) { return !local[i].empty(); });
  auto last_end = [&](uint32_t begin, uint32_t count) {
    double t = 0.0;
    for (uint32_t f = begin; f < begin + count; ++f) t = std::max(t, (*flag_end)[f]);
    return t;
  };
  std::vector<double> gate_open(mine.size());
  for (size_t o = 0; o < mine.size(); ++o) gate_open[o] = last_end(table[mine[o]].chain_dep_begin, table[mine[o]].chain_dep_count) + kBoundaryClocks;
  size_t k = 0;
  auto put = [&](const st_work_item& it, double ready) {
    const double c = cost[it.tenant];
    const size_t col = by_tile ? dealer->earliest(ready, c) : k % dealer->columns();
    dealer->place(col, ready, c);
    (*flag_end)[flag_of(table[it.tenant], it)] = dealer->ends(col);
    columns[col].push_back(it);
    ++k;
  };
  if (!by_tile && mine.size() != 1) {
    std::map<int, double> open;
    for (size_t o = 0; o < mine.size(); ++o) open[mine[o]] = gate_open[o];
    for (const st_work_item& it : longest_first) put(it, open[it.tenant]);
    return;
  }
  std::vector<int> next(mine.size(), 0);       // next tile index of every op; the op that is furthest behind goes on
  for (;;) {
    size_t o = mine.size();
    double least = 2.0;
    for (size_t j = 0; j < mine.size(); ++j) {
      const double at = (double)next[j] / table[mine[j]].tiles_m;
      if (next[j] < table[mine[j]].tiles_m && at < least) { least = at; o = j; }
    }
    if (o == mine.size()) break;
    const TenantDev& T = table[mine[o]];
    const int m = next[o]++;
    double ready = gate_open[o];
    if (by_tile) ready = std::max(ready, last_end(local[mine[o]][m].begin, local[mine[o]][m].count) + kBoundaryClocks);
    for (int n = 0; n < T.tiles_n; ++n)
      for (int slice = 0; slice < T.split_k; ++slice) {
        st_work_item it;
        it.tenant = (uint16_t)mine[o];
        it.k_split_idx = (uint16_t)slice;
        it.tile_m = (uint32_t)m;
        it.tile_n = (uint32_t)n;
        it.reserved = 0;
        put(it, ready);
      }
  }
}

static void destroy_chain(st_chain* c) {
  if (!c) return;
  if (c->d_arena) (void)hipFree(c->d_arena);
  delete c;
}

extern "C" st_status st_chain_plan(const st_chain_op* ops, int32_t n_ops, const st_plan_opts* opts, st_chain** out_chain) {
  if (!out_chain) return fail(ST_ERR_INVALID_ARG, "out_chain is NULL");
  *out_chain = nullptr;
  if (n_ops < 0 || (n_ops > 0 && !ops)) return fail(ST_ERR_INVALID_ARG, "ops is NULL or n_ops negative");
  if (n_ops > 65535) return fail(ST_ERR_UNSUPPORTED, "at most 65535 ops per chain");
  st_plan_opts o;
  std::memset(&o, 0, sizeof(o));
  if (opts) o = *opts;
  const bool host_only = o.host_only != 0;
  const int want_queues = o.chain_queues;
  if (want_queues < 0 || want_queues > 2) return fail(ST_ERR_INVALID_ARG, "opts.chain_queues must be 0, 1 or 2");
  o.host_only = 1;          // the stages are planned on the host; the chain owns the one device arena
  o.order = 0;
  o.chain_queues = 0;
  int max_seq = -1;
  for (int i = 0; i < n_ops; ++i) {
    const st_chain_op& op = ops[i];
    if (op.kind != ST_OP_CONV && op.kind != ST_OP_MAXPOOL) return fail(ST_ERR_INVALID_ARG, "op %d: unknown kind %d", i, op.kind);
    if (op.sequence < 0 || op.sequence >= 4096) return fail(ST_ERR_INVALID_ARG, "op %d: sequence must be in [0, 4096)", i);
    if (op.stage < 0) return fail(ST_ERR_INVALID_ARG, "op %d: stage must be >= 0", i);
    if (op.reserved != 0) return fail(ST_ERR_INVALID_ARG, "op %d: reserved must be 0", i);
    if (op.kind == ST_OP_MAXPOOL) {
      st_status s = validate_pool(op.conv, i);
      if (s != ST_OK) return s;
    }
    max_seq = std::max(max_seq, op.sequence);
  }
  st_chain* c = new (std::nothrow) st_chain();
  if (!c) return fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  st_status status = ST_OK;
  std::vector<st_plan*> stage_plans;
  try {
    c->host_only = host_only;
    c->ops.assign(ops, ops + n_ops);
    c->info.resize(n_ops);
    c->table.resize(n_ops);
    c->n_sequences = max_seq + 1;
    // The work is laid out per XCD when every XCD gets at least one sequence (and the device is a whole 8-XCD one);
    // else there is one queue for the chip.  A host-only chain is laid out for a whole device.
    int max_wg = 2 * kNumCUs, n_xcd = kNumXCDs;
    if (!host_only && n_ops > 0) {
      const hipError_t e = (hipError_t)chain_max_workgroups(&max_wg, &n_xcd);
      if (e != hipSuccess) { delete c; return hip_fail(e, "occupancy query (chain kernel)"); }
    }
    if (want_queues == 2 && n_xcd != kNumXCDs) {
      delete c;
      return fail(ST_ERR_UNSUPPORTED, "the per-XCD layout needs a device with %d XCDs, this one shows %d", kNumXCDs, n_xcd);
    }
    c->n_queues = (want_queues == 2 || (want_queues == 0 && n_xcd == kNumXCDs && c->n_sequences >= kNumXCDs)) ? kNumXCDs : 1;
    // With one queue a pass is a launch per stage, unless the caller asked for the persistent one: entries claimed one by
    // one and completions counted at the memory side cost more than the launches (4 networks of batch 4: 879 us as one
    // launch, 524 as 50; one network of batch 8: 969 and 359; 7 of batch 1: 617 and 436).
    c->stage_launches = c->n_queues == 1 && want_queues == 0;
    // per XCD: producer and consumer of a sequence share that XCD's L2, and completion travels through it
    c->flags = c->n_queues > 1 ? kChainFlagLocalFlags : 0u;
    // The shared columns are only used when a compute unit holds two workgroups (the per-XCD layout exists on a whole
    // device only: kNumCUs compute units, max_wg / kNumCUs workgroups on each).
    const bool two_per_cu = max_wg / kNumCUs >= 2;
    const int n_sub = c->n_queues > 1 ? kNumXCDs * 2 * kChainColumns : 1;      // columns, or the one queue
    std::vector<std::vector<st_work_item>> queues((size_t)n_sub);
    std::map<int, std::vector<int>> by_stage;          // stage -> op indices, caller's order
    for (int i = 0; i < n_ops; ++i) by_stage[ops[i].stage].push_back(i);
    c->n_stages = (int)by_stage.size();
    std::vector<int64_t> done((size_t)c->n_sequences, 0);          // work items of each sequence in earlier stages
    // completion flags: one per work item; a sequence's items of one stage are contiguous, op after op
    int64_t flag_total = 0;
    std::vector<int64_t> prev_begin((size_t)c->n_sequences, 0), prev_count((size_t)c->n_sequences, 0);
    // ... and of the stage before that one: what a stage's filters wait for before they are prefetched
    std::vector<int64_t> prev2_begin((size_t)c->n_sequences, 0), prev2_count((size_t)c->n_sequences, 0);
    std::vector<ChainPrefetch> ahead[kNumXCDs];
    // queues per XCD: the ops of the sequence's previous stage, what of it every tile of an op reads, the modelled
    // clocks of an op's items, and when every work item of the stages so far ends (by flag) and every column
    std::vector<std::vector<int>> prev_ops((size_t)c->n_sequences);
    LocalRanges local((size_t)n_ops);
    std::vector<double> cost((size_t)n_ops, kPoolItemClocks), flag_end;
    std::vector<ChainDealer> dealers((size_t)kNumXCDs, ChainDealer(two_per_cu));
    // split-K workspace of a sequence: the largest need of any of its stages (its stages never overlap in time)
    std::vector<int64_t> seq_ws((size_t)c->n_sequences, 0), seq_ct((size_t)c->n_sequences, 0);
    struct Use { int op; int64_t ws_off, ct_off; };
    std::vector<Use> uses;
    for (auto& kv : by_stage) {
      std::vector<int> conv_ops, pool_ops;
      for (int i : kv.second) (ops[i].kind == ST_OP_CONV ? conv_ops : pool_ops).push_back(i);
      std::vector<st_conv_desc> descs;
      for (int i : conv_ops) descs.push_back(ops[i].conv);
      st_plan* sp = nullptr;
      status = st_conv_plan(descs.data(), (int32_t)descs.size(), &o, &sp);
      if (status != ST_OK) break;
      stage_plans.push_back(sp);
      std::vector<int64_t> stage_items((size_t)c->n_sequences, 0), stage_ws((size_t)c->n_sequences, 0), stage_ct((size_t)c->n_sequences, 0);
      for (size_t j = 0; j < conv_ops.size(); ++j) {
        const int i = conv_ops[j];
        const int q = ops[i].sequence;
        st_chain_op_info& inf = c->info[i];
        std::memset(&inf, 0, sizeof(inf));
        inf.sequence = q; inf.stage = ops[i].stage; inf.kind = ST_OP_CONV;
        inf.need = (uint32_t)done[q];
        inf.tile = sp->info[j];
        inf.item_count = sp->info[j].item_count;
        TenantDev T = sp->tenants[j];
        T.chain_seq = q;
        T.chain_need = (uint32_t)done[q];
        c->table[i] = T;
        cost[i] = sp->item_time[j];
        if (sp->info[j].split_k > 1) {
          const st_tenant_info& ti = sp->info[j];
          uses.push_back({i, stage_ws[q], stage_ct[q]});
          stage_ws[q] += (int64_t)ti.tiles_m * ti.tiles_n * ti.split_k * ti.MT * ti.NT;
          stage_ct[q] += (int64_t)ti.tiles_m * ti.tiles_n;
        }
        stage_items[q] += sp->info[j].item_count;
        c->flops += sp->info[j].flops;
        c->bytes += sp->info[j].bytes;
      }
      // queue: the stage's convolution items in the fused order (longest first), then its max-pool items
      std::vector<std::vector<st_work_item>> stage_q((size_t)c->n_queues);
      for (const st_work_item& it : sp->items_fused) {
        st_work_item g = it;
        g.tenant = (uint16_t)conv_ops[it.tenant];
        stage_q[(size_t)(ops[g.tenant].sequence % c->n_queues)].push_back(g);
      }
      for (int i : pool_ops) {
        const st_conv_desc& d = ops[i].conv;
        const int q = ops[i].sequence;
        const int es = elem_size(d.in_dtype), vec = 16 / es;
        const int P = (d.H + 2 * d.pad - d.R) / d.stride + 1, Q = (d.W + 2 * d.pad - d.R) / d.stride + 1;
        const int64_t total = (int64_t)d.N * P * Q * (d.C / vec);
        const int64_t n_it = (total + kThreads - 1) / kThreads;
        st_chain_op_info& inf = c->info[i];
        std::memset(&inf, 0, sizeof(inf));
        inf.sequence = q; inf.stage = ops[i].stage; inf.kind = ST_OP_MAXPOOL;
        inf.need = (uint32_t)done[q];
        inf.item_count = n_it;
        inf.tile.P = P; inf.tile.Q = Q;
        TenantDev T;
        std::memset(&T, 0, sizeof(T));
        T.x = d.x; T.y = d.y;
        T.C = d.C; T.H = d.H; T.W = d.W; T.K = d.C; T.R = d.R; T.S = d.R; T.stride = d.stride; T.pad = d.pad;
        T.P = P; T.Q = Q; T.PQ = P * Q; T.M = (int32_t)total;
        T.in_dtype = d.in_dtype; T.out_dtype = d.in_dtype;
        T.cfg = kChainPoolCfg; T.split_k = 1;
        T.tiles_m = (int32_t)n_it; T.tiles_n = 1;
        T.x_bytes = (uint32_t)((int64_t)d.N * d.H * d.W * d.C * es);
        T.y_bytes = (uint32_t)((int64_t)d.N * P * Q * d.C * es);
        T.chain_seq = q;
        T.chain_need = (uint32_t)done[q];
        c->table[i] = T;
        for (int64_t k = 0; k < n_it; ++k) {
          st_work_item g;
          g.tenant = (uint16_t)i; g.k_split_idx = 0; g.tile_m = (uint32_t)k; g.tile_n = 0; g.reserved = 0;
          stage_q[(size_t)(q % c->n_queues)].push_back(g);
        }
        stage_items[q] += n_it;
      }
      uint32_t needs = 0u;
      for (int i : kv.second) needs |= kernel_needs(c->table[i]);
      c->kernel_needs |= needs;
      c->stage_needs.push_back(needs);
      if (c->n_queues == 1) c->stage_begin.push_back((int64_t)queues[0].size());
      std::vector<int64_t> cursor((size_t)c->n_sequences, 0), stage_begin((size_t)c->n_sequences, 0);
      for (int q = 0; q < c->n_sequences; ++q) {
        cursor[q] = stage_begin[q] = flag_total;
        flag_total += stage_items[q];
      }
      for (int i : kv.second) {
        const int q = ops[i].sequence;
        TenantDev& T = c->table[i];
        T.chain_flag_base = (uint32_t)cursor[q];
        cursor[q] += c->info[i].item_count;
        T.chain_dep_begin = (uint32_t)prev_begin[q];
        T.chain_dep_count = (uint32_t)prev_count[q];
        if (c->n_queues > 1 && prev_count[q] > 0) {
          // waits tile by tile, if it reads exactly one op of the previous stage and nothing else of the two can collide
          int src = -1, readers = 0;
          bool apart = true;
          for (int j : prev_ops[q]) {
            apart = apart && chain_ops_disjoint(T, c->table[j]);
            if (chain_reads(T, c->table[j])) { ++readers; src = j; }
          }
          if (apart && readers == 1 && chain_reads_exactly(T, c->table[src])) {
            local[i].reserve((size_t)T.tiles_m);
            for (int m = 0; m < T.tiles_m; ++m) local[i].push_back(chain_local_range(T, c->table[src], m));
          }
        }
        if (ops[i].kind == ST_OP_CONV)
          ahead[q % kNumXCDs].push_back({(uint32_t)i, T.chain_flag_base, (uint32_t)prev2_begin[q], (uint32_t)prev2_count[q]});
      }
      if (c->n_queues > 1) {
        require_coverage(kv.second, ops, prev_begin, prev_count, &local);
        for (int i : kv.second) {
          if (local[i].empty()) continue;
          c->table[i].chain_dep_begin = (uint32_t)prev2_begin[ops[i].sequence];
          c->table[i].chain_dep_count = (uint32_t)prev2_count[ops[i].sequence];
        }
      }
      flag_end.resize((size_t)flag_total, 0.0);
      for (int x = 0; x < c->n_queues; ++x) {
        if (c->n_queues == 1) {
          queues[0].insert(queues[0].end(), stage_q[0].begin(), stage_q[0].end());
          continue;
        }
        std::vector<int> mine;
        for (int i : kv.second)
          if (ops[i].sequence % c->n_queues == x) mine.push_back(i);
        deal(c->table, mine, local, cost, stage_q[(size_t)x], &flag_end, &dealers[(size_t)x], queues.data() + (size_t)x * 2 * kChainColumns);
      }
      for (int q = 0; q < c->n_sequences; ++q) prev_ops_next(kv.second, ops, q, stage_items[q], &prev_ops[q]);
      for (int q = 0; q < c->n_sequences; ++q) {
        if (stage_items[q] > 0) {
          prev2_begin[q] = prev_begin[q]; prev2_count[q] = prev_count[q];
          prev_begin[q] = stage_begin[q]; prev_count[q] = stage_items[q];
        }
        done[q] += stage_items[q];
        seq_ws[q] = std::max(seq_ws[q], stage_ws[q]);
        seq_ct[q] = std::max(seq_ct[q], stage_ct[q]);
      }
    }
    if (c->n_queues == 1) c->stage_begin.push_back((int64_t)queues[0].size());
    if (status == ST_OK) {
      int64_t total_items = 0;
      for (const auto& qv : queues) total_items += (int64_t)qv.size();
      if (total_items >= ((int64_t)1 << 31)) status = fail(ST_ERR_UNSUPPORTED, "more than 2^31 work items");
    }
    if (status == ST_OK) {
      if (c->n_queues > 1) c->colbegin.assign((size_t)n_sub + 1, 0u);
      for (int qi = 0; qi < n_sub; ++qi) {
        if (c->n_queues > 1) c->colbegin[(size_t)qi] = (uint32_t)c->items.size();
        c->items.insert(c->items.end(), queues[(size_t)qi].begin(), queues[(size_t)qi].end());
      }
      if (c->n_queues > 1) {
        c->colbegin[(size_t)n_sub] = (uint32_t)c->items.size();
        for (int x = 0; x < kNumXCDs; ++x) {
          c->prefetch_begin[x] = (uint32_t)c->prefetch.size();
          c->prefetch.insert(c->prefetch.end(), ahead[x].begin(), ahead[x].end());
        }
        c->prefetch_begin[kNumXCDs] = (uint32_t)c->prefetch.size();
        c->deps.reserve(c->items.size());
        for (const st_work_item& it : c->items) {
          const TenantDev& T = c->table[it.tenant];
          const ChainDep d = local[it.tenant].empty() ? ChainDep{0u, 0u} : local[it.tenant][it.tile_m];
          const bool waits = T.chain_need != 0u;
          c->deps.push_back({flag_of(T, it), waits ? T.chain_dep_begin : 0u, waits ? T.chain_dep_count : 0u, d.begin, d.count});
        }
      }
    }
    if (status == ST_OK) {
      // arena: [op table][queue][control blocks, persistent launch only][split-K counters][completion flags][column boundaries][prefetch list][entries' dependencies][split-K partial tiles]
      auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
      c->ctl_slots = (uint32_t)(kChainCtlSeq + c->n_sequences);
      int64_t ws_total = 0, ct_total = 0;
      std::vector<int64_t> ws_base((size_t)c->n_sequences, 0), ct_base((size_t)c->n_sequences, 0);
      for (int q = 0; q < c->n_sequences; ++q) {
        ws_base[q] = ws_total; ct_base[q] = ct_total;
        ws_total += seq_ws[q]; ct_total += seq_ct[q];
      }
      c->workspace_bytes = ws_total * 4 + ct_total * 4;
      const size_t off_items = up((size_t)n_ops * sizeof(TenantDev));
      const size_t off_ctl = off_items + up(c->items.size() * sizeof(st_work_item));
      const size_t ctl_words = c->stage_launches ? 0 : (size_t)c->ctl_slots * kChainCtlStride + kChainRankWords;   // one control block
      const size_t off_ct = off_ctl + up(ctl_words * 4 * kChainCtlBlocks);
      const size_t off_flags = off_ct + up((size_t)ct_total * 4);
      const size_t off_cols = off_flags + up(c->n_queues > 1 ? c->items.size() * 4 : 0);
      const size_t off_pf = off_cols + up(c->colbegin.size() * 4);
      const size_t off_deps = off_pf + up(c->prefetch.size() * sizeof(ChainPrefetch));
      const size_t off_ws = off_deps + up(c->deps.size() * sizeof(ChainDep));
      const size_t total = off_ws + (size_t)ws_total * 4;
      if (!host_only && n_ops > 0) {
        hipError_t e = hipMalloc((void**)&c->d_arena, total);
        if (e != hipSuccess) status = hip_fail(e, "hipMalloc (chain arena)");
        if (status == ST_OK) {
          for (const Use& u : uses) {
            const int q = ops[u.op].sequence;
            c->table[u.op].ws = (float*)(c->d_arena + off_ws) + ws_base[q] + u.ws_off;
            c->table[u.op].counters = (uint32_t*)(c->d_arena + off_ct) + ct_base[q] + u.ct_off;
          }
          std::vector<char> host(off_ws, 0);
          std::memcpy(host.data(), c->table.data(), (size_t)n_ops * sizeof(TenantDev));
          coded_items(c->table, c->items, (st_work_item*)(host.data() + off_items));
          if (!c->colbegin.empty()) std::memcpy(host.data() + off_cols, c->colbegin.data(), c->colbegin.size() * 4);
          if (!c->prefetch.empty()) std::memcpy(host.data() + off_pf, c->prefetch.data(), c->prefetch.size() * sizeof(ChainPrefetch));
          for (size_t k = 0; k < c->deps.size(); ++k) ((ChainDep*)(host.data() + off_deps))[k] = {c->deps[k].tiles_begin, c->deps[k].tiles_count};
          e = hipMemcpy(c->d_arena, host.data(), off_ws, hipMemcpyHostToDevice);
          if (e != hipSuccess) status = hip_fail(e, "hipMemcpy (chain tables)");
          c->d_ops = (TenantDev*)c->d_arena;
          c->d_items = (st_work_item*)(c->d_arena + off_items);
          if (!c->stage_launches) {
            for (int b = 0; b < kChainCtlBlocks; ++b) c->d_ctl[b] = (uint32_t*)(c->d_arena + off_ctl) + (size_t)b * ctl_words;
          }
          c->d_counters = c->d_arena + off_ct;
          c->counters_bytes = (size_t)ct_total * 4;
          if (c->n_queues > 1) {
            c->d_item_flags = (uint32_t*)(c->d_arena + off_flags);
            c->item_flags_bytes = c->items.size() * 4;
            c->d_colbegin = (uint32_t*)(c->d_arena + off_cols);
            c->d_prefetch = (ChainPrefetch*)(c->d_arena + off_pf);
            c->d_deps = (ChainDep*)(c->d_arena + off_deps);
          }
        }
      }
      // one queue: no more workgroups than entries; queues per XCD: every resident slot (a workgroup for which no column
      // is left goes home at once)
      c->workgroups = c->n_queues > 1 ? max_wg : (int)std::min<int64_t>((int64_t)c->items.size(), max_wg);
    }
  } catch (const std::bad_alloc&) {
    status = fail(ST_ERR_OUT_OF_MEMORY, "host allocation failed");
  }
  for (st_plan* sp : stage_plans) st_conv_plan_destroy(sp);
  if (status != ST_OK) {
    destroy_chain(c);
    return status;
  }
  *out_chain = c;
  return ST_OK;
}

// Whether what is queued on the stream goes into a graph.  (The default stream cannot be captured; asking about it fails while
// another one is.)
static bool capturing(void* stream) {
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  if (!stream) return false;
  if (hipStreamIsCapturing((hipStream_t)stream, &status) != hipSuccess) {
    (void)hipGetLastError();          // the launch says what is wrong with the stream
    return false;
  }
  return status != hipStreamCaptureStatusNone;
}

static st_status chain_launch(st_chain* c, void* stream, uint64_t* prof_dev) {
  if (!c) return fail(ST_ERR_INVALID_ARG, "chain is NULL");
  if (c->host_only) return fail(ST_ERR_UNSUPPORTED, "chain was built host-only and cannot run");
  if (c->items.empty()) return ST_OK;
  if (c->stage_launches) {
    for (size_t g = 0; g + 1 < c->stage_begin.size(); ++g) {
      const int64_t b = c->stage_begin[g], n = c->stage_begin[g + 1] - b;
      ST_HIP((hipError_t)launch_conv(c->stage_needs[g], c->d_ops, c->d_items + b, n, stream, prof_dev ? prof_dev + b * kProfSlots : nullptr));
    }
    return ST_OK;
  }
  auto launch = [&](uint32_t* ctl, uint32_t* ctl_other, uint32_t run_number) {
    return (hipError_t)launch_chain(c->kernel_needs, c->d_ops, c->d_items, (uint32_t)c->items.size(), c->d_colbegin, c->d_deps, (uint32_t)c->n_queues, c->d_prefetch, c->prefetch_begin, ctl,
                                    ctl_other, c->ctl_slots, c->d_item_flags, run_number, c->spin_limit_ticks, c->flags,
                                    c->launch_workgroups > 0 ? c->launch_workgroups : c->workgroups, stream, prof_dev);
  };
  if (capturing(stream)) {
    // A graph replays the launch with these arguments, any number of times and between other runs: a control block and a run
    // number that no other run uses, made new by a launch ahead of it, and nothing of the host's numbering moves.
    ST_HIP((hipError_t)launch_chain_reset(c->d_ctl[2], c->ctl_slots, c->d_item_flags, (uint32_t)(c->item_flags_bytes / 4), stream));
    ST_HIP(launch(c->d_ctl[2], c->d_ctl[3], kChainCapturedRun));
    return ST_OK;
  }
  const unsigned p = c->run_parity;
  if (++c->run_number == kChainCapturedRun) {
    // the run numbers have wrapped: forget every flag of the old numbering
    if (c->d_item_flags) ST_HIP((hipError_t)launch_zero(c->d_item_flags, (int64_t)((c->item_flags_bytes + 15) & ~(size_t)15), stream));
    c->run_number = 1u;
  }
  ST_HIP(launch(c->d_ctl[p], c->d_ctl[p ^ 1u], c->run_number));
  c->run_parity = p ^ 1u;
  return ST_OK;
}

extern "C" st_status st_chain_run(st_chain* chain, void* hip_stream) { return chain_launch(chain, hip_stream, nullptr); }

extern "C" st_status st_chain_run_profiled(st_chain* chain, void* hip_stream, uint64_t* stamps, int64_t capacity) {
  if (!chain) return fail(ST_ERR_INVALID_ARG, "chain is NULL");
  const int64_t n = (int64_t)chain->items.size();
  if (!stamps || capacity < n * kProfSlots) return fail(ST_ERR_INVALID_ARG, "stamps buffer too small: need %lld entries", (long long)(n * kProfSlots));
  if (chain->host_only) return fail(ST_ERR_UNSUPPORTED, "chain was built host-only and cannot run");
  if (n == 0) return ST_OK;
  uint64_t* d = nullptr;
  ST_HIP(hipMalloc((void**)&d, (size_t)n * kProfSlots * 8));
  hipError_t e = (hipError_t)launch_zero(d, n * kProfSlots * 8, hip_stream);
  st_status s = ST_OK;
  if (e == hipSuccess) s = chain_launch(chain, hip_stream, d);
  if (e == hipSuccess && s == ST_OK) e = hipStreamSynchronize((hipStream_t)hip_stream);
  if (e == hipSuccess && s == ST_OK) e = hipMemcpy(stamps, d, (size_t)n * kProfSlots * 8, hipMemcpyDeviceToHost);
  (void)hipFree(d);
  if (s != ST_OK) return s;
  if (e != hipSuccess) return hip_fail(e, "st_chain_run_profiled");
  return ST_OK;
}

extern "C" st_status st_chain_aborted(st_chain* chain, int32_t* aborted) {
  if (!chain || !aborted) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  *aborted = 0;
  if (chain->host_only || chain->items.empty()) return ST_OK;
  ST_HIP(hipDeviceSynchronize());
  if (chain->stage_launches) return ST_OK;           // nothing waits inside a launch, nothing can give up
  bool lost = false;
  for (int b = 0; b < 3; ++b) {
    const uint32_t* ctl = chain->d_ctl[b];
    uint32_t words[kChainCtlHead * kChainCtlStride];
    ST_HIP(hipMemcpy(words, ctl, sizeof(words), hipMemcpyDeviceToHost));
    // (the counts wrap at 2^32, all alike)
    lost = lost || words[kChainCtlLost * kChainCtlStride] != 0u ||
           words[kChainCtlDone * kChainCtlStride] != words[kChainCtlStarted * kChainCtlStride] * (uint32_t)chain->items.size();
  }
  if (lost) {
    // an abandoned pass has left its queue head, its sequence counters and some split-K arrival counters anywhere
    ST_HIP(hipMemset(chain->d_ctl[0], 0, ((size_t)chain->ctl_slots * kChainCtlStride + kChainRankWords) * 4 * kChainCtlBlocks));
    if (chain->counters_bytes) ST_HIP(hipMemset(chain->d_counters, 0, chain->counters_bytes));
    ST_HIP(hipDeviceSynchronize());                  // before a run on a stream that does not wait for this one
    *aborted = 1;
  }
  return ST_OK;
}

extern "C" st_status st_chain_set_wait_limit_us(st_chain* chain, int64_t microseconds) {
  if (!chain) return fail(ST_ERR_INVALID_ARG, "chain is NULL");
  if (microseconds < 0 || microseconds > 40000000) return fail(ST_ERR_INVALID_ARG, "limit must be between 0 and 40 s");
  chain->spin_limit_ticks = (uint32_t)(microseconds * 100);
  return ST_OK;
}

extern "C" st_status st_chain_set_workgroups(st_chain* chain, int32_t workgroups) {
  if (!chain) return fail(ST_ERR_INVALID_ARG, "chain is NULL");
  if (workgroups < 0 || workgroups > chain->workgroups) return fail(ST_ERR_INVALID_ARG, "workgroups must be between 0 and %d", chain->workgroups);
  chain->launch_workgroups = workgroups;
  return ST_OK;
}

extern "C" st_status st_chain_get_info(const st_chain* chain, st_chain_info* out) {
  if (!chain || !out) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  std::memset(out, 0, sizeof(*out));
  out->n_ops = (int32_t)chain->ops.size();
  out->n_sequences = chain->n_sequences;
  out->n_stages = chain->n_stages;
  out->workgroups = chain->workgroups;
  out->n_items = (int64_t)chain->items.size();
  out->flops = chain->flops;
  out->bytes = chain->bytes;
  out->workspace_bytes = chain->workspace_bytes;
  out->host_only = chain->host_only ? 1 : 0;
  out->n_queues = chain->n_queues;
  const int64_t n = (int64_t)chain->items.size();
  for (int q = 0; q <= kNumXCDs; ++q)
    out->queue_begin[q] = chain->n_queues > 1 ? chain->colbegin[(size_t)q * 2 * kChainColumns] : (q == 0 ? 0 : n);
  for (int q = 0; q < kNumXCDs; ++q)
    out->shared_begin[q] = chain->n_queues > 1 ? chain->colbegin[(size_t)q * 2 * kChainColumns + kChainColumns] : out->queue_begin[q + 1];
  out->columns = chain->n_queues > 1 ? kChainColumns : 0;
  return ST_OK;
}

extern "C" st_status st_chain_get_op_info(const st_chain* chain, int32_t op, st_chain_op_info* out) {
  if (!chain || !out) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  if (op < 0 || (size_t)op >= chain->info.size()) return fail(ST_ERR_INVALID_ARG, "op index out of range");
  *out = chain->info[op];
  return ST_OK;
}

extern "C" st_status st_chain_worklist(const st_chain* chain, const st_work_item** items, int64_t* n_items) {
  if (!chain || !items || !n_items) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  *items = chain->items.data();
  *n_items = (int64_t)chain->items.size();
  return ST_OK;
}

extern "C" st_status st_chain_columns(const st_chain* chain, const uint32_t** begins, int64_t* n) {
  if (!chain || !begins || !n) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  *begins = chain->colbegin.empty() ? nullptr : chain->colbegin.data();
  *n = (int64_t)chain->colbegin.size();
  return ST_OK;
}

extern "C" st_status st_chain_dependencies(const st_chain* chain, const st_chain_dep** deps, int64_t* n) {
  if (!chain || !deps || !n) return fail(ST_ERR_INVALID_ARG, "NULL argument");
  *deps = chain->deps.empty() ? nullptr : chain->deps.data();
  *n = (int64_t)chain->deps.size();
  return ST_OK;
}

extern "C" void st_chain_destroy(st_chain* chain) { destroy_chain(chain); }
