"""The work that users of the fused multi-tenant convolution library have it do, as cases to time.

A case is one of four kinds:

  launch    one fused launch over a set of tenants' layers through a plan made beforehand (st_conv_run);
  arrival   a short trace of steps whose set of ready tenants changes from step to step, each set met twice, on other
            buffers the second time; a step is a plan-cache lookup and its launch (st_plan_cache_get, st_conv_run);
  pipeline  several independent batches in flight, each a fused launch on the next stream of a ring (st_pipeline_*);
  stack     a pass of every tenant through a 53-layer ResNet-50-shaped network (stack.ResNetStack), either as one
            persistent launch ("chain") or as one fused launch per layer group ("layers").

Inputs are U(-1, 1) and weights N(0, gain / fan_in), as in paper_1901_00041_amd/synth.py; they are made on the GPU from
the seed.  Everything runs on the caller's current stream, except the pipeline, which owns its streams.
"""
import random

import torch

from paper_1901_00041_amd import st_conv as sc
from paper_1901_00041_amd import synth
from paper_1901_00041_amd.stack import ResNetStack
from paper_1901_00041_amd.synth import ConvShape

DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
ES = {"f32": 4, "bf16": 2, "f16": 2}
LADDER = ((64, 56), (128, 28), (256, 14), (512, 7))     # channels and image side of the network's four stages
# the problem shapes of the paper's Table 1 as convolutions: N, C, H, W, K, R, S, stride, pad
TABLE1 = {"conv": (1, 128, 16, 16, 128, 3, 3, 1, 1), "matvec": (1, 512, 1, 1, 512, 1, 1, 1, 0), "square": (1, 256, 16, 16, 256, 1, 1, 1, 0)}


def listed():
    return [
        # the smallest configuration: two tenants, one small fp32 layer each; launch latency is most of it
        {"name": "pair_f32", "kind": "launch", "set": "config", "config": 1, "epilogue": "plain"},
        # four tenants at different depths of one network, batch 1: little work, few tiles, long reductions
        {"name": "ladder_b1", "kind": "launch", "set": "config", "config": 2, "epilogue": "plain"},
        # tenants of one architecture with their own weights and different batch sizes
        {"name": "same_layer_8", "kind": "launch", "set": "config", "config": 3, "epilogue": "plain"},
        # unlike tenants in one launch: 1x1, 3x3 and 7x7 stem layers, batches up to 8
        {"name": "mixed_16", "kind": "launch", "set": "config", "config": 4, "epilogue": "plain"},
        # the paper's own experiment in its own precision: R tenants of one fp32 layer
        {"name": "table1_conv_f32_r20", "kind": "launch", "set": "table1", "shape": "conv", "tenants": 20, "dtype": "f32", "out": "f32",
         "epilogue": "plain"},
        # its recurrent-network shape: a matrix-vector product per tenant, bound by the weights
        {"name": "table1_matvec_bf16_r40", "kind": "launch", "set": "table1", "shape": "matvec", "tenants": 40, "dtype": "bf16", "out": "f32",
         "epilogue": "plain"},
        # odd sizes: channel and filter counts off the vector width, rectangular filters, every stride and dtype
        {"name": "ragged_24", "kind": "launch", "set": "ragged", "tenants": 24, "shapes": 11, "epilogue": "relu"},
        # a server that merges whichever tenants are ready, on fresh buffers, through the plan cache
        {"name": "arrival_8", "kind": "arrival", "pool": 8, "sets": 5, "ready": 0.7, "trace": 11},
        # a server with several batches in flight
        {"name": "pipeline_4", "kind": "pipeline", "depth": 4, "batches": 8, "batch": 1},
        # whole networks: eight tenants, one request each, as one launch
        {"name": "stack_8x1_chain", "kind": "stack", "tenants": 8, "batch": 1, "image": 224, "form": "chain"},
        # fewer tenants with batched requests, a launch per layer
        {"name": "stack_4x4_layers", "kind": "stack", "tenants": 4, "batch": 4, "image": 224, "form": "layers"},
        # the largest: eight tenants, eight requests each
        {"name": "stack_8x8_chain", "kind": "stack", "tenants": 8, "batch": 8, "image": 224, "form": "chain"},
    ]


def _log_int(rng, lo, hi):
    """An integer in [lo, hi], spread evenly over its logarithm."""
    return min(hi, max(lo, int(lo * (hi / lo + 1e-9) ** rng.random() + rng.random())))


def draw(rng):
    pick = rng.random()
    if pick < 0.2:
        tenants = rng.choice((1, 2, 3, 4, 5, 6, 8, 8))
        return {"kind": "stack", "tenants": tenants, "batch": _log_int(rng, 1, 8), "image": rng.choice((128, 160, 176, 192, 224)),
                "form": "chain" if rng.random() < 0.6 else "layers"}
    if pick < 0.3:
        return {"kind": "arrival", "pool": rng.randint(3, 10), "sets": rng.randint(2, 6), "ready": round(rng.uniform(0.4, 0.9), 2),
                "trace": rng.randrange(1 << 20)}
    if pick < 0.4:
        depth = rng.choice((2, 3, 4))
        return {"kind": "pipeline", "depth": depth, "batches": depth * rng.randint(1, 3), "batch": _log_int(rng, 1, 4)}
    epilogue = rng.choice(("plain", "relu", "residual"))
    if pick < 0.55:
        dtype = rng.choice(("f32", "bf16", "f16"))
        return {"kind": "launch", "set": "table1", "shape": rng.choice(sorted(TABLE1)), "tenants": _log_int(rng, 2, 120), "dtype": dtype,
                "out": rng.choice(("f32", dtype)), "epilogue": epilogue}
    if pick < 0.7:
        return {"kind": "launch", "set": "ragged", "tenants": _log_int(rng, 3, 40), "shapes": rng.randrange(1 << 20), "epilogue": epilogue}
    if pick < 0.85:
        return {"kind": "launch", "set": "mixed", "tenants": _log_int(rng, 2, 32), "batch": _log_int(rng, 1, 8), "shapes": rng.randrange(1 << 20),
                "epilogue": epilogue}
    dtype = rng.choice(("f32", "bf16", "bf16", "f16"))
    while True:
        case = {"kind": "launch", "set": "even", "tenants": _log_int(rng, 1, 24), "batch": _log_int(rng, 1, 8), "channels": 8 * _log_int(rng, 2, 96),
                "filters": 8 * _log_int(rng, 2, 96), "side": _log_int(rng, 5, 80), "window": rng.choice((1, 3, 3, 5)), "stride": rng.choice((1, 1, 2)),
                "dtype": dtype, "out": rng.choice(("f32", dtype)), "epilogue": epilogue}
        if work(case)["flops"] < (2e10 if dtype == "f32" else 1e11) and work(case)["bytes"] < 4e8:
            return case


# ---- shapes -------------------------------------------------------------------------------------------------------
def _mixed(n, batch, seed):
    """1x1, 3x3 and stem layers as in configuration 4."""
    rng, out = random.Random(seed), []
    for t in range(n):
        b = rng.randint(1, batch)
        if t % 8 == 7:
            out.append(ConvShape(b, 3, 224, 224, 64, 7, 7, 2, 3))
        elif t % 2 == 0:
            h = rng.choice((7, 14, 28, 56))
            out.append(ConvShape(b, rng.choice((64, 128, 256, 512, 1024)), h, h, rng.choice((64, 128, 256, 512, 1024)), 1, 1, 1, 0))
        else:
            c, h = rng.choice((64, 128, 256, 512)), rng.choice((7, 14, 28, 56))
            out.append(ConvShape(b, c, h, h, c, 3, 3, 1, 1))
    return out


def _ragged(n, seed):
    """Layers off every round number, in every dtype, with fp32 or 16-bit outputs; one in seven is an ordinary one."""
    rng, out = random.Random(seed), []
    while len(out) < n:
        dtype = ("bf16", "f16", "f32")[len(out) % 3]
        r, s = rng.choice(((1, 1), (3, 3), (3, 3), (5, 5), (1, 7), (7, 1), (2, 3)))
        c = 8 * rng.randint(1, 32) if rng.random() < 0.5 else rng.randint(1, 260)
        k = rng.choice((8 * rng.randint(1, 32), rng.randint(1, 260)))
        shape = ConvShape(rng.randint(1, 4), c, rng.randint(3, 40), rng.randint(3, 40), k, r, s, rng.choice((1, 1, 2, 3)), rng.randint(0, max(r, s) // 2),
                          dtype, "f32" if rng.random() < 0.5 else dtype)
        if shape.H + 2 * shape.pad >= r and shape.W + 2 * shape.pad >= s:
            out.append(shape)
    return out


def _shapes(case):
    kind = case["kind"]
    if kind == "arrival":
        return [ConvShape(1, *_ladder(t)) for t in range(case["pool"])]
    if kind == "pipeline":
        return [ConvShape(case["batch"], *_ladder(t)) for t in range(4)]
    which = case["set"]
    if which == "config":
        return synth.config_shapes(case["config"])
    if which == "table1":
        return [ConvShape(*TABLE1[case["shape"]], case["dtype"], case["out"])] * case["tenants"]
    if which == "ragged":
        return _ragged(case["tenants"], case["shapes"])
    if which == "mixed":
        return _mixed(case["tenants"], case["batch"], case["shapes"])
    w = case["window"]
    return [ConvShape(case["batch"], case["channels"], case["side"], case["side"], case["filters"], w, w, case["stride"], w // 2, case["dtype"],
                      case["out"])] * case["tenants"]


def _ready_sets(case):
    """The tenants that are ready, for each of the trace's distinct steps."""
    rng, sets = random.Random(case["trace"]), []
    for _ in range(case["sets"]):
        sets.append([t for t in range(case["pool"]) if rng.random() < case["ready"]] or [rng.randrange(case["pool"])])
    return sets


def _ladder(t):
    c, h = LADDER[t % 4]
    return c, h, h, c, 3, 3, 1, 1


# ---- states -------------------------------------------------------------------------------------------------------
class _Maker:
    """Seeded device tensors."""

    def __init__(self, seed):
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def uniform(self, shape, dtype):
        return torch.empty(shape, device="cuda").uniform_(-1.0, 1.0, generator=self.gen).to(DT[dtype])

    def normal(self, shape, std, dtype):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=self.gen).to(DT[dtype])

    def layer(self, s, epilogue="plain", weight=None, out=None):
        """Descriptor of one layer on fresh tensors, and the tensors (input, weight, output, residual)."""
        x = self.uniform((s.N, s.H, s.W, s.C), s.dtype)
        w = weight if weight is not None else self.normal((s.K, s.R, s.S, s.C), (1.0 / (s.C * s.R * s.S)) ** 0.5, s.dtype)
        y = out if out is not None else torch.zeros((s.N, s.P, s.Q, s.K), dtype=DT[s.out_dtype], device="cuda")
        res = self.uniform((s.N, s.P, s.Q, s.K), s.out_dtype) if epilogue == "residual" else None
        epi = {"plain": 0, "relu": sc.ST_EPI_RELU, "residual": sc.ST_EPI_RELU | sc.ST_EPI_RESIDUAL}[epilogue]
        return sc.make_desc(s.N, s.C, s.H, s.W, s.K, s.R, s.S, s.stride, s.pad, s.dtype, s.out_dtype, x, w, y, res, epi), (x, w, y, res)


def prepare(case, seed):
    make, kind = _Maker(seed), case["kind"]
    if kind == "stack":
        stack = ResNetStack(n_tenants=case["tenants"], batch=case["batch"], image=case["image"], seeded_weights=False)
        stack.buf[0].uniform_(-1.0, 1.0, generator=make.gen)
        for st, row in zip(stack.steps, stack.weights):
            for w in row:
                w.normal_(0.0, (2.0 / (st.shape.C * st.shape.R * st.shape.S)) ** 0.5, generator=make.gen)
        if case["form"] == "chain":
            stack.build_chain()
        last = stack.steps[-1]
        s = last.shape
        out = stack.buf[last.dst][:, :s.N * s.P * s.Q * s.K]        # the network's output is the front of this buffer
        return {"kind": kind, "stack": stack, "policy": "fused_chain" if case["form"] == "chain" else "fused", "out": out}
    shapes = _shapes(case)
    if kind == "launch":
        # tenants of one shape keep their outputs in one tensor
        whole = None
        if len(set(shapes)) == 1:
            s = shapes[0]
            whole = torch.zeros((len(shapes), s.N, s.P, s.Q, s.K), dtype=DT[s.out_dtype], device="cuda")
        made = [make.layer(s, case["epilogue"], out=None if whole is None else whole[t]) for t, s in enumerate(shapes)]
        plan = sc.st_conv_plan([d for d, _ in made], keep=[t for _, t in made])
        return {"kind": kind, "plan": plan, "out": [t[2] for _, t in made] if whole is None else whole}
    if kind == "arrival":
        # two sets of request buffers per tenant, one set of weights; the plans are in the cache, as in a running server
        first = [make.layer(s) for s in shapes]
        second = [make.layer(s, weight=t[1]) for s, (_, t) in zip(shapes, first)]
        sets = _ready_sets(case)
        trace = [[made[t][0] for t in ready] for made in (first, second) for ready in sets]
        cache = sc.PlanCache(64)
        for descs in trace:
            cache.get(descs)
        return {"kind": kind, "cache": cache, "trace": trace, "keep": (first, second), "out": [t[2] for made in (first, second) for _, t in made]}
    pipe = sc.Pipeline(case["depth"])
    weights = [make.normal((s.K, s.R, s.S, s.C), (1.0 / (s.C * s.R * s.S)) ** 0.5, s.dtype) for s in shapes]
    batches = [[make.layer(s, weight=w) for s, w in zip(shapes, weights)] for _ in range(case["batches"])]
    plans = [sc.st_conv_plan([d for d, _ in b], sc.plan_opts(target_items=pipe.slots), keep=[t for _, t in b]) for b in batches]
    return {"kind": kind, "pipe": pipe, "plans": plans, "out": [t[2] for b in batches for _, t in b]}


def run(state):
    kind = state["kind"]
    if kind == "launch":
        sc.st_conv_run(state["plan"], torch.cuda.current_stream())
    elif kind == "stack":
        state["stack"].run(state["policy"], torch.cuda.current_stream())
    elif kind == "arrival":
        stream = torch.cuda.current_stream()
        for descs in state["trace"]:
            plan, _ = state["cache"].get(descs, stream)
            sc.st_conv_run(plan, stream)
    else:
        state["pipe"].run_many(state["plans"])
    return state["out"]


# ---- what a pass cannot do without --------------------------------------------------------------------------------
def work(case):
    if case["kind"] == "stack":
        steps, n = synth.resnet50_steps(case["batch"], case["image"]), case["tenants"]
        flops = n * sum(st.shape.flops for st in steps)
        if case["form"] == "layers":        # every layer's tensors go through the caller's buffers
            return {"bytes": n * sum(st.shape.bytes for st in steps), "flops": flops}
        first, last = steps[0].shape, steps[-1].shape
        weights = sum(st.shape.K * st.shape.C * st.shape.R * st.shape.S for st in steps)
        return {"bytes": n * 2 * (first.N * first.C * first.H * first.W + weights + last.N * last.K * last.P * last.Q), "flops": flops}
    shapes = _shapes(case)
    if case["kind"] == "arrival":
        ready = [shapes[t] for tenants in _ready_sets(case) for t in tenants]
        return {"bytes": 2 * sum(s.bytes for s in ready), "flops": 2 * sum(s.flops for s in ready)}
    times = case["batches"] if case["kind"] == "pipeline" else 1
    total = {"bytes": times * sum(s.bytes for s in shapes), "flops": times * sum(s.flops for s in shapes)}
    if case["kind"] == "launch" and case["epilogue"] == "residual":
        total["bytes"] += sum(s.N * s.P * s.Q * s.K * ES[s.out_dtype] for s in shapes)
    return total


def tolerance(case):
    if case["kind"] == "stack":
        # 53 layers whose activations are rounded to bf16 (2^-9 each): two correct summation orders drift apart until
        # their rounding errors are independent, about 1 % of the output each
        return {"rel": 2e-2, "max": 0.3}
    out = {s.out_dtype for s in _shapes(case)}
    if "bf16" in out:
        return {"rel": 2e-3, "max": 1e-2}       # a sum at a rounding boundary moves by one step, 2^-8
    if "f16" in out:
        return {"rel": 5e-4, "max": 2e-3}
    return {"rel": 1e-5, "max": 4e-4}           # products of 16-bit inputs are exact; fp32 sums in another order
