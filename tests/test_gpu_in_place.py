"""A residual that is the output itself: every element is read by the tile that writes it, before it is written, on every way out of a
tile (a 16-bit residual staged in LDS, one loaded in the epilogue, stores by element, the last slice of a split reduction) and by
no other tile.  Bitwise what the same layer gives on a residual of its own."""
import pytest

from paper_1901_00041_amd import st_conv as sc
from paper_1901_00041_amd import synth
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


def _shapes(dtype):
    return [ConvShape(2, 64, 9, 11, 40, 1, 1, 1, 0, dtype, dtype), ConvShape(1, 640, 9, 11, 200, 1, 1, 1, 0, dtype, dtype),        # one step, many
            ConvShape(1, 128, 13, 9, 72, 3, 3, 2, 1, dtype, dtype), ConvShape(2, 24, 11, 10, 136, 3, 3, 1, 1, dtype, "f32"),
            ConvShape(5, 64, 7, 7, 72, 3, 3, 1, 1, dtype, dtype), ConvShape(1, 128, 8, 11, 136, 3, 3, 1, 0, dtype, dtype),        # patches
            ConvShape(1, 67, 7, 9, 40, 3, 3, 1, 1, dtype, dtype), ConvShape(1, 13, 9, 8, 65, 3, 3, 2, 1, dtype, "f32"),           # pieces, gathered
            ConvShape(2, 3, 20, 37, 40, 7, 7, 2, 3, dtype, dtype), ConvShape(1, 4, 9, 19, 24, 3, 7, 1, 3, dtype, "f32"),          # rows
            ConvShape(1, 64, 9, 9, 30, 1, 1, 1, 0, dtype, dtype), ConvShape(1, 256, 9, 9, 33, 1, 1, 1, 0, dtype, dtype)]          # by element


@pytest.mark.parametrize("split_k", [1, 3])
@pytest.mark.parametrize("tile_cfg", [0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_output_is_the_residual(dtype, tile_cfg, split_k):
    import torch
    from tests import helpers
    tenants = []
    for t, s in enumerate(_shapes(dtype)):
        res = synth.to_storage(synth.uniform_pm1(synth.stream_state(92, t, 0, 3), s.N * s.K * s.P * s.Q), s.out_dtype).reshape(s.N, s.K, s.P, s.Q)
        tenants.append(helpers.Tenant(s, synth.gen_input(92, t, 0, s), synth.gen_weight(92, t, 0, s, 2.0), residual=res, relu=t % 3 != 2))
    opts = dict(tile_cfg=tile_cfg, split_k=split_k)
    plan = helpers.plan_for(tenants, **opts)
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    want = []
    for i, t in enumerate(tenants):
        helpers.check_tenant(t, f"apart {i}")
        want.append(t.dy.clone())
    first = [t.dres.clone() for t in tenants]
    for t in tenants:
        t.dy = t.dres
    singles = [helpers.plan_for([t], **opts) for t in tenants]           # the kernels of one type
    together = helpers.plan_for(tenants, **opts)

    def run_singles():
        for p in singles:
            sc.st_conv_run(p)
    ops = [sc.make_chain_op(sc.ST_OP_CONV, i, 0, t.desc()) for i, t in enumerate(tenants)]
    chains = [sc.Chain(ops, sc.plan_opts(chain_queues=q, **opts), keep=tenants) for q in (0, 1, 2)]
    for what, run in [("one launch", lambda: sc.st_conv_run(together)), ("a launch each", run_singles)] + [(f"chain {k}", c.run) for k, c in enumerate(chains)]:
        if what == "a launch each" and tile_cfg == 0:
            continue               # planned alone, other tiles may be chosen
        for t, r in zip(tenants, first):
            t.dy.copy_(r)
        torch.cuda.synchronize()
        run()
        torch.cuda.synchronize()
        for i, t in enumerate(tenants):
            assert torch.equal(t.dy, want[i]), f"{what}: tenant {i} {t.shape} {opts}"
    assert not any(c.aborted() for c in chains)


def test_a_pass_is_repeatable_and_a_step_in_place_adds_anew():
    """A stack's blocks add to their shortcut in place: whole passes give the same bits again, a single step run twice adds twice."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=2, image=64, seeded_weights=False)
    last = stack.steps[-1]
    outs = []
    for _ in range(3):
        stack.run("fused")
        torch.cuda.synchronize()
        outs.append(stack.buf[last.dst].clone())
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2]) and float(outs[0].float().abs().max()) > 0
    st = next(st for st in stack.steps if st.res is not None)
    assert st.dst == st.res and st.src != st.dst
    s = st.shape
    runs = []
    for _ in range(3):
        runs.append(stack.view(st.dst, 0, s.N, s.P, s.Q, s.K).float().clone())
        stack.run_step(st.index)
        torch.cuda.synchronize()
    assert (runs[2] >= 0).all() and not torch.equal(runs[1], runs[2])
    stack.run("fused")
    torch.cuda.synchronize()
    assert torch.equal(stack.buf[last.dst], outs[0])
