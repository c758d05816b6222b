"""ReLU in the epilogues on the values a comparison treats specially: NaN and negative values give zero, infinity stays, in every way
out of a tile (16-bit outputs, fp32 outputs, stores by element, with and without a residual).  Compared bit for bit: what is zero is
+0, also for -0 and for what is too small for the type."""
import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu

VALUES = (float("nan"), float("inf"), float("-inf"), -0.0, 0.0, 1e-38, -1e-38, 3.0, -3.0, 1e30)


def _dtype(name):
    import torch
    return {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}[name]


def _same_bits(y, want, what=""):
    import torch
    bits = torch.int32 if y.dtype == torch.float32 else torch.int16
    assert torch.equal(y.view(bits), want.to(y.dtype).contiguous().view(bits)), what


def _pointwise(C, K, dtype, out, residual):
    """A 1x1 layer that copies channel 0 of its input, which holds the values, into every filter; what it has to give; its tensors."""
    import torch
    side = 13
    x = torch.zeros((1, side, side, C), dtype=_dtype(dtype), device="cuda")
    v = torch.tensor([VALUES[i % len(VALUES)] for i in range(side * side)], device="cuda").to(_dtype(dtype))
    x[0, :, :, 0] = v.view(side, side)
    w = torch.zeros((K, 1, 1, C), dtype=_dtype(dtype), device="cuda")
    w[:, 0, 0, 0] = 1
    y = torch.full((1, side, side, K), 7.0, dtype=_dtype(out), device="cuda")
    res = torch.full_like(y, residual) if residual is not None else None
    epi = sc.ST_EPI_RELU | (sc.ST_EPI_RESIDUAL if res is not None else 0)
    s = v.float() + (residual or 0.0)
    want = torch.where(s > 0, s, torch.zeros_like(s)).view(1, side, side, 1).expand(-1, -1, -1, K)
    return sc.make_desc(1, C, side, side, K, 1, 1, 1, 0, dtype, out, x, w, y, res, epi), want, y, (x, w, res)


def _run_all(desc, opts, y, want, keep, queues=()):
    import torch
    plan = sc.st_conv_plan([desc], sc.plan_opts(**opts), keep=keep)
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    _same_bits(y, want, "launch")
    for q in queues:
        y.fill_(7.0)
        chain = sc.Chain([sc.make_chain_op(sc.ST_OP_CONV, 0, 0, desc)], sc.plan_opts(chain_queues=q, **opts), keep=keep)
        chain.run()
        torch.cuda.synchronize()
        assert not chain.aborted()
        _same_bits(y, want, f"chain_queues={q}")
    return plan


@pytest.mark.parametrize("dtype,out", [("bf16", "bf16"), ("bf16", "f32"), ("f16", "f16"), ("f32", "f32")])
@pytest.mark.parametrize("K", [128, 20])                   # whole vectors of filters, and not
@pytest.mark.parametrize("residual", [None, -1.0, -0.0])
@pytest.mark.parametrize("tile", [0, 1, 4, 6])             # the planner's choice, 128x128, 64x64, 16x64
def test_relu_of_special_values(dtype, out, K, residual, tile):
    desc, want, y, keep = _pointwise(64, K, dtype, out, residual)
    _run_all(desc, dict(tile_cfg=tile), y, want, keep)


@pytest.mark.parametrize("dtype,out", [("bf16", "bf16"), ("bf16", "f32"), ("f32", "f32")])
@pytest.mark.parametrize("C,form", [(67, sc.ST_FORM_PIECES), (3, sc.ST_FORM_GATHERED)])
@pytest.mark.parametrize("K", [129, 128])                  # the end of the rows by element behind whole vectors, and whole vectors
@pytest.mark.parametrize("residual", [None, -1.0])
def test_relu_in_the_kernel_for_everything(dtype, out, C, form, K, residual):
    desc, want, y, keep = _pointwise(C, K, dtype, out, residual)
    plan = _run_all(desc, dict(tile_cfg=4), y, want, keep, queues=(1, 2))
    assert sc.st_conv_plan_tenant_form(plan, 0) == form


@pytest.mark.parametrize("dtype,out", [("bf16", "bf16"), ("f32", "f32")])
@pytest.mark.parametrize("residual", [None, -1.0])
def test_relu_behind_a_split_reduction(dtype, out, residual):
    desc, want, y, keep = _pointwise(320, 72, dtype, out, residual)
    plan = _run_all(desc, dict(tile_cfg=4, split_k=3), y, want, keep, queues=(1, 2))
    assert sc.st_conv_plan_tenant_info(plan, 0).split_k == 3


@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_relu_in_the_row_tile(out):
    """A stem that copies the middle of its window: the values lie so far apart that no window holds two, so an output is its value, or
    zero, or zero times a value beside it, which is NaN and becomes zero."""
    import torch
    N, C, H, W, K, R, stride, pad = 1, 3, 33, 128, 64, 7, 2, 3
    x = torch.zeros((N, H, W, C), dtype=torch.bfloat16, device="cuda")
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    want = torch.zeros((N, P, Q, 1), device="cuda")
    k = 0
    for p in range(0, P, 4):
        for q in range(0, Q, 4):
            v = torch.tensor(VALUES[k % len(VALUES)]).to(torch.bfloat16)
            x[0, stride * p, stride * q, 0] = v
            want[0, p, q, 0] = v.float() if v > 0 else 0.0
            k += 1
    w = torch.zeros((K, R, R, C), dtype=torch.bfloat16, device="cuda")
    w[:, R // 2, R // 2, 0] = 1
    y = torch.full((N, P, Q, K), 7.0, dtype=_dtype(out), device="cuda")
    desc = sc.make_desc(N, C, H, W, K, R, R, stride, pad, "bf16", out, x, w, y, None, sc.ST_EPI_RELU)
    plan = _run_all(desc, dict(tile_cfg=7), y, want.expand(-1, -1, -1, K), (x, w), queues=(1, 2))
    assert sc.st_conv_plan_tenant_info(plan, 0).row_tiled == 1
