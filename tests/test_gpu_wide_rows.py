"""Output rows so long that the rows of a tile past the last pixel lie more than 2^32 bytes into the tensor: nothing of them may come
round into it.  The operands are small integers, so every sum is exact in the output's type."""
import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu


def _layer(K, C, H, W, R, stride, pad, dtype, out, residual):
    """A layer of K filters on small integers, and what it has to give."""
    import torch
    import torch.nn.functional as F
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
    g = torch.Generator(device="cuda").manual_seed(K + W)
    x = torch.randint(1, 3, (1, H, W, C), generator=g, device="cuda").to(dt[dtype])
    w = torch.randint(-2, 3, (K, R, R, C), generator=g, device="cuda", dtype=torch.int8).to(dt[dtype])
    P, Q = (H + 2 * pad - R) // stride + 1, (W + 2 * pad - R) // stride + 1
    # windows by hand, [pixel][tap and channel]
    windows = F.unfold(x.permute(0, 3, 1, 2).float(), R, padding=pad, stride=stride).view(C, R * R, P * Q).permute(2, 1, 0).reshape(P * Q, R * R * C)
    want = windows @ w.view(K, R * R * C).float().t()
    res = None
    if residual:
        res = torch.randint(-3, 4, (1, P, Q, K), generator=g, device="cuda", dtype=torch.int8).to(dt[out])
        want += res.view(P * Q, K).float()
    y = torch.full((1, P, Q, K), 77.0, dtype=dt[out], device="cuda")
    desc = sc.make_desc(1, C, H, W, K, R, R, stride, pad, dtype, out, x, w, y, res, sc.ST_EPI_RESIDUAL if residual else 0)
    return desc, y, want, (x, w, res)


def _check(y, want, what):
    import torch
    torch.cuda.synchronize()
    assert torch.equal(y.view(want.shape).float(), want), what


def _run_plan(desc, opts, y, want, keep):
    plan = sc.st_conv_plan([desc], sc.plan_opts(**opts), keep=keep)
    sc.st_conv_run(plan)
    _check(y, want, "launch")
    return plan


@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("K,W,tile", [((1 << 22) - 8, 3, 1),         # 127 rows end just below 2^31 bytes (16-bit), 128x128 tiles
                                      (1 << 25, 3, 1), ((1 << 25) + 4, 2, 1), (1 << 25, 1, 4)])
def test_rows_past_the_last_pixel_stay_out(out, residual, K, W, tile):
    print(f"wide rows: K={K} W={W} tile={tile} out={out} residual={residual}", flush=True)
    desc, y, want, keep = _layer(K, 8, 1, W, 1, 1, 0, "bf16", out, residual)
    _run_plan(desc, dict(tile_cfg=tile), y, want, keep)


@pytest.mark.parametrize("K", [1 << 25, (1 << 25) + 4])
@pytest.mark.parametrize("dtype,out,residual", [("f16", "f16", False), ("f16", "f16", True), ("f32", "f32", False), ("f32", "f32", True)])
def test_other_operand_types(dtype, out, residual, K):
    print(f"wide rows: K={K} dtype={dtype} out={out} residual={residual}", flush=True)
    desc, y, want, keep = _layer(K, 8, 1, 2, 1, 1, 0, dtype, out, residual)
    _run_plan(desc, dict(tile_cfg=2), y, want, keep)


@pytest.mark.parametrize("K", [1 << 25, (1 << 25) + 3])              # whole vectors, and the end of the rows by element behind them
@pytest.mark.parametrize("C", [9, 3])                                # in pieces, and gathered: the kernel for everything
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_any_channel_count(K, C, out):
    print(f"wide rows: K={K} C={C} out={out}", flush=True)
    desc, y, want, keep = _layer(K, C, 1, 3, 1, 1, 0, "bf16", out, False)
    plan = _run_plan(desc, dict(tile_cfg=2), y, want, keep)
    assert sc.st_conv_plan_tenant_form(plan, 0) == (sc.ST_FORM_PIECES if C == 9 else sc.ST_FORM_GATHERED)


@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("residual", [False, True])
def test_row_tile(out, residual):
    """Several output rows and slices of a row: a row of outputs ends inside the tensor, where only the comparison keeps stores out."""
    K = 1 << 23
    print(f"wide rows: row tile, out={out} residual={residual}", flush=True)
    desc, y, want, keep = _layer(K, 3, 5, 40, 3, 2, 1, "bf16", out, residual)
    plan = _run_plan(desc, dict(tile_cfg=7), y, want, keep)
    assert sc.st_conv_plan_tenant_info(plan, 0).row_tiled == 1


def test_split_reduction():
    K = 1 << 22
    print("wide rows: split reduction", flush=True)
    desc, y, want, keep = _layer(K, 128, 1, 3, 1, 1, 0, "bf16", "bf16", True)
    plan = _run_plan(desc, dict(tile_cfg=2, split_k=2), y, want, keep)
    assert sc.st_conv_plan_tenant_info(plan, 0).split_k == 2


@pytest.mark.parametrize("chain_queues", [1, 2])
@pytest.mark.parametrize("K", [1 << 25, (1 << 25) + 4])              # rows stored as vectors, and by element (one queue: behind a release fence)
@pytest.mark.parametrize("out", ["bf16", "f32"])
def test_a_chain_reads_them_back(out, K, chain_queues):
    """Two layers in one launch, the second with the long rows that the first has written as its residual: read on other compute units,
    with one queue on other XCDs, too."""
    import torch
    print(f"wide rows: chain_queues={chain_queues} K={K} out={out}", flush=True)
    desc, y, want, keep = _layer(K, 8, 1, 3, 1, 1, 0, "bf16", out, False)
    _, z, want2, (x2, w2, _) = _layer(K, 16, 1, 3, 1, 1, 0, "bf16", out, False)
    want2 = want2 + want
    second = sc.make_desc(1, 16, 1, 3, K, 1, 1, 1, 0, "bf16", out, x2, w2, z, y, sc.ST_EPI_RESIDUAL)
    chain = sc.Chain([sc.make_chain_op(sc.ST_OP_CONV, 0, 0, desc), sc.make_chain_op(sc.ST_OP_CONV, 0, 1, second)],
                     sc.plan_opts(chain_queues=chain_queues, tile_cfg=1), keep=[keep, x2, w2, y, z])
    chain.set_wait_limit_us(2_000_000)                              # 262144 tiles on one XCD before the second layer's last may start
    for _ in range(3):
        y.fill_(77.0)
        z.fill_(55.0)
        chain.run()
        _check(y, want, "first layer")
        _check(z, want2, "second layer")
    assert not chain.aborted()
