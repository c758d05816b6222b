"""ReLU in the epilogues on the values a comparison treats specially: NaN and negative values give zero, infinity stays, in every way
out of a tile (16-bit outputs, fp32 outputs, stores by element, with and without a residual)."""
import pytest

pytestmark = pytest.mark.gpu

VALUES = (float("nan"), float("inf"), float("-inf"), -0.0, 0.0, 1e-38, -1e-38, 3.0, -3.0, 1e30)


@pytest.mark.parametrize("dtype,out", [("bf16", "bf16"), ("bf16", "f32"), ("f16", "f16"), ("f32", "f32")])
@pytest.mark.parametrize("K", [128, 20])                   # whole vectors of filters, and not
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("tile", [0, 1, 4, 6])             # the planner's choice, 128x128, 64x64, 16x64
def test_relu_of_special_values(dtype, out, K, residual, tile):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16}
    side, C = 13, 64
    x = torch.zeros((1, side, side, C), dtype=dt[dtype], device="cuda")
    v = torch.tensor([VALUES[i % len(VALUES)] for i in range(side * side)], device="cuda").to(dt[dtype])
    x[0, :, :, 0] = v.view(side, side)
    w = torch.zeros((K, 1, 1, C), dtype=dt[dtype], device="cuda")
    w[:, 0, 0, 0] = 1
    y = torch.full((1, side, side, K), 7.0, dtype=dt[out], device="cuda")
    res = torch.full_like(y, -1.0) if residual else None
    epi = sc.ST_EPI_RELU | (sc.ST_EPI_RESIDUAL if residual else 0)
    plan = sc.st_conv_plan([sc.make_desc(1, C, side, side, K, 1, 1, 1, 0, dtype, out, x, w, y, res, epi)], sc.plan_opts(tile_cfg=tile))
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    s = v.float() + (-1.0 if residual else 0.0)
    want = torch.where(s > 0, s, torch.zeros_like(s)).to(dt[out]).view(1, side, side, 1).expand(-1, -1, -1, K)
    assert torch.equal(y, want)
