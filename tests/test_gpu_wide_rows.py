"""Output rows so long that the rows of a tile past the last pixel lie more than 2^32 bytes into the tensor: nothing of them may come
round into it.  The operands are small integers, so every sum is exact in the output's type."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out", ["bf16", "f32"])
@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("K,W,tile", [((1 << 22) - 8, 3, 1),         # the longest rows stored as vectors, 128x128 tiles
                                      (1 << 25, 3, 1), ((1 << 25) + 4, 2, 1), (1 << 25, 1, 4)])
def test_rows_past_the_last_pixel_stay_out(out, residual, K, W, tile):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[out]
    print(f"wide rows: K={K} W={W} tile={tile} out={out} residual={residual}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K + W)
    C = 8
    x = torch.randint(1, 3, (1, 1, W, C), generator=g, device="cuda").to(torch.bfloat16)
    w = torch.randint(-2, 3, (K, 1, 1, C), generator=g, device="cuda", dtype=torch.int8).to(torch.bfloat16)
    want = x.view(W, C).float() @ w.view(K, C).float().t()
    res = None
    if residual:
        res = torch.randint(-3, 4, (1, 1, W, K), generator=g, device="cuda", dtype=torch.int8).to(dt)
        want += res.view(W, K).float()
    y = torch.full((1, 1, W, K), 77.0, dtype=dt, device="cuda")
    plan = sc.st_conv_plan([sc.make_desc(1, C, 1, W, K, 1, 1, 1, 0, "bf16", out, x, w, y, res, sc.ST_EPI_RESIDUAL if residual else 0)],
                           sc.plan_opts(tile_cfg=tile))
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    assert torch.equal(y.view(W, K).float(), want)
