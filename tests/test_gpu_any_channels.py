"""Channel counts that are not a multiple of the 16-byte vector: vectors that cross into the next filter row, into the padding or
past the end of the reduction index, at the start and the end of the tensor.  Counts that hold a vector go through in pieces, the
others (and five fp32 channels) through the gathered tile."""
import pytest

from paper_1901_00041_amd import synth
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


def _shapes(dtype):
    out = "f32"
    return [
        ConvShape(1, 1, 5, 6, 3, 3, 3, 1, 1, dtype, out),         # one channel: a vector spans several filter rows
        ConvShape(2, 2, 7, 5, 9, 5, 2, 1, 1, dtype, out),
        ConvShape(1, 7, 9, 9, 70, 3, 3, 1, 1, dtype, out),        # filter rows of 21 elements
        ConvShape(3, 67, 5, 7, 33, 3, 3, 2, 1, dtype, out),
        ConvShape(1, 131, 6, 6, 65, 1, 1, 1, 0, dtype, out),      # only the end of the reduction index is ragged
        ConvShape(1, 9, 1, 1, 5, 1, 1, 1, 0, dtype, out),
        ConvShape(1, 9, 3, 3, 5, 3, 3, 1, 3, dtype, out),         # padding as wide as the filter: whole filter rows outside
        ConvShape(1, 239, 4, 5, 16, 5, 5, 3, 2, dtype, out),
        ConvShape(1, 33, 6, 4, 40, 1, 4, 1, 2, dtype, out),
    ]


@pytest.mark.parametrize("split_k", [1, 3])
@pytest.mark.parametrize("tile_cfg", [2, 4])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_any_channel_count(dtype, tile_cfg, split_k):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    tenants = [helpers.Tenant(s, synth.gen_input(93, t, 0, s), synth.gen_weight(93, t, 0, s)) for t, s in enumerate(_shapes(dtype))]
    plan = helpers.plan_for(tenants, tile_cfg=tile_cfg, split_k=split_k)
    vec = 4 if dtype == "f32" else 8
    for i, t in enumerate(tenants):
        assert sc.st_conv_plan_tenant_form(plan, i) == (sc.ST_FORM_PIECES if t.shape.C > vec else sc.ST_FORM_GATHERED)
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    for i, t in enumerate(tenants):
        helpers.check_tenant(t, f"channels[{i}] {t.shape} tile_cfg={tile_cfg} split_k={split_k}")


# N, C (16-bit types, fp32), H, W, K, R, S, stride, pad: one step or many, slices that end inside a vector, rows shorter than a vector
GATHERED = [(1, (1, 1), 20, 20, 70, 9, 9, 1, 4), (2, (3, 3), 12, 17, 65, 7, 7, 1, 3), (1, (5, 5), 9, 8, 33, 11, 3, 1, 1), (3, (7, 5), 6, 7, 130, 5, 5, 2, 2), (1, (7, 5), 31, 9, 64, 1, 1, 1, 0),
            (1, (2, 2), 15, 14, 16, 13, 13, 1, 6), (2, (6, 3), 5, 40, 24, 3, 1, 1, 2), (1, (7, 5), 14, 14, 129, 13, 1, 3, 0)]


@pytest.mark.parametrize("split_k", [1, 2, 5])
@pytest.mark.parametrize("tile_cfg", [2, 4])
@pytest.mark.parametrize("dtype,out", [("bf16", "f32"), ("f16", "f16"), ("f32", "f32")])
def test_gathered(dtype, out, tile_cfg, split_k):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    shapes = [ConvShape(n, c[dtype == "f32"], h, w, k, r, s, stride, pad, dtype, out) for n, c, h, w, k, r, s, stride, pad in GATHERED]
    tenants = [helpers.Tenant(s, synth.gen_input(94, t, 0, s), synth.gen_weight(94, t, 0, s)) for t, s in enumerate(shapes)]
    plan = helpers.plan_for(tenants, tile_cfg=tile_cfg, split_k=split_k)
    for i in range(len(tenants)):
        assert sc.st_conv_plan_tenant_form(plan, i) == sc.ST_FORM_GATHERED
        assert sc.st_conv_plan_tenant_info(plan, i).tile_cfg == tile_cfg - 1
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    for i, t in enumerate(tenants):
        helpers.check_tenant(t, f"gathered[{i}] {t.shape} tile_cfg={tile_cfg} split_k={split_k}")
