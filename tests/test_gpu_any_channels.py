"""Channel counts that are not a multiple of the 16-byte vector: vectors that cross into the next filter row, into the padding or
past the end of the reduction index, at the start and the end of the tensor."""
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
    sc.st_conv_run(plan)
    torch.cuda.synchronize()
    for i, t in enumerate(tenants):
        helpers.check_tenant(t, f"channels[{i}] {t.shape} tile_cfg={tile_cfg} split_k={split_k}")
