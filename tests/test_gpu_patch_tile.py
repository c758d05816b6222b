"""3x3 stride-1 layers whose input patch a tile keeps in LDS: rows of 2 to 70 pixels, tiles that cross images, one to nine
channel blocks, padded and not, ragged pixels and filters, split reductions; beside them layers just outside that form."""
import pytest

from paper_1901_00041_amd import synth
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu

SHAPES = [
    ConvShape(5, 64, 7, 7, 72, 3, 3, 1, 1, "bf16", "f32"),       # one channel block of 128 bytes, five images in 245 pixels
    ConvShape(1, 128, 9, 28, 64, 3, 3, 1, 1, "f16", "f32"),      # two blocks of 128 bytes, one of 256
    ConvShape(2, 256, 5, 14, 40, 3, 3, 1, 1, "bf16", "bf16"),
    ConvShape(1, 576, 8, 9, 24, 3, 3, 1, 1, "bf16", "f32"),      # nine blocks of 128 bytes: an odd number, and no 256-byte step
    ConvShape(2, 128, 8, 11, 33, 3, 3, 1, 0, "bf16", "f32"),     # no padding: gaps between output rows and between images
    ConvShape(1, 64, 6, 70, 64, 3, 3, 1, 1, "bf16", "f32"),      # wide rows
    ConvShape(1, 128, 5, 57, 64, 3, 3, 1, 0, "bf16", "f32"),     # rows at the limit of the smaller tiles' LDS
    ConvShape(1, 64, 3, 3, 16, 3, 3, 1, 0, "f16", "f16"),        # a single output pixel
    ConvShape(40, 64, 2, 2, 64, 3, 3, 1, 1, "bf16", "f32"),      # many images in one tile
    ConvShape(1, 256, 28, 29, 64, 3, 3, 1, 1, "bf16", "f32"),
    ConvShape(1, 64, 8, 8, 64, 3, 3, 1, 2, "bf16", "f32"),       # outside: more output than input
    ConvShape(1, 64, 8, 8, 64, 5, 5, 1, 2, "bf16", "f32"),       #   another filter
    ConvShape(1, 72, 8, 8, 64, 3, 3, 1, 1, "bf16", "f32"),       #   channels not a multiple of the step
]


@pytest.mark.parametrize("split_k", [1, 2])
@pytest.mark.parametrize("tile_cfg", [1, 2, 3, 4, 5])
def test_patch_tile_edges(tile_cfg, split_k):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    tenants = [helpers.Tenant(s, synth.gen_input(92, t, 0, s), synth.gen_weight(92, t, 0, s)) for t, s in enumerate(SHAPES)]
    plan = helpers.plan_for(tenants, tile_cfg=tile_cfg, split_k=split_k)
    for rep in range(2):
        for t in tenants:
            t.clear()
        sc.st_conv_run(plan)
        torch.cuda.synchronize()
        for i, t in enumerate(tenants):
            helpers.check_tenant(t, f"patch[{i}] {t.shape} tile_cfg={tile_cfg} split_k={split_k}")
