"""Split reductions of two to nine slices: fewer than, as many as and more than the slices that a tile's last workgroup reads at a
time (four or eight), on every tile shape, where whichever slice arrives last may be the one it keeps in registers."""
import pytest

from paper_1901_00041_amd import st_conv as sc
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split_k", [2, 3, 4, 5, 8, 9])
@pytest.mark.parametrize("tile_cfg", [1, 2, 3, 4, 5, 6])
def test_every_number_of_slices(tile_cfg, split_k):
    import torch
    from tests import helpers
    shapes = [ConvShape(1, 2304, 13, 11, 136, 1, 1, 1, 0, "f32", "f32"), ConvShape(1, 4608, 13, 11, 136, 1, 1, 1, 0, "bf16", "f32"),
              ConvShape(1, 4608, 5, 5, 72, 1, 1, 1, 0, "f16", "f16")]      # 72 steps of 128 bytes, 36 of 256
    tenants = helpers.make_tenants(1, shapes)
    plan = helpers.plan_for(tenants, tile_cfg=tile_cfg, split_k=split_k)
    assert all(sc.st_conv_plan_tenant_info(plan, i).split_k == split_k for i in range(len(tenants)))
    first = None
    for rep in range(4):             # the counters are left as they were found
        for t in tenants:
            t.clear()
        sc.st_conv_run(plan)
        torch.cuda.synchronize()
        if first is None:
            first = [t.dy.clone() for t in tenants]
            for i, t in enumerate(tenants):
                helpers.check_tenant(t, f"tile {tile_cfg} split {split_k} tenant {i}")
        assert all(torch.equal(t.dy, f) for t, f in zip(tenants, first)), f"run {rep}"
