"""Split reductions of two to nine slices: fewer than, as many as and more than the slices that a tile's last workgroup reads at a
time (four or eight), on every tile shape, where whichever slice arrives last may be the one it keeps in registers."""
import pytest

from paper_1901_00041_amd import st_conv as sc
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


def _shapes(split_k):
    """Slices of eight steps of 128 bytes or four of 256, the last one half a step of 256 short."""
    c = split_k * 512 - 64
    return {"f32": ConvShape(1, c // 2, 13, 11, 136, 1, 1, 1, 0, "f32", "f32"), "bf16": ConvShape(1, c, 13, 11, 136, 1, 1, 1, 0, "bf16", "f32"),
            "f16": ConvShape(1, c, 5, 5, 72, 1, 1, 1, 0, "f16", "f16")}


@pytest.mark.parametrize("split_k", [2, 3, 4, 5, 7, 8, 9])
@pytest.mark.parametrize("tile_cfg", [1, 2, 3, 4, 5, 6])
def test_every_number_of_slices(tile_cfg, split_k):
    """A launch of one type takes that type's kernel, a launch of several the one for everything, and a chain has kernels of its own, for
    bf16 and for everything, with columns and with one queue: the slices are read in another way in each, and summed in the
    same order."""
    import torch
    from tests import helpers
    shapes = _shapes(split_k)
    tenants = helpers.make_tenants(1, list(shapes.values()))
    of_type = dict(zip(shapes, tenants))
    results = {}

    def check(names, run, what):
        for rep in range(4):             # the counters are left as they were found
            for n in names:
                of_type[n].clear()
            run()
            torch.cuda.synchronize()
            for n in names:
                if n not in results:
                    helpers.check_tenant(of_type[n], f"tile {tile_cfg} split {split_k} {n}")
                    results[n] = of_type[n].dy.clone()
                assert torch.equal(of_type[n].dy, results[n]), f"{what} {n} run {rep}"

    for names in (["f32"], ["bf16"], ["f16"], list(shapes)):
        plan = helpers.plan_for([of_type[n] for n in names], tile_cfg=tile_cfg, split_k=split_k)
        assert all(sc.st_conv_plan_tenant_info(plan, i).split_k == split_k for i in range(len(names)))
        check(names, lambda: sc.st_conv_run(plan), f"launch of {len(names)}")
    for names in (["bf16"], list(shapes)):
        for queues in (1, 2):
            ops = [sc.make_chain_op(sc.ST_OP_CONV, i, 0, of_type[n].desc()) for i, n in enumerate(names)]
            chain = sc.Chain(ops, sc.plan_opts(tile_cfg=tile_cfg, split_k=split_k, chain_queues=queues), keep=tenants)
            assert all(chain.op_info(i).tile.split_k == split_k for i in range(len(names)))
            check(names, chain.run, f"chain_queues={queues} of {len(names)}")
            assert not chain.aborted()
