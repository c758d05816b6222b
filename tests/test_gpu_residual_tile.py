"""Residual and ReLU in the epilogue, per tile shape.  A 16-bit residual tile travels to LDS during the last K steps, into a
stage that depends on the number of steps and of stages: reductions of one step to more than two turns of the stages, in all
walk orders, with ragged pixels and filters.  Everything else reads the residual in the epilogue."""
import pytest

from paper_1901_00041_amd import synth
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


def _tenants(shapes, key):
    from tests import helpers
    out = []
    for t, s in enumerate(shapes):
        res = synth.to_storage(synth.uniform_pm1(synth.stream_state(key, t, 0, 3), s.N * s.K * s.P * s.Q), s.out_dtype)
        out.append(helpers.Tenant(s, synth.gen_input(key, t, 0, s), synth.gen_weight(key, t, 0, s, 2.0), residual=res.reshape(s.N, s.K, s.P, s.Q),
                                  relu=t % 3 != 2))
    return out


def _check(shapes, key, what, **opts):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    tenants = _tenants(shapes, key)
    plan = helpers.plan_for(tenants, **opts)
    for rep in range(2):
        for t in tenants:
            t.clear()
        sc.st_conv_run(plan)
        torch.cuda.synchronize()
        for i, t in enumerate(tenants):
            helpers.check_tenant(t, f"{what}[{i}] {t.shape} {opts}")
    # the same tiles in the persistent kernel, which reads activations and residuals past the caches
    want = [t.dy.clone() for t in tenants]
    ops = [sc.make_chain_op(sc.ST_OP_CONV, i, 0, t.desc()) for i, t in enumerate(tenants)]
    for queues in (1, 2):
        chain = sc.Chain(ops, sc.plan_opts(chain_queues=queues, **opts), keep=tenants)
        for t in tenants:
            t.clear()
        chain.run()
        torch.cuda.synchronize()
        assert not chain.aborted()
        for i, t in enumerate(tenants):
            assert torch.equal(t.dy, want[i]), f"{what}[{i}] {t.shape} {opts} chain_queues={queues}"


@pytest.mark.parametrize("split_k", [1, 3])
@pytest.mark.parametrize("tile_cfg", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
def test_residual_stage(dtype, tile_cfg, split_k):
    linear = [ConvShape(2, c, 9, 11, k, 1, 1, 1, 0, dtype, dtype)
              for c, k in ((64, 40), (128, 72), (192, 136), (256, 64), (320, 8), (448, 128), (640, 200), (896, 72), (1664, 24))]
    channels = [ConvShape(1, 128, 13, 9, 72, 3, 3, 2, 1, dtype, dtype), ConvShape(3, 256, 5, 7, 136, 2, 2, 1, 0, dtype, dtype),
                ConvShape(1, 64, 12, 12, 40, 1, 1, 2, 0, dtype, dtype)]
    taps = [ConvShape(1, 24, 11, 10, 72, 3, 3, 1, 1, dtype, dtype), ConvShape(2, 8, 10, 9, 16, 3, 2, 1, 0, dtype, dtype)]
    _check(linear + channels + taps, 95, "residual", tile_cfg=tile_cfg, split_k=split_k)


@pytest.mark.parametrize("tile_cfg", [2, 3, 4, 5])
def test_residual_behind_a_patch_tile(tile_cfg):
    shapes = [ConvShape(5, 64, 7, 7, 72, 3, 3, 1, 1, "bf16", "bf16"), ConvShape(1, 128, 9, 28, 64, 3, 3, 1, 1, "f16", "f16"),
              ConvShape(2, 256, 5, 14, 40, 3, 3, 1, 1, "bf16", "f32"), ConvShape(1, 64, 6, 20, 33, 3, 3, 1, 1, "bf16", "bf16"),
              ConvShape(2, 128, 8, 11, 136, 3, 3, 1, 0, "f16", "f16")]
    for split_k in (1, 2):
        _check(shapes, 96, "patch residual", tile_cfg=tile_cfg, split_k=split_k)


@pytest.mark.parametrize("tile_cfg", [2, 4, 7])
def test_residual_of_other_tiles(tile_cfg):
    """fp32 outputs, any channel count, the row tile, and filter counts that take the epilogue's plain stores."""
    shapes = [ConvShape(2, 64, 9, 11, 72, 1, 1, 1, 0, "f32", "f32"), ConvShape(1, 67, 7, 9, 40, 3, 3, 1, 1, "f16", "f16"),
              ConvShape(1, 13, 9, 8, 65, 3, 3, 2, 1, "f32", "f32"), ConvShape(2, 3, 20, 32, 40, 7, 7, 2, 3, "bf16", "bf16"),
              ConvShape(1, 4, 9, 16, 24, 3, 7, 1, 3, "f16", "f32"), ConvShape(1, 64, 9, 9, 30, 1, 1, 1, 0, "f16", "f16"),
              ConvShape(1, 64, 9, 9, 20, 1, 1, 1, 0, "bf16", "f32")]
    _check(shapes, 97, "residual", tile_cfg=tile_cfg)
