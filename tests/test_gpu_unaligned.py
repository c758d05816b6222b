"""Tensors whose addresses are multiples of the element size and of nothing more: views into a caller's larger buffer."""
import pytest

from paper_1901_00041_amd import synth
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


def _shifted(t, elements):
    """The values of t in a contiguous tensor that starts `elements` elements into its allocation."""
    import torch
    flat = torch.empty(t.numel() + elements, dtype=t.dtype, device=t.device)
    view = flat[elements:].view(t.shape)
    view.copy_(t)
    assert view.data_ptr() % 16 == (elements * t.element_size()) % 16
    return view


def _gather_shapes(dtype):
    return [ConvShape(1, 7, 9, 9, 70, 3, 3, 1, 1, dtype, "f32"), ConvShape(3, 67, 5, 7, 33, 3, 3, 2, 1, dtype, "f32"),
            ConvShape(1, 131, 6, 6, 65, 1, 1, 1, 0, dtype, "f32"), ConvShape(1, 239, 4, 5, 16, 5, 5, 3, 2, dtype, dtype)]


@pytest.mark.parametrize("elements", [1, 2, 3])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_any_channel_count_unaligned(dtype, elements):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    for tile_cfg in (2, 4):
        tenants = [helpers.Tenant(s, synth.gen_input(93, t, 0, s), synth.gen_weight(93, t, 0, s)) for t, s in enumerate(_gather_shapes(dtype))]
        for i, t in enumerate(tenants):
            t.dx, t.dw, t.dy = _shifted(t.dx, elements), _shifted(t.dw, elements + i), _shifted(t.dy, elements)
        plan = helpers.plan_for(tenants, tile_cfg=tile_cfg)
        sc.st_conv_run(plan)
        torch.cuda.synchronize()
        for i, t in enumerate(tenants):
            helpers.check_tenant(t, f"unaligned[{i}] {t.shape} tile_cfg={tile_cfg}")


def _vector_shapes(dtype):
    """Every other kind of tile: 1x1, taps of a strided 3x3, the input patch in LDS, any walk, the row tile, plain stores."""
    out = [ConvShape(2, 64, 9, 11, 72, 1, 1, 1, 0, dtype, dtype), ConvShape(1, 256, 13, 9, 40, 3, 3, 2, 1, dtype, "f32"),
           ConvShape(3, 128, 7, 7, 72, 3, 3, 1, 1, dtype, dtype), ConvShape(1, 24, 11, 10, 72, 3, 3, 1, 1, dtype, "f32"),
           ConvShape(1, 64, 9, 9, 36, 1, 1, 1, 0, dtype, dtype), ConvShape(1, 64, 9, 9, 33, 1, 1, 1, 0, dtype, "f32")]
    return out if dtype == "f32" else out + [ConvShape(2, 3, 20, 32, 40, 7, 7, 2, 3, dtype, dtype)]


@pytest.mark.parametrize("elements", [2, 1])
@pytest.mark.parametrize("dtype", ["bf16", "f16", "f32"])
def test_vector_channel_count_unaligned(dtype, elements):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    for tile_cfg in (0, 1, 4, 6):
        tenants = []
        for t, s in enumerate(_vector_shapes(dtype)):
            res = synth.to_storage(synth.uniform_pm1(synth.stream_state(93, t, 0, 3), s.N * s.K * s.P * s.Q), s.out_dtype)
            tenants.append(helpers.Tenant(s, synth.gen_input(93, t, 0, s), synth.gen_weight(93, t, 0, s), residual=res.reshape(s.N, s.K, s.P, s.Q)))
        for i, t in enumerate(tenants):
            t.dx, t.dw, t.dy, t.dres = _shifted(t.dx, elements), _shifted(t.dw, elements + i), _shifted(t.dy, elements), _shifted(t.dres, elements)
        plan = helpers.plan_for(tenants, tile_cfg=tile_cfg)
        sc.st_conv_run(plan)
        torch.cuda.synchronize()
        for i, t in enumerate(tenants):
            helpers.check_tenant(t, f"unaligned[{i}] {t.shape} tile_cfg={tile_cfg}")
