"""Planning of layers whose channel count is no multiple of the 16-byte vector (no GPU)."""
import pytest

from paper_1901_00041_amd import st_conv as sc

FAKE = 1 << 32


def _plan(layers, **opts):
    """layers: (N, C, H, W, K, R, S, stride, pad, dtype[, out[, epilogue]])"""
    descs = []
    for i, s in enumerate(layers):
        epi = s[11] if len(s) > 11 else 0
        descs.append(sc.make_desc(*s[:9], s[9], s[10] if len(s) > 10 else s[9], FAKE * (4 * i + 1), FAKE * (4 * i + 2), FAKE * (4 * i + 3),
                                  FAKE * (4 * i + 4) if epi & sc.ST_EPI_RESIDUAL else None, epi))
    plan = sc.st_conv_plan(descs, sc.plan_opts(host_only=1, **opts))
    return plan, [sc.st_conv_plan_tenant_info(plan, i) for i in range(len(layers))]


# a vector of fp32 channels is four, of 16-bit channels eight
@pytest.mark.parametrize("dtype,channels", [("bf16", (9, 61, 126, 243)), ("f16", (15, 130)), ("f32", (6, 9, 126, 243))])
@pytest.mark.parametrize("tile_cfg", [2, 4, 5, 6])
def test_a_forced_shape_is_the_shape(dtype, channels, tile_cfg):
    for c in channels:
        for window in ((1, 1, 0), (3, 3, 1), (5, 5, 2)):
            _, (ti,) = _plan([(2, c, 14, 14, 70, window[0], window[1], 1, window[2], dtype)], tile_cfg=tile_cfg)
            assert ti.tile_cfg == tile_cfg - 1, (c, window)


@pytest.mark.parametrize("dtype,channels", [("bf16", 126), ("f32", 126), ("bf16", 7), ("f32", 3)])
def test_a_forced_shape_that_such_layers_do_not_have_is_the_nearest_one(dtype, channels):
    # 128x128 and the row tile become 128x64, 64x128 becomes 64x64; with fewer channels than a vector, so do 32x64 and 16x64
    narrow = channels < 8
    for tile_cfg, want in [(1, 1), (3, 3), (7, 1)] + ([(5, 3), (6, 3)] if narrow else []):
        _, (ti,) = _plan([(2, channels, 14, 13, 70, 3, 3, 1, 1, dtype)], tile_cfg=tile_cfg)
        assert ti.tile_cfg == want, tile_cfg
