"""Planning of layers whose channel count is no multiple of the 16-byte vector (no GPU)."""
import random

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


def _random_layers(rng, n):
    out = []
    for _ in range(n):
        dtype = rng.choice(("bf16", "f16", "f32"))
        r, s = rng.choice(((1, 1), (3, 3), (5, 5), (1, 7), (2, 3)))
        epi = rng.choice((0, sc.ST_EPI_RELU, sc.ST_EPI_RESIDUAL))
        out.append((rng.randint(1, 4), rng.randint(1, 260), rng.randint(7, 40), rng.randint(7, 40), rng.randint(1, 260), r, s, rng.choice((1, 1, 2)), rng.randint(0, max(r, s) // 2),
                    dtype, rng.choice((dtype, "f32")), epi))
    return out


def _choice(plan, i, ti):
    return ti.tile_cfg, ti.split_k, ti.rows_per_tile, sc.st_conv_plan_tenant_form(plan, i), ti.k_steps, ti.k_steps_per_split


@pytest.mark.parametrize("seed", range(12))
def test_a_layer_planned_alone_on_its_tile_and_split_takes_the_same_form(seed):
    rng = random.Random(seed)
    layers = _random_layers(rng, rng.randint(2, 40))
    plan, infos = _plan(layers)
    for i, (layer, ti) in enumerate(zip(layers, infos)):
        alone, (ta,) = _plan([layer], tile_cfg=ti.tile_cfg + 1, split_k=ti.split_k, rows_per_tile=ti.rows_per_tile)
        assert _choice(plan, i, ti) == _choice(alone, 0, ta), layer


@pytest.mark.parametrize("layer", [(1, 5, 16, 16, 64, 5, 5, 1, 2, "f32"), (1, 6, 16, 16, 64, 3, 3, 1, 1, "f32"), (1, 9, 16, 16, 64, 3, 3, 1, 1, "bf16"),
                                   (1, 243, 16, 16, 64, 1, 1, 1, 0, "f16")])
@pytest.mark.parametrize("tile_cfg", [2, 4, 5, 6])
def test_company_does_not_change_the_form(layer, tile_cfg):
    alone, (ta,) = _plan([layer], tile_cfg=tile_cfg, split_k=1)
    many, infos = _plan([layer] * 200, tile_cfg=tile_cfg, split_k=1)
    assert _choice(alone, 0, ta) == _choice(many, 0, infos[0])


def test_forms_are_reported():
    plan, _ = _plan([(1, 64, 14, 14, 64, 1, 1, 1, 0, "bf16"), (1, 64, 14, 14, 64, 3, 3, 1, 1, "bf16"), (1, 67, 14, 14, 64, 3, 3, 1, 1, "bf16"),
                     (1, 7, 14, 14, 64, 3, 3, 1, 1, "bf16"), (1, 5, 14, 14, 64, 3, 3, 1, 1, "f32")], tile_cfg=4, split_k=1)
    assert [sc.st_conv_plan_tenant_form(plan, i) for i in range(5)] == [sc.ST_FORM_VECTORS, sc.ST_FORM_PATCH, sc.ST_FORM_PIECES, sc.ST_FORM_GATHERED, sc.ST_FORM_GATHERED]
    plan, _ = _plan([(1, 3, 224, 224, 64, 7, 7, 2, 3, "bf16")])
    assert sc.st_conv_plan_tenant_form(plan, 0) == sc.ST_FORM_ROWS
    with pytest.raises(sc.StError):
        sc.st_conv_plan_tenant_form(plan, 1)


def _steps(c, window, dtype, kb):
    """K steps of whole vectors and of left-over channels, from the layout of the reduction index."""
    es = 4 if dtype == "f32" else 2
    vec = 16 // es
    taps = window[0] * window[1]
    return -(-taps * (c // vec * vec) * es // kb), -(-taps * 16 // kb)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("c,window", [(9, (5, 5)), (61, (1, 1)), (125, (1, 1)), (67, (3, 3)), (243, (3, 3)), (13, (7, 7))])
@pytest.mark.parametrize("tile_cfg", [2, 4, 5, 6])
@pytest.mark.parametrize("split", [1, 2, 3, 5])
def test_steps_and_slices_are_the_kernels_own(dtype, c, window, tile_cfg, split):
    plan, (ti,) = _plan([(1, c, 16, 16, 64, window[0], window[1], 1, window[0] // 2, dtype)], tile_cfg=tile_cfg, split_k=split)
    assert sc.st_conv_plan_tenant_form(plan, 0) == sc.ST_FORM_PIECES
    main, left = _steps(c, window, dtype, sc.st_tile_shape(ti.tile_cfg)[2])
    assert ti.k_steps == main + left
    assert ti.k_steps_per_split == -(-ti.k_steps // ti.split_k) and (ti.split_k - 1) * ti.k_steps_per_split < ti.k_steps
    assert ti.split_k <= split


def test_slices_of_left_over_channels_start_first():
    """Nine channels, 5x5: four steps of whole vectors, then four of the channel left over, which take longer."""
    layer = (1, 9, 32, 32, 64, 5, 5, 1, 2, "bf16")
    plan, (ti,) = _plan([layer], tile_cfg=4, split_k=2)
    assert (ti.k_steps, ti.k_steps_per_split) == (8, 4)
    slices = sc.st_conv_plan_worklist(plan, 0)["k_split_idx"].tolist()
    assert slices == sorted(slices, reverse=True)
    plan, (ti,) = _plan([layer], tile_cfg=4, split_k=4)         # two of each
    slices = sc.st_conv_plan_worklist(plan, 0)["k_split_idx"].tolist()
    assert sorted(slices[:len(slices) // 2]) == [2] * ti.tiles_m + [3] * ti.tiles_m


def test_stores_by_element_are_priced():
    """Among small layers, 1x1 with 251 filters and a residual: its rows are no whole vectors, and a 128x128 tile spends 27500 clocks
    storing them, twice what any other work item of the launch takes in all."""
    R = sc.ST_EPI_RESIDUAL
    layers = [(2, 145, 20, 35, 32, 3, 3, 1, 1, "bf16", "bf16", R), (4, 120, 5, 40, 251, 1, 1, 3, 0, "f16", "f16", R), (1, 91, 7, 30, 25, 1, 7, 1, 3, "f32", "f32", R),
              (4, 8, 5, 34, 96, 3, 3, 1, 1, "bf16", "bf16", R), (3, 92, 32, 13, 109, 5, 5, 1, 1, "f16", "f32", R), (1, 160, 23, 18, 214, 1, 1, 3, 0, "f32", "f32", R)]
    _, infos = _plan(layers)
    assert infos[1].MT * infos[1].NT <= 64 * 64
    assert infos[5].MT * infos[5].NT <= 32 * 64


def test_steps_of_pieces_are_priced():
    """226 channels, 3x3: beside a second workgroup a 128x64 step takes twice what it takes with a multiple of 64 channels.  Unsplit on
    that tile this layer ran 83000 clocks, half as long again as anything else in its launch."""
    layers = [(1, 128, 31, 26, 45, 3, 3, 3, 0, "bf16", "f32"), (4, 226, 11, 39, 72, 3, 3, 3, 1, "f16", "f16"), (4, 120, 16, 17, 222, 3, 3, 1, 1, "f32", "f32"),
              (2, 152, 23, 37, 50, 5, 5, 1, 1, "f32", "f32"), (4, 199, 28, 11, 1, 3, 3, 1, 0, "f32", "f32"), (2, 112, 9, 25, 56, 5, 5, 2, 2, "f32", "f32"),
              (4, 184, 36, 40, 32, 3, 3, 1, 0, "f16", "f32"), (3, 72, 28, 10, 197, 3, 3, 1, 0, "f16", "f32")]
    plan, infos = _plan(layers)
    assert sc.st_conv_plan_tenant_form(plan, 1) == sc.ST_FORM_PIECES
    assert infos[1].MT * infos[1].NT // infos[1].split_k <= 64 * 64


def test_stores_by_element_are_priced_by_what_is_stored():
    """67 filters fill half of a 128-filter tile: 2156 items of 32x64 ran a fifth longer than 539 of 128x64.  And fp32 results with a
    residual cost more on 64x128 tiles than on 128x64 (39000 clocks, 32500): 227 us and 182."""
    _, infos = _plan([(4, 208, 28, 28, 67, 1, 1, 1, 0, "bf16", "bf16", sc.ST_EPI_RELU)] * 11)
    assert infos[0].MT * infos[0].NT >= 128 * 64
    _, infos = _plan([(3, 64, 56, 56, 469, 3, 3, 1, 1, "bf16", "f32", sc.ST_EPI_RELU | sc.ST_EPI_RESIDUAL)] * 7)
    assert (infos[0].MT, infos[0].NT) == (128, 64)
