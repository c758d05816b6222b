"""Launches of tenants with one layer shape are planned in whole rounds of workgroup slots (no GPU)."""
import pytest

from paper_1901_00041_amd import st_conv as sc

FAKE = 1 << 32


def _plan(shapes, **opts):
    descs = [sc.make_desc(*s, "f32", "f32", FAKE * (3 * i + 1), FAKE * (3 * i + 2), FAKE * (3 * i + 3)) for i, s in enumerate(shapes)]
    plan = sc.st_conv_plan(descs, sc.plan_opts(host_only=1, **opts))
    return plan, [sc.st_conv_plan_tenant_info(plan, i) for i in range(len(shapes))]


CONV = (1, 128, 16, 16, 128, 3, 3, 1, 1)


@pytest.mark.parametrize("tenants", [1, 2, 5, 20, 48, 90])
def test_alike_tenants_get_one_choice_and_no_small_second_round(tenants):
    plan, infos = _plan([CONV] * tenants)
    assert len({(t.tile_cfg, t.split_k) for t in infos}) == 1
    items = int(sc.st_conv_plan_info(plan).n_items)
    assert items == sum(t.item_count for t in infos)
    if tenants == 20:
        assert items <= 512          # 640 items of the smallest tile would leave a quarter of a second round


def test_a_callers_share_and_unlike_tenants_are_planned_as_before():
    for opts in ({"target_items": 300}, {"tile_cfg": 6, "split_k": 1}):
        _, infos = _plan([CONV] * 20, **opts)
        assert len({(t.tile_cfg, t.split_k) for t in infos}) == 1
    assert _plan([CONV] * 20, tile_cfg=6, split_k=1)[1][0].tile_cfg == 5
    _, infos = _plan([CONV] * 19 + [(1, 128, 16, 15, 128, 3, 3, 1, 1)])
    assert infos[0].tile_cfg == 5 and infos[0].split_k == 1
