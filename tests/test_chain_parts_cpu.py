"""How many sequences a tenant's batch is divided into for a chain."""
import pytest

from paper_1901_00041_amd.stack import XCDS, _share, chain_parts


@pytest.mark.parametrize("image", [64, 128, 224])
@pytest.mark.parametrize("n_tenants", [1, 2, 3, 5, 7, 8, 12])
def test_parts_fill_the_xcds_and_hold_every_image(n_tenants, image):
    for batch in list(range(1, 18)) + [64]:
        k = chain_parts(n_tenants, batch, image)
        share = _share(batch, k)
        assert sum(share) == batch and min(share) >= 1 and max(share) - min(share) <= 1
        if k > 1:
            assert XCDS <= n_tenants * k <= 4 * XCDS and n_tenants < XCDS
            load = [sum(share[s // n_tenants] for s in range(x, n_tenants * k, XCDS)) for x in range(XCDS)]
            assert max(load) * XCDS <= 1.5 * n_tenants * batch
    assert chain_parts(n_tenants, 1, image) == 1


def test_whole_where_whole_is_faster():
    assert [chain_parts(8, b) for b in (1, 2, 8)] == [1, 1, 1]
    assert chain_parts(2, 5) == 1 and chain_parts(3, 3) == 1 and chain_parts(3, 2) == 1
    assert chain_parts(4, 4) == 2 and chain_parts(1, 8) == 8 and chain_parts(6, 4, 224) == 4 and chain_parts(6, 4, 128) == 2
