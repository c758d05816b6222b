"""Host-side tests of the fused list's placement when many tenants cost the same (no GPU): the list stays a permutation of
the tenant-major one, and a tenant's tiles sit on as few XCDs (launch position mod 8) as an XCD's share of the launch
allows."""
import numpy as np
import pytest

from paper_1901_00041_amd import st_conv as sc
from paper_1901_00041_amd.synth import ConvShape


def _plan(shapes, **opts):
    descs = [sc.make_desc(s.N, s.C, s.H, s.W, s.K, s.R, s.S, s.stride, s.pad, s.dtype, s.out_dtype, 0x10000, 0x20000, 0x30000) for s in shapes]
    return sc.st_conv_plan(descs, sc.plan_opts(host_only=1, **opts))


@pytest.mark.parametrize("n,split", [(7, 1), (8, 1), (9, 1), (16, 1), (21, 1), (120, 1), (9, 3), (24, 5)])
def test_alike_tenants_keep_to_few_xcds(n, split):
    shape = ConvShape(1, 128, 16, 16, 128, 3, 3, 1, 1)
    p = _plan([shape] * n, tile_cfg=4, split_k=split)
    fused, major = sc.st_conv_plan_worklist(p, 0), sc.st_conv_plan_worklist(p, 1)
    assert np.array_equal(np.sort(fused, order=["tenant", "tile_m", "tile_n", "k_split_idx"]), np.sort(major, order=["tenant", "tile_m", "tile_n", "k_split_idx"]))
    used = [len(set((np.nonzero(fused["tenant"] == t)[0] % 8).tolist())) for t in range(n)]
    if n < 8:
        assert max(used) == 8          # too few tenants to give every XCD one of its own: all are spread
    elif n % 8 == 0 and split == 1:
        assert max(used) == 1
    else:                              # uneven shares: some items move to XCDs that would have run dry
        assert np.mean(used) < 4


def test_unequal_sizes_share_evenly():
    """Configuration-3-like batches: a tenant with more tiles than an XCD's share is cut, the XCDs stay evenly loaded."""
    shapes = [ConvShape(b, 256, 14, 14, 256, 3, 3, 1, 1) for b in (2, 1, 4, 1, 1, 4, 2, 1)]
    p = _plan(shapes)
    fused = sc.st_conv_plan_worklist(p, 0)
    per_xcd = [len({(int(i["tenant"])) for i in fused[x::8]}) for x in range(8)]
    assert max(per_xcd) <= 4           # a share of 28 items holds a tenant or two, plus what was dealt over
