"""New pointers for all of a plan's tenants: counts around the sizes in which the pointers travel."""
import pytest

from paper_1901_00041_amd import synth
from paper_1901_00041_amd.synth import ConvShape

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 17, 112, 113, 230])
def test_rebind_all_counts(n):
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from tests import helpers
    s = ConvShape(1, 8, 3, 4, 8, 1, 1, 1, 0, "bf16", "f32")
    made = [[helpers.Tenant(s, synth.gen_input(94 + b, t, 0, s), synth.gen_weight(94 + b, t, 0, s)) for t in range(n)] for b in range(2)]
    plan = helpers.plan_for(made[0])
    for tenants in (made[1], made[0]):
        sc.st_conv_plan_rebind_all(plan, [t.desc() for t in tenants], torch.cuda.current_stream(), keep=[t for b in made for t in b])
        sc.st_conv_run(plan, torch.cuda.current_stream())
        torch.cuda.synchronize()
        for i, t in enumerate(tenants):
            helpers.check_tenant(t, f"tenant {i} of {n}")
            t.clear()
