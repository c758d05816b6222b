"""The row tile over its filter shapes: filter rows of one and of two half steps, full and with a tail, seven rows (held in
registers) and other numbers of them (read again for every output row), as a layer launch and in a chain laid out per XCD.  An
infinite input reaches the outputs whose window holds it and no others."""
import numpy as np
import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("R,S,C", [(7, 7, 3), (7, 4, 4), (7, 5, 3), (7, 8, 4), (7, 9, 1), (3, 3, 3), (5, 7, 4), (8, 7, 3), (2, 8, 1)])
def test_filter_shapes(R, S, C, dtype):
    import torch
    import torch.nn.functional as F
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[dtype]
    N, H, W, K, stride, pad = 2, 21, 144, 72, 4 if C == 1 else 2, min(R, S) // 2
    gen = torch.Generator().manual_seed(R * 100 + S * 10 + C)
    x = (torch.rand((N, H, W, C), generator=gen) * 2 - 1).to(dt)
    w = (torch.randn((K, R, S, C), generator=gen) * (1.0 / (R * S * C)) ** 0.5).to(dt)
    x[1, 2 * stride - pad + R // 2, 17 * stride - pad + S // 2, 0] = float("inf")       # inside the window of output (2, 17)
    ref = F.conv2d(x.double().permute(0, 3, 1, 2), w.double().permute(0, 3, 1, 2), stride=stride, padding=pad).permute(0, 2, 3, 1)
    # the reference multiplies the padding, too, but only an input that is there can be infinite
    P, Q = ref.shape[1:3]
    dx, dw = x.cuda(), w.cuda()
    for form in ("launch", "chain"):
        y = torch.full((N, P, Q, K), float("nan"), dtype=dt, device="cuda")
        d = sc.make_desc(N, C, H, W, K, R, S, stride, pad, dtype, dtype, dx, dw, y)
        if form == "launch":
            plan = sc.st_conv_plan([d], sc.plan_opts(tile_cfg=7), keep=[dx, dw, y])
            assert sc.st_conv_plan_tenant_info(plan, 0).row_tiled == 1
            sc.st_conv_run(plan)
        else:
            chain = sc.Chain([sc.make_chain_op(sc.ST_OP_CONV, 0, 0, d)], sc.plan_opts(tile_cfg=7, chain_queues=2), keep=[dx, dw, y])
            chain.run()
        torch.cuda.synchronize()
        got = y.cpu().double()
        fin = torch.isfinite(ref)
        assert torch.equal(torch.isfinite(got), fin), form
        assert 0 < int((~fin).sum()) < fin.numel()
        # the output's rounding (2^-9, 2^-12 of it) and fp32 sums of R*S*C products of at most 1
        tol = ref.abs() * (2.0 ** -8 if dtype == "bf16" else 2.0 ** -10) + R * S * C * 2.0 ** -22
        assert ((got - ref).abs() <= tol)[fin].all(), form
