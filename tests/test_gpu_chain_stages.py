"""Chains of fewer than 8 sequences run as one launch per stage unless a persistent launch is asked for: same bits either
way, and as the layer-by-layer launches."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tenants,batch", [(1, 1), (3, 2), (7, 1)])
def test_stage_launches_match_layer_launches_bitwise(n_tenants, batch):
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=n_tenants, batch=batch, image=64, seeded_weights=False)
    last = stack.steps[-1]
    stack.run("fused")
    torch.cuda.synchronize()
    want = stack.buf[last.dst].clone()
    assert float(want.float().abs().max()) > 0
    for chain_queues in (0, 1):
        stack.build_chain(chain_queues)
        assert stack.chain.info().n_queues == 1
        for rep in range(3):
            for i, b in stack.buf.items():
                if i != 0:
                    b.zero_()
            stack.run("fused_chain")
            torch.cuda.synchronize()
            n = last.shape.N * last.shape.P * last.shape.Q * last.shape.K
            assert torch.equal(stack.buf[last.dst][:, :n], want[:, :n]), f"chain_queues={chain_queues} pass {rep}"
        assert not stack.chain.aborted()
    stamps = stack.chain.run_profiled()
    assert (stamps[:, 6] > 0).all()
