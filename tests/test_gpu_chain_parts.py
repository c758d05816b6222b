"""A chain whose tenants' batches are divided into sequences of their own."""
import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_tenants,batch,parts", [(4, 2, None), (1, 8, None), (3, 4, None), (5, 3, 2), (2, 5, 4), (8, 3, 2)])      # even and uneven parts, 1 to 3 sequences on an XCD
def test_divided_chain_matches_layer_launches_bitwise(n_tenants, batch, parts):
    """With the tile shape fixed every output is summed in the same order however the images are grouped, so the network's
    output is bitwise the layer launches'; parts that touched each other's images would differ.  Many passes in a row: the parts of one
    pass drift apart in depth."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=n_tenants, batch=batch, image=64, seeded_weights=False, plan_opts=sc.plan_opts(tile_cfg=4, split_k=1))
    stack.buf[0].uniform_(-1.0, 1.0)
    last = stack.steps[-1]
    stack.run("fused")
    torch.cuda.synchronize()
    want = stack.buf[last.dst].clone()
    assert want.numel() == n_tenants * batch * last.shape.P * last.shape.Q * last.shape.K and float(want.float().abs().max()) > 0
    stack.build_chain(0, parts)
    assert stack.chain_parts > 1 and stack.chain.info().n_queues == 8 and stack.chain.info().n_sequences == n_tenants * stack.chain_parts
    for rep in range(5):
        for i, b in stack.buf.items():
            if i != 0:
                b.fill_(float("nan"))
        for _ in range(6):
            stack.run("fused_chain")
        torch.cuda.synchronize()
        assert torch.equal(stack.buf[last.dst], want), f"round {rep}"
    assert not stack.chain.aborted()


@pytest.mark.parametrize("n_tenants,batch", [(4, 2), (1, 8), (6, 4)])
def test_nothing_is_divided_unasked(n_tenants, batch):
    """Fewer than eight tenants stay a launch per stage, which asks for no co-residency, in the order of sums of the layer launches,
    with the planner's own tiles and splits."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack, chain_parts
    stack = ResNetStack(n_tenants=n_tenants, batch=batch, image=64, seeded_weights=False)
    assert chain_parts(n_tenants, batch, 64) > 1
    stack.buf[0].uniform_(-1.0, 1.0)
    last = stack.steps[-1]
    stack.run("fused")
    torch.cuda.synchronize()
    want = stack.buf[last.dst].clone()
    for i, b in stack.buf.items():
        if i != 0:
            b.fill_(float("nan"))
    stack.run("fused_chain")          # builds the chain
    info = stack.chain.info()
    assert info.n_queues == 1 and info.n_sequences == n_tenants and stack.chain_parts == 1
    assert {o.sequence for o in stack.chain_ops} == set(range(n_tenants))
    stack.chain.set_wait_limit_us(0)          # nothing waits inside a launch
    stack.run("fused_chain")
    torch.cuda.synchronize()
    assert torch.equal(stack.buf[last.dst], want)
    assert not stack.chain.aborted()


def test_divided_chain_in_a_graph():
    """A captured pass of a divided chain can be replayed."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=4, batch=2, image=64, seeded_weights=False, plan_opts=sc.plan_opts(tile_cfg=4, split_k=1))
    stack.build_chain(parts=None)
    assert stack.chain_parts == 2
    last = stack.steps[-1]
    stack.run("fused_chain", torch.cuda.current_stream())
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        stack.run("fused_chain", torch.cuda.current_stream())
    for rep in range(3):
        stack.buf[0].uniform_(-1.0, 1.0)
        stack.run("fused_chain", torch.cuda.current_stream())
        torch.cuda.synchronize()
        want = stack.buf[last.dst].clone()
        stack.buf[last.dst].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(stack.buf[last.dst], want), f"replay {rep}"
    assert not stack.chain.aborted()
