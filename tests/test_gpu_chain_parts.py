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


@pytest.mark.parametrize("n_tenants,batch,parts,image,tile_cfg,split_k", [(4, 4, None, 64, 4, 2), (3, 5, 4, 64, 6, 3), (2, 5, 4, 75, 5, 2), (1, 9, 8, 75, 2, 1)])
def test_divided_chain_with_split_reductions_bitwise(n_tenants, batch, parts, image, tile_cfg, split_k):
    """Tile and split fixed, so the sums are the layer launches'; workspaces and counters per sequence, several sequences on an XCD, images
    of odd sizes, whose parts start on any element."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=n_tenants, batch=batch, image=image, seeded_weights=False, plan_opts=sc.plan_opts(tile_cfg=tile_cfg, split_k=split_k))
    stack.buf[0].uniform_(-1.0, 1.0)
    last = stack.steps[-1]
    stack.run("fused")
    torch.cuda.synchronize()
    want = stack.buf[last.dst].clone()
    stack.build_chain(0, parts)
    assert stack.chain_parts > 1 and stack.chain.info().n_queues == 8
    assert any(stack.chain.op_info(i).tile.split_k == split_k for i in range(len(stack.chain_ops)))
    for rep in range(4):
        for i, b in stack.buf.items():
            if i != 0:
                b.fill_(float("nan"))
        stack.run("fused_chain")
        torch.cuda.synchronize()
        assert torch.equal(stack.buf[last.dst], want), f"pass {rep}"
    assert not stack.chain.aborted()


@pytest.mark.parametrize("n_tenants,batch,image", [(4, 2, 128), (1, 8, 128), (6, 4, 64), (2, 8, 96)])
def test_divided_chain_with_the_planners_tiles(n_tenants, batch, image):
    """As build_chain(parts=None) plans it: other tiles and splits than the layer launches', so within the rounding of 53 bf16 layers of
    them (two summation orders drift apart by about 1 % of the output's norm), and the same bits in every pass."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=n_tenants, batch=batch, image=image, seeded_weights=False)
    stack.buf[0].uniform_(-1.0, 1.0)
    last = stack.steps[-1]
    stack.run("fused")
    torch.cuda.synchronize()
    layers = stack.buf[last.dst].float()
    stack.build_chain(parts=None)
    assert stack.chain_parts > 1
    first = None
    for rep in range(6):
        for i, b in stack.buf.items():
            if i != 0:
                b.fill_(float("nan"))
        stack.run("fused_chain")
        torch.cuda.synchronize()
        got = stack.buf[last.dst].clone()
        if first is None:
            first = got
            assert float((got.float() - layers).norm() / layers.norm()) < 2e-2
        assert torch.equal(got, first), f"pass {rep}"
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


def test_two_stacks_of_few_tenants_side_by_side():
    """Launches per stage ask nothing of what runs beside them: passes of two stacks on two streams, queued in turn, are all complete."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stacks = [ResNetStack(n_tenants=4, batch=2, image=128, seeded_weights=False) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in stacks]
    want = []
    for stack in stacks:
        stack.buf[0].uniform_(-1.0, 1.0)
        stack.run("fused")
        torch.cuda.synchronize()
        want.append(stack.buf[stack.steps[-1].dst].clone())
        stack.buf[stack.steps[-1].dst].fill_(float("nan"))
        stack.build_chain()
    torch.cuda.synchronize()
    for _ in range(20):
        for stack, stream in zip(stacks, streams):
            stack.run("fused_chain", stream)
    torch.cuda.synchronize()
    for stack, w in zip(stacks, want):
        assert torch.equal(stack.buf[stack.steps[-1].dst], w)
        assert not stack.chain.aborted()
