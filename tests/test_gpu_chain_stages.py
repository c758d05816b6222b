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


@pytest.mark.parametrize("n_tenants,chain_queues", [(2, 0), (2, 1), (8, 0)])      # a launch per stage; persistent: one queue, columns
def test_stamps_of_every_entry(n_tenants, chain_queues):
    """Time stamps of a profiled pass: every entry, those of the max-pool too, starts and ends inside the pass on the 100 MHz
    clock, and slot 7 is time spent waiting for a dependency: none where a launch holds a single stage."""
    import numpy as np
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=n_tenants, image=64, seeded_weights=False)
    stack.build_chain(chain_queues)
    stack.run("fused_chain")
    torch.cuda.synchronize()
    chain = stack.chain
    kinds = np.array([chain.op_info(i).kind for i in range(len(stack.chain_ops))])[chain.worklist()["tenant"]]
    assert (kinds == sc.ST_OP_MAXPOOL).any()
    stamps = chain.run_profiled().astype(np.int64)
    start, end, waited = stamps[:, 4], stamps[:, 6], stamps[:, 7]
    assert (start > 0).all() and (end >= start).all() and (end.max() - start.min()) < 100_000_000      # a second
    if chain_queues == 0 and n_tenants < 8:
        assert (waited == 0).all()
    else:
        assert (waited >= 0).all() and (waited <= end.max() - start.min()).all() and waited.max() > 0
    assert not chain.aborted()


def test_persistent_launch_hooks_do_nothing_to_stage_launches():
    """The wait limit and the size of the launch are accepted and checked, and leave a pass that is a launch per stage alone."""
    import torch
    from paper_1901_00041_amd import st_conv as sc
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=2, image=64, seeded_weights=False)
    last = stack.steps[-1]
    stack.run("fused")
    torch.cuda.synchronize()
    want = stack.buf[last.dst].clone()
    stack.build_chain(0)
    chain = stack.chain
    with pytest.raises(sc.StError):
        chain.set_workgroups(chain.info().workgroups + 1)
    chain.set_workgroups(1)
    chain.set_wait_limit_us(0)
    for i, b in stack.buf.items():
        if i != 0:
            b.zero_()
    stack.run("fused_chain")
    torch.cuda.synchronize()
    n = last.shape.N * last.shape.P * last.shape.Q * last.shape.K
    assert torch.equal(stack.buf[last.dst][:, :n], want[:, :n])
    assert not chain.aborted()
