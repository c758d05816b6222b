"""Passes of the persistent chain that give up: what st_chain_aborted says of them, and the limits of a wait.  Every kernel here exits
by itself: a wait that ends early, or a column that nobody works through, only leaves its pass incomplete."""
import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu


def _stack(chain_queues):
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=8, seeded_weights=False)
    stack.run("fused")
    torch.cuda.synchronize()
    want = stack.buf[stack.steps[-1].dst].clone()
    stack.build_chain(chain_queues)
    return stack, want


def _right_again(stack, want, passes=2):
    import torch
    for _ in range(passes):
        for i, b in stack.buf.items():
            if i != 0:
                b.zero_()
        stack.run("fused_chain")
        torch.cuda.synchronize()
        assert torch.equal(stack.buf[stack.steps[-1].dst], want)
    assert not stack.chain.aborted()


@pytest.mark.parametrize("chain_queues", [0, 1])
@pytest.mark.parametrize("later", [1, 2, 3])              # runs that use either of the two control blocks, or both
def test_an_abandoned_pass_is_reported_after_later_passes(chain_queues, later):
    import torch
    stack, want = _stack(chain_queues)
    chain = stack.chain
    chain.set_wait_limit_us(0)
    stack.run("fused_chain")
    chain.set_wait_limit_us(100000)
    for _ in range(later):
        stack.run("fused_chain")
    torch.cuda.synchronize()
    assert chain.aborted()
    assert not chain.aborted()                            # reported once
    _right_again(stack, want)


@pytest.mark.parametrize("later", [0, 1, 2])
def test_an_incomplete_pass_without_waits_is_reported_after_later_passes(later):
    """One stage, so nothing waits and nothing gives up; with one workgroup all columns but one stay undone."""
    import torch
    from tests import helpers
    from paper_1901_00041_amd import synth
    s = synth.ConvShape(1, 64, 24, 24, 64, 3, 3, 1, 1, "bf16", "bf16")
    tenants = [helpers.Tenant(s, synth.gen_input(96, t, 0, s), synth.gen_weight(96, t, 0, s)) for t in range(8)]
    chain = sc.Chain([sc.make_chain_op(sc.ST_OP_CONV, t, 0, ten.desc()) for t, ten in enumerate(tenants)], None, keep=tenants)
    assert chain.info().n_queues == 8
    chain.set_workgroups(1)
    chain.run()
    chain.set_workgroups(0)
    for _ in range(later):
        chain.run()
    assert chain.aborted()
    assert not chain.aborted()
    for t in tenants:
        t.clear()
    chain.run()
    torch.cuda.synchronize()
    for i, t in enumerate(tenants):
        helpers.check_tenant(t, f"tenant {i}")
    assert not chain.aborted()


def test_a_wait_lasts_as_long_as_its_limit():
    """The count of looks that also bounds a wait is far above what fits into the limit: with one workgroup per compute unit nobody
    draws the shared columns, and their dependants wait for the whole limit."""
    import time
    import torch
    stack, want = _stack(0)
    chain = stack.chain
    assert chain.info().workgroups == 512
    chain.set_workgroups(256)
    chain.set_wait_limit_us(2_000_000)
    torch.cuda.synchronize()
    t0 = time.monotonic()
    stack.run("fused_chain")
    torch.cuda.synchronize()
    assert 2.0 <= time.monotonic() - t0 < 10.0
    assert chain.aborted()
    chain.set_workgroups(0)
    chain.set_wait_limit_us(100000)
    _right_again(stack, want)
