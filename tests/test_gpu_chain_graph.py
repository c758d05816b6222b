"""Chains in graphs: a captured pass can be replayed any number of times, in a row and between other passes of the chain, whatever
stream it was captured on, and leaves the passes that are not captured alone."""
import contextlib
import ctypes

import pytest

from paper_1901_00041_amd import st_conv as sc

pytestmark = pytest.mark.gpu

# tenants, batch, chain_queues, parts: columns per XCD, one queue, a launch per stage, and a divided batch
FORMS = [(8, 1, 0, 1), (8, 1, 1, 1), (3, 1, 0, 1), (4, 2, 0, None), (2, 1, 1, 1)]


@contextlib.contextmanager
def _raw_graph(queue_work):
    """queue_work(stream) captured on a stream of the runtime's that torch knows nothing of; yields a call that replays it there."""
    hip = sc.lib()              # the library's own runtime: its handle resolves the symbols of its dependencies too
    stream, graph, ready = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(stream)) == 0
    assert hip.hipStreamBeginCapture(stream, 2) == 0
    try:
        queue_work(stream.value)
    finally:
        ended = hip.hipStreamEndCapture(stream, ctypes.byref(graph))
    assert ended == 0
    assert hip.hipGraphInstantiate(ctypes.byref(ready), graph, None, None, ctypes.c_size_t(0)) == 0

    def replay():
        assert hip.hipGraphLaunch(ready, stream) == 0 and hip.hipStreamSynchronize(stream) == 0
    try:
        yield replay
    finally:
        assert hip.hipGraphExecDestroy(ready) == 0 and hip.hipGraphDestroy(graph) == 0 and hip.hipStreamDestroy(stream) == 0


def _stack(n_tenants, batch, chain_queues, parts):
    """A stack with its chain, four inputs, and the network's outputs for them by passes that are not captured."""
    import torch
    from paper_1901_00041_amd.stack import ResNetStack
    stack = ResNetStack(n_tenants=n_tenants, batch=batch, image=64, seeded_weights=False)
    stack.build_chain(chain_queues, parts)
    inputs = [torch.empty_like(stack.buf[0]).uniform_(-1.0, 1.0) for _ in range(4)]
    want = []
    for x in inputs:
        stack.buf[0].copy_(x)
        stack.run("fused_chain")
        torch.cuda.synchronize()
        want.append(stack.buf[stack.steps[-1].dst].clone())
    assert not stack.chain.aborted() and not torch.equal(want[0], want[1])
    return stack, inputs, want


def _pass(stack, x, want, run, what):
    import torch
    for i, b in stack.buf.items():
        if i != 0:
            b.fill_(float("nan"))
    stack.buf[0].copy_(x)
    torch.cuda.synchronize()
    run()
    torch.cuda.synchronize()
    assert torch.equal(stack.buf[stack.steps[-1].dst], want), what


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("through", ["stack", "chain"])
def test_replays_of_a_captured_pass(form, through):
    stack, inputs, want = _stack(*form)
    eager = lambda: stack.run("fused_chain")          # noqa: E731
    queue_work = (lambda s: stack.run("fused_chain", s)) if through == "stack" else stack.chain.run
    with _raw_graph(queue_work) as replay:
        # capturing queued nothing: the passes after it are right
        for i in range(2):
            _pass(stack, inputs[i], want[i], eager, f"pass {i} after the capture")
        for i in range(4):
            _pass(stack, inputs[i], want[i], replay, f"replay {i} in a row")
        for i, run in enumerate((eager, replay, eager, eager, replay, replay, eager)):
            _pass(stack, inputs[i % 4], want[i % 4], run, f"mixed {i}")
        assert not stack.chain.aborted()
        _pass(stack, inputs[3], want[3], replay, "replay after a look at the chain's state")
    assert not stack.chain.aborted()


def test_two_passes_in_one_graph_on_the_current_stream():
    import torch
    stack, inputs, want = _stack(8, 1, 0, 1)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(2):
            stack.run("fused_chain", torch.cuda.current_stream())
    for i in range(3):
        _pass(stack, inputs[i], want[i], graph.replay, f"replay {i}")
        _pass(stack, inputs[i + 1], want[i + 1], lambda: stack.run("fused_chain"), f"pass {i}")
    assert not stack.chain.aborted()


def test_an_abandoned_replay_is_reported():
    """Captured with a wait limit of nothing, a pass gives up at its first dependency that is not complete yet; passes that are not
    captured are right again."""
    stack, inputs, want = _stack(8, 1, 0, 1)
    stack.chain.set_wait_limit_us(0)
    with _raw_graph(stack.chain.run) as replay:
        stack.chain.set_wait_limit_us(100000)
        replay()
        assert stack.chain.aborted() and not stack.chain.aborted()
        for i in range(3):
            _pass(stack, inputs[i], want[i], lambda: stack.run("fused_chain"), f"pass {i}")
    assert not stack.chain.aborted()
