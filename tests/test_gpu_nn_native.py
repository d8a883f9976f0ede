"""The native autograd node of the torch layer: gradients asked for one by one, graph freed after use, non-contiguous
inputs, no graph without gradients, calls on two streams at once."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def qnn():
    import paper_2505_14669_amd.nn as nn
    return nn


def _case(seed, t=96, i=64, o=160):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return [torch.randn(s, generator=g, device=DEV).to(torch.bfloat16) for s in ((t, i), (o, i), (t, o))]


def _grads(qnn, x, w, dy, seed=9):
    x, w = x.clone().requires_grad_(True), w.clone().requires_grad_(True)
    y = qnn.QuartetLinearFunction.apply(x, w, seed, 0)
    y.backward(dy)
    return y.detach(), x.grad, w.grad


@pytest.mark.parametrize("need", [(True, False), (False, True)])
def test_one_gradient_only(qnn, need):
    x, w, dy = _case(1)
    _, dx, dw = _grads(qnn, x, w, dy)
    x, w = x.clone().requires_grad_(need[0]), w.clone().requires_grad_(need[1])
    qnn.QuartetLinearFunction.apply(x, w, 9, 0).backward(dy)
    assert (x.grad is None) == (not need[0]) and (w.grad is None) == (not need[1])
    assert torch.equal(x.grad, dx) if need[0] else torch.equal(w.grad, dw)


def test_graph_is_freed_and_absent_without_gradients(qnn):
    x, w, dy = _case(2)
    x.requires_grad_(True)
    y = qnn.QuartetLinearFunction.apply(x, w, 3, 1)
    y.backward(dy)
    with pytest.raises(RuntimeError):
        y.backward(dy)
    with torch.no_grad():
        z = qnn.QuartetLinearFunction.apply(x, w, 3, 1)
    assert z.grad_fn is None and torch.equal(z, y)


def test_non_contiguous_inputs_and_gradient(qnn):
    x, w, dy = _case(3, 128, 96, 96)
    y0, dx0, dw0 = _grads(qnn, x, w, dy)
    xt, wt = x.t().contiguous().t().requires_grad_(True), w.t().contiguous().t().requires_grad_(True)
    y = qnn.QuartetLinearFunction.apply(xt, wt, 9, 0)
    y.backward(dy.t().contiguous().t())
    assert torch.equal(y, y0) and torch.equal(xt.grad, dx0) and torch.equal(wt.grad, dw0)


def test_two_streams_do_not_share_scratch(qnn):
    cases = [_case(10 + s, 2048, 1024, 1024) for s in range(2)]
    want = [_grads(qnn, *c) for c in cases]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    got = [None, None]
    for _ in range(4):
        for s, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[s] = _grads(qnn, *cases[s])
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        assert all(torch.equal(a, b) for a, b in zip(g, w))


@pytest.mark.parametrize("which", [0, 1])
def test_forward_mode_derivatives_are_refused(qnn, which):
    # there is no forward-mode rule: a result without a tangent would be taken for a zero derivative
    import torch.autograd.forward_ad as fwad
    x, w, _ = _case(4)
    with fwad.dual_level():
        pair = [x, w]
        pair[which] = fwad.make_dual(pair[which], torch.ones_like(pair[which]))
        with pytest.raises(NotImplementedError):
            qnn.QuartetLinearFunction.apply(*pair, 9, 0)


def test_traced_layer_calls_the_function(qnn):
    # the trace holds a call of the function (it held the allocation of the result alone, so the traced layer returned whatever lay there)
    x, w, dy = _case(5)
    traced = torch.jit.trace(lambda a: qnn.QuartetLinearFunction.apply(a, w, 9, 0), x, check_trace=False)
    assert [n.kind() for n in traced.graph.nodes() if n.kind() == "aten::empty"] == []
    for seed in (6, 7):
        z = _case(seed)[0]
        assert torch.equal(traced(z), qnn.QuartetLinearFunction.apply(z, w, 9, 0))
    # and it can be differentiated
    a, b = x.clone().requires_grad_(True), x.clone().requires_grad_(True)
    traced(a).backward(dy)
    qnn.QuartetLinearFunction.apply(b, w, 9, 0).backward(dy)
    assert torch.equal(a.grad, b.grad)


def test_function_transforms_are_refused_by_name(qnn):
    x, w, _ = _case(8)
    f = lambda a, b: qnn.QuartetLinearFunction.apply(a, b, 9, 0)
    for call in (lambda: torch.vmap(lambda s: f(x, w) * s)(torch.ones(2, device=DEV)), lambda: torch.vmap(lambda a: f(a, w))(torch.stack([x, x])),
                 lambda: torch.func.grad(lambda a: f(a, w).float().sum())(x), lambda: torch.func.functionalize(f)(x, w)):
        with pytest.raises(RuntimeError, match="functorch transforms"):
            call()


def test_backward_from_several_threads_over_one_graph(qnn):
    # every thread gets the whole gradient, or the error of a graph that another thread has freed: nothing in between
    import threading
    x, w, dy = _case(12)
    _, dx, _ = _grads(qnn, x, w, dy)
    for _ in range(20):
        a = x.clone().requires_grad_(True)
        y = qnn.QuartetLinearFunction.apply(a, w, 9, 0)
        got = []

        def one():
            try:
                got.append(torch.autograd.grad(y, a, dy)[0])
            except RuntimeError as e:
                assert "second time" in str(e)
                got.append(None)
        threads = [threading.Thread(target=one) for _ in range(4)]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
        torch.cuda.synchronize()
        assert len(got) == 4 and any(g is not None for g in got) and all(g is None or torch.equal(g, dx) for g in got)


@pytest.mark.parametrize("block", [0, -32, 48, 512, 2 ** 32 + 32])
def test_hadamard_block_is_checked_before_it_is_narrowed(qnn, block):
    x, w, _ = _case(14)
    with pytest.raises(ValueError):
        qnn.QuartetLinearFunction.apply(x, w, 9, 0, block)
