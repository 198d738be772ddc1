"""What NRLogLik's backward may hand to the library as raw memory: a grad_out that
is not a plain array in memory takes the tensor operations instead.  On the CPU, with
a stand-in for the problem, whose one-launch path fails the test."""
from types import SimpleNamespace

import numpy as np
import pytest
import torch

import paper_2509_06924_amd as nr

N, ROWS = 3, (2, 4, 3)  # items, rows of each


@pytest.fixture
def setup(monkeypatch):
    gen = torch.Generator().manual_seed(1)
    f = dict(dtype=torch.float64, generator=gen)
    layers, g_rows, g_inst = torch.rand(9, 4, **f), torch.rand(9, 4, **f), torch.rand(N, 2, **f)
    problem = SimpleNamespace(
        plan=SimpleNamespace(handle=1, n_items=N), device=torch.device("cpu"), layers=layers,
        loglik_grad=lambda *a: (torch.zeros(N, dtype=torch.float64), g_rows, g_inst),
        row_item=torch.as_tensor(np.repeat(np.arange(N), ROWS)))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: None)  # the CPU's index
    calls = []

    def one_launch(problem, g_rows, g_inst, grad_out):
        calls.append(grad_out)
        return (g_rows * grad_out[problem.row_item].unsqueeze(1), g_inst[:, 0] * grad_out,
                g_inst[:, 1] * grad_out)
    monkeypatch.setattr(nr, "_scale_gradient", one_launch)
    leaves = [layers.clone().requires_grad_(), *(torch.ones(N, dtype=torch.float64).requires_grad_()
                                                 for _ in range(2))]
    ll = nr.NRLogLik.apply(*leaves, problem)

    def want(go):
        return (g_rows * go[..., problem.row_item, None], g_inst[:, 0] * go, g_inst[:, 1] * go)
    return SimpleNamespace(ll=ll, leaves=leaves, calls=calls, want=want)


GO = torch.tensor([0.5, -2.0, 3.0], dtype=torch.float64)


def _same(got, want):
    return all(torch.equal(a, b) for a, b in zip(got, want))


def test_plain_array_takes_one_launch(setup):
    got = torch.autograd.grad(setup.ll, setup.leaves, GO)
    assert len(setup.calls) == 1 and _same(got, setup.want(GO))


def test_batched(setup):
    go = torch.stack([GO, 2.0 * GO, -GO, GO.flip(0)])
    got = torch.autograd.grad(setup.ll, setup.leaves, go, is_grads_batched=True)
    assert not setup.calls and _same(got, setup.want(go))


def test_zero_tensor_without_memory(setup):
    go = torch._efficientzerotensor(N, dtype=torch.float64)
    assert go.data_ptr() == 0
    got = torch.autograd.grad(setup.ll, setup.leaves, go)
    assert not setup.calls and all(torch.count_nonzero(g) == 0 for g in got)


def test_negated_view(setup):
    # what the backward of conj() and imag() hands on: the memory holds -go
    go = torch._neg_view(GO)
    assert go.is_neg()
    got = torch.autograd.grad(setup.ll, setup.leaves, go)
    assert not setup.calls and _same(got, setup.want(-GO))


def test_forward_mode_tangent(setup):
    import torch.autograd.forward_ad as fw
    t = torch.tensor([1.0, 0.0, -4.0], dtype=torch.float64)
    with fw.dual_level():
        got = torch.autograd.grad(setup.ll, setup.leaves, fw.make_dual(GO, t))
        primal, tangent = zip(*(fw.unpack_dual(g) for g in got))
    assert not setup.calls and _same(primal, setup.want(GO)) and _same(tangent, setup.want(t))


def test_gradients_are_modified_one_by_one(monkeypatch):
    """The gradients by scale and bkg come from one launch; in-place work on one
    leaves graphs that saved the other alone."""
    monkeypatch.setattr(nr._n, "lib", lambda: SimpleNamespace(nr_scale_gradient=lambda *a: 0))
    monkeypatch.setattr(nr, "_stream", lambda stream: 0)
    problem = SimpleNamespace(plan=SimpleNamespace(handle=1, n_items=N),
                              device=torch.device("cpu"))
    g = torch.zeros(9, 4, dtype=torch.float64), torch.zeros(N, 2, dtype=torch.float64)
    _, by_scale, by_bkg = nr._scale_gradient(problem, *g, GO)
    by_scale.fill_(2.0)
    w = torch.ones(N, dtype=torch.float64, requires_grad=True)
    y = (by_scale * w).sum()
    by_bkg.mul_(3.0)
    y.backward()
    assert torch.equal(w.grad, torch.full((N,), 2.0, dtype=torch.float64))


def test_traced_backward(setup):
    """Under a dispatch mode (make_fx, operation counters) the backward consists of
    operations that the mode sees: a trace's result depends on grad_out."""
    from torch.fx.experimental.proxy_tensor import make_fx
    traced = make_fx(lambda go: torch.autograd.grad(setup.ll, setup.leaves, go,
                                                    retain_graph=True))(GO)
    assert not setup.calls and _same(traced(-3.0 * GO), setup.want(-3.0 * GO))
