"""The backward pass of NRLogLik through nr_scale_gradient: every layout of
grad_out, and the ways round it (a graph of the backward, a closed plan), give
the tensor operations' values bit for bit (one product per entry)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def setup():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    from paper_2509_06924_amd import inputs
    batch = inputs.random_batch(np.random.default_rng(3), n_items=7, L_choices=[0, 1, 5, 21],
                                nq_choices=[20, 70], dqq_choices=[0.05, 0.0])
    prob = nr.Problem.from_batch(batch)
    row_item = torch.as_tensor(np.repeat(np.arange(7), np.diff(batch.row_off)), device="cuda")
    return torch, nr, prob, row_item


def _leaves(prob):
    return [t.clone().requires_grad_() for t in (prob.layers, prob.scale, prob.bkg)]


@pytest.mark.parametrize("form", ["ones", "expanded", "strided", "reversed", "graph"])
def test_backward_layouts(setup, form):
    torch, nr, prob, row_item = setup
    _, g_rows, g_inst = prob.loglik_grad()
    x = _leaves(prob)
    ll = nr.NRLogLik.apply(*x, prob)
    base = torch.linspace(-2.0, 3.0, 14, dtype=torch.float64, device="cuda")
    go = {"ones": torch.ones(7, dtype=torch.float64, device="cuda"), "expanded": base[3].expand(7),
          "strided": base[::2], "reversed": base[:7].flip(0), "graph": base[:7].clone()}[form]
    if form == "graph":
        go.requires_grad_()
        got = torch.autograd.grad(ll, x, go, create_graph=True)
        (back,) = torch.autograd.grad(got[1].sum(), go)  # d(sum_b go_b g_b)/d go
        assert torch.equal(back, g_inst[:, 0])
    else:
        got = torch.autograd.grad(ll, x, go)
    go = go.detach()
    assert torch.equal(got[0], g_rows * go[row_item].unsqueeze(1))
    assert torch.equal(got[1], g_inst[:, 0] * go) and torch.equal(got[2], g_inst[:, 1] * go)


def test_plan_closed_before_backward(setup):
    torch, nr, _, _ = setup
    from paper_2509_06924_amd import inputs
    batch = inputs.random_batch(np.random.default_rng(4), n_items=2, L_choices=[3],
                                nq_choices=[20], dqq_choices=[0.05])
    prob = nr.Problem.from_batch(batch)
    x = _leaves(prob)
    _, g_rows, _ = prob.loglik_grad()
    ll = nr.NRLogLik.apply(*x, prob)
    prob.plan.close()
    got = torch.autograd.grad(2.0 * ll.sum(), x)
    assert torch.equal(got[0], 2.0 * g_rows)
