"""Smallest smeared plans: split units of one node per lane, whose gradient
kernels count nodes per lane, and value units split over 17 groups, against the
oracle and against the same plan in whole units."""
import numpy as np
import pytest

from nr_check import check_R, check_grad, check_logL, logL_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    return nr


def _batch(L, nq):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(100 * L + nq)
    Q = inputs.log_grid(0.008, 0.3, nq)
    curve = inputs.synthetic_curve(Q, rng)
    return inputs._pack("one", [(Q, *curve, 0.05)],
                        [(0, inputs.draw_stack(rng, L), 0.97, 1.3e-7) for _ in range(3)], {})


@pytest.mark.parametrize("L", [6, 20, 23, 24, 29, 36, 37, 40])
@pytest.mark.parametrize("nq", [1, 64, 130])
def test_fp64_against_the_oracle(nr, orc, L, nq):
    batch = _batch(L, nq)
    prob = nr.Problem.from_batch(batch)
    ll, g, gi = (t.cpu().numpy() for t in prob.loglik_grad())
    R = prob.reflectivity().cpu().numpy()
    for b in range(batch.n_items):
        Q, Robs, e, d = batch.data_of(b)
        rows = batch.rows_of(b)
        Ro = orc.model_curve(rows, 0.97, 1.3e-7, Q, d)
        check_R(R[b * nq:(b + 1) * nq], Ro)
        llo, go, gio = orc.loglik_grad_cs(rows, 0.97, 1.3e-7, Q, Robs, e, d)
        check_logL(ll[b], llo, logL_bound(Ro, Robs, e))
        check_grad(g[batch.row_off[b]:batch.row_off[b + 1]], gi[b], go, gio)


# The nodes of a lane are the same FP32 recursion in both layouts; the compiler
# may contract its products differently, 2^-24 each over up to 40 levels of some
# ten rounded operations on each of which the result depends linearly: 3e-5.
@pytest.mark.parametrize("L", [10, 12, 14, 24, 28, 32, 40])
def test_fp32_against_whole_units(nr, L):
    batch = _batch(L, 130)
    one = nr.Problem.from_batch(batch, precision=nr.NR_F32)
    whole = nr.Problem.from_batch(batch, precision=nr.NR_F32, options={"split_tails": 0})
    for x, y in zip(one.loglik_grad(), whole.loglik_grad()):
        x, y = x.cpu().numpy(), y.cpu().numpy()
        if x.ndim == 1:
            assert np.max(np.abs(x - y)) <= 3e-5 * np.max(np.abs(y))
        else:
            assert np.all(np.max(np.abs(x - y), axis=0) <= 3e-5 * np.max(np.abs(y), axis=0))
