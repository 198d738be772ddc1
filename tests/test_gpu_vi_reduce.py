"""The mean-field ELBO reduction at sample counts around its 256 sample lanes
and entry counts around its blocks of four, against NumPy sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S", [1, 255, 256, 257, 1030])
@pytest.mark.parametrize("L", [0, 1, 40])
def test_sums_over_samples(S, L):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(S + L)
    rows = inputs.draw_stack(rng, L)
    Q = inputs.log_grid(0.01, 0.3, 3)
    batch = inputs._pack("vi", [(Q, *inputs.synthetic_curve(Q, rng), 0.0)],
                         [(0, rows, 1.0, 1e-7)] * S, {})
    prob = nr.Problem.from_batch(batch)
    P = rows.size + 2
    mu = np.concatenate([rows.ravel(), [1.0, 1e-7]])
    mask = (rng.random(P) < 0.7).astype(np.uint8)
    mask[:4] = 0
    omega = np.log(np.expm1(1e-3 * np.abs(mu) + 1e-12))
    eps = rng.standard_normal((S, P))
    elbo, gmu, gom, ll = (t.cpu().numpy() for t in prob.vi_elbo_grad(mu, omega, mask, eps))
    # the samples' own gradients, at the positions the sampler formed (to
    # rounding of theta: relative 2 eps, far inside the 1e-9 bound below)
    s = np.log1p(np.exp(omega))
    th = np.where(mask != 0, mu + s * eps, mu)
    lay, sc, bk = (torch.as_tensor(np.ascontiguousarray(x), device=prob.device)
                   for x in (th[:, :-2].reshape(-1, 4), th[:, -2], th[:, -1]))
    l2, gr, gi = (t.cpu().numpy() for t in prob.loglik_grad(lay, sc, bk))
    g = np.concatenate([gr.reshape(S, -1), gi], 1)
    slope = 1.0 / (1.0 + np.exp(-omega))
    on = mask != 0
    np.testing.assert_allclose(ll, l2, rtol=1e-9)
    np.testing.assert_allclose(elbo[0], l2.mean() + np.log(s[on]).sum(), rtol=1e-9)
    # sums of S terms: rounding (S + 8) eps of the terms' absolute sum, plus
    # 1e-9 of it for the positions' rounding through the gradient
    tol_mu = 1e-9 * np.abs(g).mean(0)
    tol_om = 1e-9 * (np.abs(g * eps).mean(0) * slope + slope / s)
    assert np.all(np.abs(gmu - np.where(on, g.mean(0), 0.0)) <= tol_mu)
    assert np.all(np.abs(gom - np.where(on, (g * eps).mean(0) * slope + slope / s, 0.0)) <= tol_om)
