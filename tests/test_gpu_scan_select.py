"""The plain scan gradient of deep stacks (nr_scan_select.hip): depths around
its lane and wave boundaries, stacks in and out of the above-edge form's range
(strong contrasts, thick absorbing and evanescent slabs, where the cotangents
come from determinants instead of matrix products), against the oracle; and the
scan kernel that the recompute option names, whose records lie in item order."""
import numpy as np
import pytest

from nr_check import check_grad, check_logL, logL_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    return nr


def _stacks(rng, L):
    from paper_2509_06924_amd import inputs
    thin = inputs.draw_stack(rng, L, d=(2.0, 12.0), sigma=(0.5, 2.0))
    lossless = thin.copy()
    lossless[:, 2] = 0.0
    opaque = thin.copy()
    opaque[1:, 2] = 2e-6              # never in the range of the above form
    buried = thin.copy()
    buried[3, :3] = 3000.0, 6e-6, 1e-8  # evanescent at low q: what lies below is dark
    return [thin, lossless, opaque, buried, inputs.microsliced_stack(rng, L)]


@pytest.mark.parametrize("L", [41, 62, 63, 64, 127, 130, 257, 511, 512, 1024])
def test_depths(nr, orc, L):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(L)
    Q = np.array([0.008, 0.0175, 0.04, 0.11, 0.28])
    curve = inputs.synthetic_curve(Q, rng)
    batch = inputs._pack("scan", [(Q, *curve, 0.05), (Q, *curve, 0.0)],
                         [(s, r, 1.02, 1e-7) for r in _stacks(rng, L) for s in (0, 1)], {})
    prob = nr.Problem.from_batch(batch)
    ll, g, gi = (t.cpu().numpy() for t in prob.loglik_grad())
    assert int(prob.item_status.abs().sum().item()) == 0
    for b in range(batch.n_items):
        rows = batch.rows_of(b)
        d = batch.data_of(b)[3]
        if L > 130 and d > 0.0:  # (the oracle's cost: smeared nodes on the shallower ones)
            continue
        Ro = orc.model_curve(rows, 1.02, 1e-7, Q, d)
        llo, go, gio = orc.loglik_grad_cs(rows, 1.02, 1e-7, Q, *curve, d)
        check_logL(ll[b], llo, logL_bound(Ro, *curve), what=f"item {b}")
        check_grad(g[batch.row_off[b]:batch.row_off[b + 1]], gi[b], go, gio, what=f"item {b}")


def test_beside_shallow_items_and_the_recompute_scan(nr):
    """Deep and shallow items in one plan, and the same with the recompute
    option on the deepest bucket alone (the scan kernel then reads the deep
    items' records in item order beside the select form's); status bits of a
    NaN and of w = 0 exactly."""
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(8)
    Q = inputs.log_grid(0.01, 0.25, 12)
    curve = inputs.synthetic_curve(Q, rng)
    stacks = [inputs.draw_stack(rng, L, d=(2.0, 12.0)) for L in (10, 60, 3, 700, 45, 20)]
    stacks[4][7, 1] = np.nan
    four_pi = 12.566370614359172
    want = (0.25 * Q[5]) * Q[5]
    for r in (want / four_pi, np.nextafter(want / four_pi, 1.0), np.nextafter(want / four_pi, 0.0)):
        if four_pi * r == want:
            stacks[1][-1, 1:3] = r, 0.0
            break
    else:
        pytest.skip("no SLD puts this point on the edge exactly")
    batch = inputs._pack("mixed", [(Q, *curve, 0.0)], [(0, r, 1.0, 1e-7) for r in stacks], {})
    out = []
    for options in (None, {"grad_variant": {str(nr.bucket_lmax()[-1]): nr._n.NR_VARIANT_RECOMPUTE}}):
        prob = nr.Problem.from_batch(batch, options=options)
        out.append([t.cpu().numpy() for t in prob.loglik_grad()] + [prob.item_status.cpu().numpy()])
    a, b = out
    assert np.array_equal(a[3], b[3])
    assert a[3][1] == nr.NR_ITEM_EDGE_SINGULAR and a[3][4] & nr.NR_ITEM_NONFINITE
    for i in (0, 2, 3, 5):
        r0, r1 = batch.row_off[i], batch.row_off[i + 1]
        # (rounding of two schedules, as between the store and recompute forms)
        check_grad(a[1][r0:r1], a[2][i], b[1][r0:r1], b[2][i], tol=1e-10, what=f"item {i}")
