"""The value kernels (nr_reflectivity, nr_loglik) at the edges of their units:
group sizes around 64 points, odd and even depths (levels go in pairs), every
number of node groups that the plan size selects, both precisions."""
import numpy as np
import pytest

from nr_check import R_TOL, check_logL, check_R, logL_bound

pytestmark = pytest.mark.gpu

# the FP32 variant's R against the oracle (test_gpu_fp32.py)
R_TOL_F32 = 1e-4


@pytest.fixture(scope="module")
def nr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    return nr


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("nq", [1, 3, 63, 64, 65, 130])
def test_group_sizes_and_depths(nr, orc, nq, precision):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(nq)
    datasets, items = [], []
    for s, (lo, dqq) in enumerate(((0.006, 0.05), (0.03, 0.08), (0.006, 0.0))):
        Q = inputs.log_grid(lo, 0.3, nq)
        datasets.append((Q, *inputs.synthetic_curve(Q, rng), dqq))
        for L in (0, 1, 2, 3, 10, 41):
            items.append((s, inputs.draw_stack(rng, L, d=(10.0, 60.0)), 0.98, 1e-7))
    batch = inputs._pack("value", datasets, items, {})
    f32 = precision == "f32"
    prob = nr.Problem.from_batch(batch, precision=nr.NR_F32 if f32 else nr.NR_F64)
    R, ll = prob.reflectivity().cpu().numpy(), prob.loglik().cpu().numpy()
    assert int(prob.item_status.abs().sum().item()) == 0
    for b in range(batch.n_items):
        Q, Robs, e, d = batch.data_of(b)
        Ro = orc.model_curve(batch.rows_of(b), 0.98, 1e-7, Q, d)
        tol = R_TOL_F32 if f32 else R_TOL
        check_R(R[prob.out_off[b]:prob.out_off[b + 1]], Ro, tol=tol, what=f"R item {b}")
        llo = orc.loglik(batch.rows_of(b), 0.98, 1e-7, Q, Robs, e, d)
        check_logL(ll[b], llo, logL_bound(Ro, Robs, e, tol=tol), what=f"logL item {b}")


@pytest.mark.parametrize("n", [100, 250, 900, 1600])  # 9, 6, 2 and 1 node groups
def test_plan_sizes(nr, orc, n):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(5)
    Q = inputs.log_grid(0.006, 0.3, 70)  # a whole group and one of 6 points
    curve = inputs.synthetic_curve(Q, rng)
    rows = inputs.draw_stack(rng, 5)
    batch = inputs._pack("sizes", [(Q, *curve, 0.05)], [(0, rows, 1.0, 1e-7)] * n, {})
    prob = nr.Problem.from_batch(batch)
    R, ll = prob.reflectivity().cpu().numpy().reshape(n, -1), prob.loglik().cpu().numpy()
    assert np.all(R == R[0]) and np.all(ll == ll[0])
    Ro = orc.model_curve(rows, 1.0, 1e-7, Q, 0.05)
    check_R(R[0], Ro)
    check_logL(ll[0], orc.loglik(rows, 1.0, 1e-7, Q, *curve, 0.05), logL_bound(Ro, *curve))
