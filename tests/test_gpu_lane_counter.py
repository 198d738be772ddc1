"""Gradient launches of one node per lane, plain and with the resolution derivative,
where the nodes are counted per lane and where per wave (few and many waves, every
kind of bucket), against the same plan in whole units."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    return nr


# The nodes of a lane are the same recursion in both layouts: FP64 to 1e-10 (rounding
# of two schedules), FP32 to 3e-5 (see tests/test_gpu_one_node.py).
@pytest.mark.parametrize("precision,tol", [("f64", 1e-10), ("f32", 3e-5)])
@pytest.mark.parametrize("L", [1, 2, 4, 6, 8, 12, 14, 16, 18, 20, 24, 32, 40])
@pytest.mark.parametrize("items", [1, 14])  # 44 and 616 waves of 3 points
def test_against_whole_units(nr, L, items, precision, tol):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(100 * L + items)
    Q = inputs.log_grid(0.008, 0.3, 130)
    batch = inputs._pack("one", [(Q, *inputs.synthetic_curve(Q, rng), 0.05)],
                         [(0, inputs.draw_stack(rng, L), 0.97, 1.3e-7)] * items, {})
    prec = nr.NR_F32 if precision == "f32" else nr.NR_F64
    one = nr.Problem.from_batch(batch, precision=prec, options={"node_groups": 17})
    assert [x["units"] for x in one.plan.launches()] == [44 * items]
    whole = nr.Problem.from_batch(batch, precision=prec, options={"split_tails": 0})
    for call in ("loglik_grad", "loglik_grad_res"):
        for x, y in zip(getattr(one, call)(), getattr(whole, call)()):
            x, y = x.cpu().numpy(), y.cpu().numpy()
            assert np.all(np.isfinite(x))
            scale = np.max(np.abs(y), axis=0)
            assert np.all(np.max(np.abs(x - y), axis=0) <= tol * scale), call
