"""What the rules of a plan's schedule come to, by the launch list: each line was
measured, and a change that moves it shows here instead of as a slower call."""
import numpy as np
import pytest

from nr_check import check_R, check_logL, logL_bound

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the lines are those of 1024 SIMDs")
    import paper_2509_06924_amd as nr
    return nr


def _batch(L, nq, items, dqq=0.05):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(1)
    Q = inputs.log_grid(0.008, 0.3, nq)
    Ls = L if isinstance(L, (list, tuple)) else [L] * items
    return inputs._pack("schedule", [(Q, *inputs.synthetic_curve(Q, rng), dqq)],
                        [(0, inputs.draw_stack(rng, k), 0.97, 1.3e-7) for k in Ls], {})


# value units of 64 points: node groups per point, and waves of 3 points at 17 groups
@pytest.mark.parametrize("precision,L,items,groups", [
    ("f64", 5, 64, 17), ("f64", 5, 65, 9), ("f64", 5, 256, 6), ("f32", 5, 102, 17),
    ("f32", 5, 103, 9), ("f32", 12, 256, 6), ("f32", 13, 511, 9), ("f32", 13, 512, 6)])
def test_value_groups_of_small_plans(nr, precision, L, items, groups):
    p = nr.Problem.from_batch(_batch(L, 64, items),
                              precision=nr.NR_F32 if precision == "f32" else nr.NR_F64)
    (launch,) = p.plan.launches(nr.NR_OP_LOGLIK)
    points = 64 // groups
    assert launch["units"] == items * -(-64 // points)


@pytest.mark.parametrize("items", [46, 47])  # 1012 and 1034 waves
def test_fp32_value_kernels_about_one_wave_per_simd(nr, orc, items):
    batch = _batch(20, 64, items)
    p = nr.Problem.from_batch(batch, precision=nr.NR_F32)
    R = p.reflectivity().cpu().numpy().reshape(items, 64)
    for b in (0, items - 1):
        Q, *_, d = batch.data_of(b)
        # (the FP32 variant's bound, tests/test_gpu_fp32.py)
        check_R(R[b], orc.model_curve(batch.rows_of(b), 0.97, 1.3e-7, Q, d), tol=1e-4)


# unsmeared, waves and points x levels of an item about the lines of the one form
@pytest.mark.parametrize("L,nq,items,forms", [
    (1, 64, 2048, True), (1, 64, 2049, False), (7, 162, 700, False), (7, 163, 700, True)])
def test_value_form_of_items_of_little_work(nr, orc, L, nq, items, forms):
    batch = _batch(L, nq, items, dqq=0.0)
    p = nr.Problem.from_batch(batch)
    (launch,) = p.plan.launches(nr.NR_OP_REFLECTIVITY)
    assert launch["form"] == (nr._n.NR_FORM_SELECT if forms else nr._n.NR_FORM_RECOMPUTE)
    R = p.reflectivity().cpu().numpy().reshape(items, nq)
    ll = p.loglik().cpu().numpy()
    assert int(p.item_status.abs().sum().item()) == 0
    for b in (0, 1, items - 1):
        Q, Robs, e, d = batch.data_of(b)
        Ro = orc.model_curve(batch.rows_of(b), 0.97, 1.3e-7, Q, d)
        check_R(R[b], Ro)
        llo = orc.loglik(batch.rows_of(b), 0.97, 1.3e-7, Q, Robs, e, d)
        check_logL(ll[b], llo, logL_bound(Ro, Robs, e))


def test_resolution_calls_have_units_of_their_own(nr):
    """Split in node groups, the plain call is the faster, the one with the resolution
    derivative the slower (14 layers FP64: its split kernel spills twice as much)."""
    import torch
    batch = _batch(14, 100, 1536)
    p = nr.Problem.from_batch(batch)
    assert {x["mode"] for x in p.plan.launches()} == {nr._n.NR_MODE_SPLIT}
    whole = nr.Problem.from_batch(batch, options={"split_tails": 3})
    assert {x["mode"] for x in whole.plan.launches()} == {nr._n.NR_MODE_FULL}
    for x, y in zip(p.loglik_grad_res(), whole.loglik_grad_res()):
        assert torch.equal(x, y)
    # the plain call's records and the other schedule's share the workspace
    want = [t.clone() for t in p.loglik_grad()]
    p.loglik_grad_res()
    assert all(torch.equal(x, y) for x, y in zip(p.loglik_grad(), want))


def _streams(p):
    return [x["stream"] for x in p.plan.launches()]


def test_split_launch_comes_after_whole_units_that_fill_their_rounds(nr):
    # 400 points: six whole units per item and a tail of 16, in a split launch
    p = nr.Problem.from_batch(_batch(6, 400, 4096))
    assert [(x["mode"], x["units"], x["stream"]) for x in p.plan.launches()] == [
        (nr._n.NR_MODE_FULL, 6 * 4096, 0), (nr._n.NR_MODE_SPLIT, 4096, 0)]
    # three waves per SIMD, and room in the last round
    assert _streams(nr.Problem.from_batch(_batch(6, 400, 3072))) == [0, 1]
    assert _streams(nr.Problem.from_batch(_batch(6, 400, 4200))) == [0, 1]


def test_launches_shorter_than_a_fork_stay_in_a_row(nr):
    assert _streams(nr.Problem.from_batch(_batch([20, 2], 200, 2))) == [0, 0]
    assert max(_streams(nr.Problem.from_batch(_batch([36, 28], 200, 2)))) == 1
    assert max(_streams(nr.Problem.from_batch(_batch([40, 30, 20, 10], 300, 4)))) == 3


@pytest.mark.parametrize("precision,L", [("f64", 40), ("f32", 33), ("f32", 40)])
def test_tails_that_would_displace_whole_units_share_waves(nr, precision, L):
    """300 items of 400 points: 1800 whole units and 300 tails are more than two rounds of
    1024 SIMDs, with four tails of 16 points in a wave they are not."""
    p32 = precision == "f32"
    batch = _batch(L, 400, 300)
    make = lambda o=None: nr.Problem.from_batch(  # noqa: E731
        batch, precision=nr.NR_F32 if p32 else nr.NR_F64, options=o)
    p, own = make(), make({"split_tails": 3})
    M = nr._n
    assert {(x["mode"], x["units"]) for x in p.plan.launches()} == {
        (M.NR_MODE_FULL, 1800), (M.NR_MODE_PACKED, 75)}
    assert {(x["mode"], x["units"]) for x in own.plan.launches()} == {
        (M.NR_MODE_FULL, 1800), (M.NR_MODE_SPLIT, 300)}
    got, want = ([t.cpu().numpy() for t in x.loglik_grad()] for x in (p, own))
    # sums in another order (tests/test_gpu_autotune.py); FP32 nodes: the variant's bound
    assert np.allclose(got[0], want[0], rtol=1e-4 if p32 else 1e-12, atol=0)
    units = np.array([1.0, 1e-6, 1e-6, 1.0])
    scale = np.max(np.abs(want[1] * units))
    assert np.max(np.abs((got[1] - want[1]) * units)) <= (1e-4 if p32 else 1e-10) * scale
    # fewer whole units than SIMDs, or room for the tails: waves of their own, or groups
    for items in (100, 250):
        modes = {x["mode"] for x in nr.Problem.from_batch(
            _batch(L, 400, items), precision=p.plan.precision).plan.launches()}
        assert M.NR_MODE_PACKED not in modes
