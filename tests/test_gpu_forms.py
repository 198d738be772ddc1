"""The kernels that choose between node forms, with the launch list asserting that
they are what runs: split units at every node grouping, their bad-value and singular
paths, deep stacks of several waves per point on smeared data, and deep items beside
shallow ones."""
import numpy as np
import pytest

from nr_check import check_grad, check_logL, logL_bound

pytestmark = pytest.mark.gpu

FOURPI = 12.566370614359172


@pytest.fixture(scope="module")
def nr():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2509_06924_amd as nr
    return nr


def _recompute(nr, buckets=None, **options):
    lm = nr.bucket_lmax() if buckets is None else buckets
    return {"grad_variant": {str(k): nr._n.NR_VARIANT_RECOMPUTE for k in lm}, **options}


def _kinds(prob):
    return {(x["bucket"], x["form"], x["mode"]) for x in prob.plan.launches()}


def _stacks(rng, L):
    """Inside, outside and across the range of the above-edge form."""
    from paper_2509_06924_amd import inputs
    plain, lossless, opaque = (inputs.draw_stack(rng, L) for _ in range(3))
    lossless[:, 2] = 0.0
    opaque[1:, 2] = 2e-6
    return [plain, lossless, opaque]


def _edge_sld(Q):
    """The SLD whose 4 pi rho is (0.25 Q) Q exactly, or None."""
    want = (0.25 * Q) * Q
    near = [want / FOURPI]
    for _ in range(4):
        near += [np.nextafter(near[-1], 1.0)]
        near.insert(0, np.nextafter(near[0], 0.0))
    hit = [r for r in near if FOURPI * r == want]
    return hit[0] if hit else None


# (points, options): tails of 1, 3, 20 and 32 points split over their own node groups,
# and every point group split, with a remainder
SPLITS = [(65, {"split_tails": 3}), (67, {"split_tails": 3}), (84, {"split_tails": 3}),
          (96, {"split_tails": 3}), (70, {"node_groups": 2}), (50, {"node_groups": 3}),
          (23, {"node_groups": 6}), (16, {"node_groups": 9})]


@pytest.mark.parametrize("L", [6, 10, 14, 20, 24, 28, 36])
@pytest.mark.parametrize("nq,options", SPLITS, ids=[f"{n}-{o}" for n, o in SPLITS])
def test_split_units(nr, orc, L, nq, options):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(100 * L + nq)
    Q = inputs.log_grid(0.006, 0.3, nq)
    curve = inputs.synthetic_curve(Q, rng)
    batch = inputs._pack("split", [(Q, *curve, 0.06)],
                         [(0, r, 0.97, 1.3e-7) for r in _stacks(rng, L)], {})
    prob = nr.Problem.from_batch(batch, options=options)
    k = nr.bucket_lmax().index(L)
    assert (k, nr._n.NR_FORM_SELECT, nr._n.NR_MODE_SPLIT) in _kinds(prob)
    ll, g, gi = (t.cpu().numpy() for t in prob.loglik_grad())
    assert int(prob.item_status.abs().sum().item()) == 0
    ref = nr.Problem.from_batch(batch, options=_recompute(nr, **options))
    assert {f for _, f, _ in _kinds(ref)} == {nr._n.NR_FORM_RECOMPUTE}
    lr, gr, gir = (t.cpu().numpy() for t in ref.loglik_grad())
    for b in range(batch.n_items):
        r0, r1 = batch.row_off[b], batch.row_off[b + 1]
        Ro = orc.model_curve(batch.rows_of(b), 0.97, 1.3e-7, Q, 0.06)
        check_logL(ll[b], lr[b], logL_bound(Ro, *curve), what=f"item {b}")
        check_grad(g[r0:r1], gi[b], gr[r0:r1], gir[b], what=f"item {b}")
    # one item against the oracle
    b = L % 3
    llo, go, gio = orc.loglik_grad_cs(batch.rows_of(b), 0.97, 1.3e-7, Q, *curve, 0.06)
    check_grad(g[batch.row_off[b]:batch.row_off[b + 1]], gi[b], go, gio, what=f"item {b}")


@pytest.mark.parametrize("L", [6, 12, 20])
@pytest.mark.parametrize("options", [{"split_tails": 3}, {"node_groups": 4}], ids=["full", "split"])
def test_bad_values_and_singular_nodes(nr, L, options):
    """NaN and infinite entries, a node q <= 0 and w = 0 exactly (hit by the centre
    node, whose q is the point's) in the select form."""
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(L)
    Q = inputs.log_grid(0.008, 0.2, 70)
    Qbad = Q.copy()
    Qbad[9] = 0.0
    curve = inputs.synthetic_curve(Q, rng)
    rows = [inputs.draw_stack(rng, L) for _ in range(6)]
    rows[1][2, 1] = np.nan
    rows[2][3, 3] = np.inf
    rows[3][-1, 2] = 0.0
    at = next((i for i in range(20, 40) if _edge_sld(Q[i]) is not None), None)
    assert at is not None
    rows[3][-1, 1] = _edge_sld(Q[at])
    rows[5][2, 0] = np.nan
    batch = inputs._pack("bad", [(Q, *curve, 0.05), (Qbad, *curve, 0.05)],
                         [(int(i == 4), r, 1.0, 1e-7) for i, r in enumerate(rows)], {})
    prob = nr.Problem.from_batch(batch, options=options)
    assert {f for _, f, _ in _kinds(prob)} == {nr._n.NR_FORM_SELECT}
    ll, g, _ = (t.cpu().numpy() for t in prob.loglik_grad())
    st = prob.item_status.cpu().numpy()
    assert st[0] == 0 and np.isfinite(ll[0])
    for i in (1, 5):
        assert st[i] & nr.NR_ITEM_NONFINITE and np.isnan(ll[i])
    assert st[3] == nr.NR_ITEM_EDGE_SINGULAR and np.isfinite(ll[3])
    assert np.all(np.isfinite(g[batch.row_off[3]:batch.row_off[4]]))
    assert st[4] & nr.NR_ITEM_BAD_Q and np.isnan(ll[4])
    ref = nr.Problem.from_batch(batch, options=_recompute(nr, **options))
    lr = ref.loglik_grad()[0].cpu().numpy()
    assert np.array_equal(st, ref.item_status.cpu().numpy())
    assert np.array_equal(np.isnan(ll), np.isnan(lr))


@pytest.mark.parametrize("L", [600, 1030])
def test_smeared_deep_stack_against_the_oracle(nr, orc, L):
    """Two and four waves per point, 17 nodes in a row of both forms."""
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(L)
    Q = np.array([0.0185])
    curve = inputs.synthetic_curve(Q, rng)
    rows = inputs.draw_stack(rng, L, d=(2.0, 12.0), sigma=(0.5, 2.0))
    batch = inputs._pack("deep", [(Q, *curve, 0.06)], [(0, rows, 1.02, 1e-7)], {})
    prob = nr.Problem.from_batch(batch)
    assert {f for _, f, _ in _kinds(prob)} == {nr._n.NR_FORM_SELECT}
    ll, g, gi = (t.cpu().numpy() for t in prob.loglik_grad())
    Ro = orc.model_curve(rows, 1.02, 1e-7, Q, 0.06)
    llo, go, gio = orc.loglik_grad_cs(rows, 1.02, 1e-7, Q, *curve, 0.06)
    check_logL(ll[0], llo, logL_bound(Ro, *curve))
    check_grad(g, gi[0], go, gio)


@pytest.mark.parametrize("L", [41, 64, 300, 511, 512, 1000, 1023, 1024, 1500, 2047])
def test_smeared_deep_stacks_against_the_recompute_scan(nr, L):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(L)
    Q = np.array([0.006, 0.0165, 0.018, 0.03, 0.12, 0.3])
    curve = inputs.synthetic_curve(Q, rng)
    stacks = [inputs.draw_stack(rng, L, d=(2.0, 12.0), sigma=(0.5, 2.0)) for _ in range(4)]
    stacks[1][:, 2] = 0.0
    stacks[2][1:, 2] = 2e-6
    stacks[3][3, :3] = 3000.0, 6e-6, 1e-8
    batch = inputs._pack("deep", [(Q, *curve, 0.05)], [(0, r, 1.0, 1e-7) for r in stacks], {})
    out = []
    for options, form in ((None, nr._n.NR_FORM_SELECT), (_recompute(nr), nr._n.NR_FORM_RECOMPUTE)):
        prob = nr.Problem.from_batch(batch, options=options)
        assert {f for _, f, _ in _kinds(prob)} == {form}
        out.append([t.cpu().numpy() for t in prob.loglik_grad()])
        assert int(prob.item_status.abs().sum().item()) == 0
    for b in range(batch.n_items):
        r0, r1 = batch.row_off[b], batch.row_off[b + 1]
        check_grad(out[0][1][r0:r1], out[0][2][b], out[1][1][r0:r1], out[1][2][b],
                   what=f"item {b}")


def test_deep_beside_shallow_items(nr):
    """The scan's record order beside item order in one workspace, the recompute scan
    beside the select form, and status bits of both."""
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(8)
    Q = inputs.log_grid(0.01, 0.25, 12)
    curve = inputs.synthetic_curve(Q, rng)
    stacks = [inputs.draw_stack(rng, L, d=(2.0, 12.0)) for L in (10, 60, 3, 700, 45, 20, 1100)]
    stacks[4][7, 1] = np.nan
    at = next((i for i in range(4, 10) if _edge_sld(Q[i]) is not None), None)
    assert at is not None
    stacks[1][-1, 1:3] = _edge_sld(Q[at]), 0.0
    batch = inputs._pack("mixed", [(Q, *curve, 0.05)], [(0, r, 1.0, 1e-7) for r in stacks], {})
    deep, sel, rec = nr._n.NR_NUM_BUCKETS, nr._n.NR_FORM_SELECT, nr._n.NR_FORM_RECOMPUTE
    shallow = [nr.bucket_lmax().index(k) for k in (10, 20)]
    out = []
    for options, scan in (({"node_groups": 4}, sel),
                          (_recompute(nr, [nr.bucket_lmax()[-1]], node_groups=4), rec),
                          (_recompute(nr, node_groups=4), None)):
        prob = nr.Problem.from_batch(batch, options=options)
        forms = {(b, f) for b, f, _ in _kinds(prob)}
        if scan is not None:
            assert {(k, sel) for k in shallow} <= forms
            assert {f for b, f in forms if b == deep} == {scan}
        out.append([t.cpu().numpy() for t in prob.loglik_grad()] + [prob.item_status.cpu().numpy()])
    want = out[2]
    assert want[3][1] == nr.NR_ITEM_EDGE_SINGULAR and want[3][4] & nr.NR_ITEM_NONFINITE
    for got in out[:2]:
        assert np.array_equal(got[3], want[3])
        for i in (0, 2, 3, 5, 6):
            r0, r1 = batch.row_off[i], batch.row_off[i + 1]
            check_grad(got[1][r0:r1], got[2][i], want[1][r0:r1], want[2][i], what=f"item {i}")
