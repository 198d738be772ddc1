"""Plans of two callers, each on a stream of its own: a small call issued while
the other stream is busy does not wait for it, and captured and eager calls of one plan
do not disturb each other."""
import time

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


def _ragged(nr, items, seed, precision):
    from paper_2509_06924_amd import inputs
    rng = np.random.default_rng(seed)
    datasets, its = [], []
    for b in range(items):
        Q = inputs.log_grid(0.008, 0.3, int(rng.integers(100, 400)))
        datasets.append((Q, *inputs.synthetic_curve(Q, rng), 0.05))
        its.append((b, inputs.draw_stack(rng, int(rng.integers(2, 41))), 1.0, 1e-7))
    batch = inputs._pack("ragged", datasets, its, {})
    prob = nr.Problem.from_batch(batch, precision=precision)
    assert max(x["stream"] for x in prob.plan.launches()) > 0
    return prob


def test_a_call_does_not_wait_for_another_callers_stream(nr):
    import torch
    big, small = _ragged(nr, 1024, 1, nr.NR_F32), _ragged(nr, 24, 2, nr.NR_F32)
    want = small.loglik_grad()
    big_out = big.loglik_grad()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    big.loglik_grad(out=big_out)
    torch.cuda.synchronize()
    calls = int(0.3 / (time.perf_counter() - t0)) + 1
    s0 = torch.cuda.Stream()
    others = [torch.cuda.Stream() for _ in range(8)]
    x = torch.zeros(1, device="cuda")
    out = tuple(torch.empty_like(t) for t in want)
    torch.cuda.synchronize()
    for _ in range(calls):
        big.loglik_grad(stream=s0, out=big_out)
    end = torch.cuda.Event()
    end.record(s0)
    # a stream whose hardware queue holds none of the busy ones
    marks = []
    for s in others:
        with torch.cuda.stream(s):
            x + 1.0
            marks.append(torch.cuda.Event())
            marks[-1].record()
    time.sleep(0.05)
    free = [s for s, m in zip(others, marks) if m.query()]
    if not free or end.query():
        torch.cuda.synchronize()
        pytest.skip("every hardware queue is busy")
    small.loglik_grad(stream=free[0], out=out)
    free[0].synchronize()
    waited = end.query()
    torch.cuda.synchronize()
    assert not waited, "the small call ended after 0.3 s of another caller's work"
    for a, b in zip(out, want):
        assert torch.equal(a, b)


def test_captured_first_call_beside_eager_ones(nr):
    """The plan's first forked call is a captured one; replays and eager calls
    alternate."""
    import torch
    prob = _ragged(nr, 12, 3, nr.NR_F64)
    prob.workspace(nr.NR_OP_LOGLIK_GRAD)
    out = (torch.empty(12, dtype=torch.float64, device="cuda"), torch.empty_like(prob.layers),
           torch.empty(12, 2, dtype=torch.float64, device="cuda"))
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        prob.loglik_grad(out=out)
    want = [t.clone() for t in prob.loglik_grad()]
    for _ in range(3):
        for t in out:
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, want))
        assert all(torch.equal(a, b) for a, b in zip(prob.loglik_grad(), want))
