"""Performance cases: what a program that fits or samples reflectivity models asks of the library.

A case is a dict of plain values.  `kind` says which public entry points a pass goes through:

  grad      Problem.loglik_grad: logL and its gradient (optimisers, samplers)
  autograd  NRLogLik.apply and its backward pass (a loss inside a PyTorch program)
  value     Problem.loglik: logL alone (Metropolis tests, model comparison)
  curves    Problem.reflectivity: model curves (posterior predictive bands)
  vjp       NRReflectivity.apply and its backward pass (a likelihood of the caller's own)
  cofit     loglik_grad of a co-fit under several contrasts, and the tie-sum onto shared parameters
  leapfrog  an HMC proposal: the current position copied in, then a captured leapfrog step replayed
  vi        Problem.vi_elbo_grad: the mean-field reparameterised ELBO gradient
  deep      loglik_grad of microsliced profiles (more than 40 slabs)

`items` parameter draws or data sets, each of layers_lo..layers_hi layers; data sets of points_lo..points_hi points, log-spaced in Q, one
for all items (`shared`) or one each; dQ/Q in smear_lo..smear_hi (0: unsmeared); `precision` f64 or f32.  Values are drawn like those of
paper_2509_06924_amd.inputs.  The structure (layer counts, lengths) depends on the case alone, the values on the seed too."""
import math

import numpy as np
import torch

import paper_2509_06924_amd as nr
from paper_2509_06924_amd import inputs

NODES = 17
UNITS = (1.0, 1e-6, 1e-6, 1.0)  # natural units of d, rho_re, rho_im, sigma
CONTRASTS = (2.07e-6, 4.0e-6, 6.35e-6)  # backing SLDs of a co-fit
DT = 1e-3  # leapfrog step in natural units
# FLOP per node and layer, FMA = 2, with a square root or a division at 10, exp 20, sin and cos 40: value 257, value and adjoint 424
FLOPS_VALUE, FLOPS_GRAD = 257, 424
# layer-steps of the largest listed case, which a drawn case stays below
MOST_STEPS = 3.4e9


def _case(kind, items, layers, points, smear, precision="f64", shared=True, name=None):
    c = {"kind": kind, "items": items, "layers_lo": layers[0], "layers_hi": layers[1], "points_lo": points[0],
         "points_hi": points[1], "smear_lo": smear[0], "smear_hi": smear[1], "precision": precision, "shared": shared}
    return dict(c, name=name) if name else c


def listed():
    S5, S28 = (0.05, 0.05), (0.02, 0.08)
    return [
        # one oxide film on silicon, unsmeared: the smallest call, one step of an interactive fit; launches and latency
        _case("grad", 1, (1, 1), (200, 200), (0.0, 0.0), name="film"),
        # one 10-layer model against one smeared data set inside a PyTorch optimiser loop
        _case("autograd", 1, (10, 10), (400, 400), S5, name="fit"),
        # thousands of draws of one model: parallel chains or Monte-Carlo samples; the library's headline workload
        _case("grad", 4096, (10, 10), (400, 400), S5, name="draws"),
        # the same in the FP32 variant
        _case("grad", 4096, (10, 10), (400, 400), S5, precision="f32", name="draws_f32"),
        # the same draws, value only: Metropolis tests, importance weights
        _case("value", 4096, (10, 10), (400, 400), S5, name="draws_value"),
        # curves of models of every depth on grids of their own: predictive bands, simulated data
        _case("curves", 1024, (2, 40), (100, 1000), S28, shared=False, name="curves"),
        # curves and their vector-Jacobian product: a likelihood of the caller's own, for a batch of 6-layer models
        _case("vjp", 256, (6, 6), (300, 300), S5, name="curve_vjp"),
        # co-fit of 12-layer devices under three contrasts with uneven grids, 50 parameters shared by each draw's items
        _case("cofit", 1024, (12, 12), (250, 350), S5, name="cofit"),
        # one HMC leapfrog step over 16384 independent ragged data sets, replayed from a graph: the largest call
        _case("leapfrog", 16384, (2, 40), (100, 1000), S28, shared=False, name="ragged_leapfrog"),
        # a ragged batch in the FP32 variant
        _case("grad", 2048, (2, 40), (100, 1000), S28, precision="f32", shared=False, name="ragged_f32"),
        # mean-field variational inference of a 20-layer stack on a long data set
        _case("vi", 1024, (20, 20), (1000, 1000), S5, name="vi"),
        # microsliced profiles of a thousand slabs
        _case("deep", 64, (1000, 1000), (200, 200), S5, name="deep"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(("grad", "grad", "ragged", "ragged", "autograd", "value", "curves", "vjp", "cofit", "leapfrog", "vi", "deep"))
        f32 = rng.random() < 0.3
        smear = (0.0, 0.0) if rng.random() < 0.15 else (round(rng.uniform(0.02, 0.08), 4),) * 2
        if kind == "ragged":
            c = _case("grad", _log_int(rng, 16, 16384), (2, 40), (100, 1000), (0.02, 0.08), shared=False)
        elif kind in ("curves", "leapfrog") and rng.random() < 0.5:
            c = _case(kind, _log_int(rng, 4, 8192), (2, 40), (100, 1000), (0.02, 0.08), shared=False)
        elif kind == "cofit":
            n = rng.randint(100, 500)
            c = _case(kind, _log_int(rng, 8, 2048), (rng.randint(2, 24),) * 2, (n, n + rng.randint(0, 200)), smear)
        elif kind == "vi":
            c = _case(kind, _log_int(rng, 8, 8192), (rng.randint(2, 30),) * 2, (rng.randint(100, 1000),) * 2, smear)
        elif kind == "deep":
            c = _case(kind, _log_int(rng, 1, 64), (_log_int(rng, 45, 1500),) * 2, (rng.randint(50, 200),) * 2, smear)
        else:
            c = _case(kind, _log_int(rng, 1, 8192), (_log_int(rng, 1, 40),) * 2, (_log_int(rng, 50, 1000),) * 2, smear)
        if f32 and kind != "deep":
            c["precision"] = "f32"
        if steps(c) <= (0.1 if kind == "deep" else 1.0) * MOST_STEPS:
            return c


def structure(c):
    """Layer counts per item, points and dQ/Q per data set, and each item's data set."""
    rng = np.random.default_rng([2509069240, c["items"], c["layers_hi"], c["points_hi"]])
    n = c["items"]
    if c["kind"] == "cofit":
        k = len(CONTRASTS)
        layers = np.full(n * k, c["layers_lo"], np.int64)
        points = np.linspace(c["points_lo"], c["points_hi"], k).astype(np.int64)
        of = np.tile(np.arange(k, dtype=np.int32), n)
    else:
        layers = rng.integers(c["layers_lo"], c["layers_hi"] + 1, n)
        sets = 1 if c["shared"] else n
        points = rng.integers(c["points_lo"], c["points_hi"] + 1, sets)
        of = np.zeros(n, np.int32) if c["shared"] else np.arange(n, dtype=np.int32)
    smear = rng.uniform(c["smear_lo"], c["smear_hi"], points.size) if c["smear_hi"] > c["smear_lo"] else np.full(points.size, c["smear_lo"])
    return layers, points, smear, of


def steps(c):
    """Layer-steps of one evaluation: nodes times interfaces, over all items and points."""
    layers, points, smear, of = structure(c)
    return int(np.sum(points[of] * np.where(smear[of] > 0, NODES, 1) * (layers + 1)))


def work(c):
    layers, points, smear, of = structure(c)
    rows, n, q = int(np.sum(layers + 2)), of.size, int(points.sum())
    out = int(points[of].sum())
    par = 8 * (4 * rows + 2 * n)  # parameters, or a gradient
    data = 24 * q
    b = {"value": par + data + 8 * n, "curves": par + 8 * q + 8 * out, "vjp": 2 * par + 8 * q + 16 * out,
         "leapfrog": 6 * par + data + 8 * n, "vi": 2 * par + data + 8 * n}.get(c["kind"], 2 * par + data + 8 * n)
    return {"bytes": b, "flops": steps(c) * (FLOPS_VALUE if c["kind"] in ("value", "curves") else FLOPS_GRAD)}


def host_values(c, seed):
    """The batch as host arrays: grids, data, rows, instrument."""
    layers, points, smear, of = structure(c)
    rng = np.random.default_rng([int(seed), 1])
    n, kind = of.size, c["kind"]
    lo, hi = (0.008, 0.3) if c["smear_hi"] == 0 and n == 1 else (0.005, 0.3) if kind == "deep" else (0.005, 0.35)
    q_off = np.concatenate([[0], np.cumsum(points)])
    at = np.arange(q_off[-1]) - np.repeat(q_off[:-1], points)
    Q = lo * np.exp(math.log(hi / lo) * at / np.repeat(np.maximum(points - 1, 1), points))
    r_obs, r_err = inputs.synthetic_curve(Q, rng)
    row_off = np.concatenate([[0], np.cumsum(layers + 2)])
    rows = np.zeros((row_off[-1], 4))
    first, last = row_off[:-1], row_off[1:] - 1
    scale, bkg = rng.uniform(0.9, 1.1, n), rng.uniform(0.5e-7, 1.5e-7, n)
    if kind == "deep":
        for b in range(n):
            rows[row_off[b]:row_off[b + 1]] = inputs.microsliced_stack(rng, int(layers[b]))
    else:
        d, rho, sigma = ((20.0, 80.0), (0.5e-6, 4.5e-6), (2.0, 10.0)) if kind == "cofit" else ((10.0, 300.0), (-0.5e-6, 6.5e-6), (1.0, 15.0))
        m = rows.shape[0]
        rows[:] = np.stack([rng.uniform(*d, m), rng.uniform(*rho, m), rng.uniform(0.0, 1e-8, m), rng.uniform(*sigma, m)], 1)
        if n == 1 and layers[0] == 1:  # an oxide film
            rows[1] = rng.uniform(500.0, 1500.0), 3.47e-6, 0.0, rng.uniform(2.0, 10.0)
        if kind == "cofit":  # a draw's items differ in the backing only
            k = len(CONTRASTS)
            rows = rows.reshape(n // k, k, -1, 4)
            rows = np.repeat(rows[:, :1], k, axis=1).reshape(m, 4)
            scale[:], bkg = 1.0, np.repeat(bkg[::k], k)
        if kind == "vi":  # every item starts at the same stack
            rows = np.tile(rows[:row_off[1]], (n, 1))
            scale[:], bkg[:] = 1.0, 1e-7
        rows[first] = 0.0
        rows[last, 0], rows[last, 2] = 0.0, 0.0
        rows[last, 1] = np.asarray(CONTRASTS)[of] if kind == "cofit" else inputs.SI_SLD
    return {"q_off": q_off, "Q": Q, "r_obs": r_obs, "r_err": r_err, "smear": smear, "of": of, "row_off": row_off, "rows": rows, "scale": scale, "bkg": bkg}


def tie_map(h):
    """Shared parameters of a co-fit draw: its layers' entries, the backing's roughness and the background."""
    k, n = len(CONTRASTS), h["of"].size
    m = int(h["row_off"][1])
    per = 4 * (m - 2) + 2
    own = -np.ones((m, 4), np.int64)
    own[1:-1] = np.arange(per - 2).reshape(-1, 4)
    own[-1, 3] = per - 2
    draw_of = np.repeat(np.arange(n // k), k) * per
    rows = np.where(own >= 0, own + draw_of[:, None, None], -1)
    inst = np.stack([np.full(n, -1), draw_of + per - 1], 1)
    return nr.tie_map_to_csr(np.concatenate([rows.reshape(-1), inst.reshape(-1)]), n // k * per)


def vi_args(c, h, seed):
    """Means, widths (softplus of omega), the mask of variational entries, and the standard normal draws."""
    m = int(h["row_off"][1])
    mu = np.concatenate([h["rows"][:m].reshape(-1), [1.0, 1e-7]])
    mask = np.zeros(mu.size, np.uint8)
    mask[4:4 * (m - 1)] = 1
    mask[-2:] = 1
    omega = np.log(np.expm1(np.maximum(0.01 * np.abs(mu), 1e-12)))
    return mu, omega, mask, np.random.default_rng([int(seed), 2]).standard_normal((c["items"], mu.size))


def momenta(h, seed):
    rng = np.random.default_rng([int(seed), 3])
    return rng.standard_normal(h["rows"].shape) / UNITS, rng.standard_normal((h["of"].size, 2)) / (1.0, 1e-7)


def prepare(c, seed):
    h = host_values(c, seed)
    plan = nr.Plan(h["q_off"], h["smear"], h["of"], h["row_off"], nr.NR_F32 if c["precision"] == "f32" else nr.NR_F64)
    prob = nr.Problem(plan, h["Q"], h["r_obs"], h["r_err"], h["rows"], h["scale"], h["bkg"])
    s = {"kind": c["kind"], "prob": prob}
    dev = prob.device
    if c["kind"] in ("autograd", "vjp"):
        s["params"] = [t.clone().requires_grad_() for t in (prob.layers, prob.scale, prob.bkg)]
        s["row_item"] = prob.row_item
    if c["kind"] == "vjp":
        s["seeds"] = torch.as_tensor(np.random.default_rng([int(seed), 4]).standard_normal(int(prob.out_off[-1])), device=dev)
    if c["kind"] == "cofit":
        s["tie"] = [torch.as_tensor(t, device=dev) for t in tie_map(h)]
    if c["kind"] == "vi":
        s["vi"] = [torch.as_tensor(t, device=dev) for t in vi_args(c, h, seed)]
    if c["kind"] == "leapfrog":
        rows, inst = momenta(h, seed)
        im = (np.tile(np.square(UNITS), (rows.shape[0], 1)), np.tile((1.0, 1e-14), (inst.shape[0], 1)))
        st = s["hmc"] = nr.HmcState(prob, rows, inst, *im)
        s["at"] = [t.clone() for t in (st.layers, st.scale, st.bkg, st.mom_rows, st.mom_inst, st.g_rows, st.g_inst)]
        s["graph"] = nr.LeapfrogGraph(prob, st, DT, 1)
    return s


def run(s):
    prob, kind = s["prob"], s["kind"]
    if kind == "value":
        return prob.loglik()
    if kind == "curves":
        return prob.reflectivity()
    if kind == "autograd":
        logL = nr.NRLogLik.apply(*s["params"], prob)
        return (logL, *torch.autograd.grad(logL.sum(), s["params"]))
    if kind == "vjp":
        R = nr.NRReflectivity.apply(*s["params"], prob)
        return (R, *torch.autograd.grad(R, s["params"], s["seeds"]))
    if kind == "cofit":
        logL, g_rows, g_inst = prob.loglik_grad()
        return logL, nr.tie_sum(*s["tie"], torch.cat([g_rows.reshape(-1), g_inst.reshape(-1)]))
    if kind == "vi":
        return prob.vi_elbo_grad(*s["vi"])
    if kind == "leapfrog":
        st = s["hmc"]
        for to, at in zip((st.layers, st.scale, st.bkg, st.mom_rows, st.mom_inst, st.g_rows, st.g_inst), s["at"]):
            to.copy_(at)
        s["graph"].launch()
        return st.layers, st.scale, st.bkg, st.mom_rows, st.mom_inst, st.logL, st.g_rows, st.g_inst
    return prob.loglik_grad()


# ---- the same in plain 64-bit torch ----


def _rule():
    x, w = np.polynomial.legendre.leggauss(NODES)
    t = 3.5 * x
    w = w * np.exp(-0.5 * t * t)
    return t, w / w.sum()


def _root(x, b):
    """sqrt(x - i b) with Re >= 0, Im <= 0, for b >= 0."""
    z = torch.sqrt(torch.complex(x.abs(), b.expand_as(x)))
    up = x >= 0
    return torch.complex(torch.where(up, z.real, z.imag), -torch.where(up, z.imag, z.real))


def _curve(rows, q):
    """R(q): rows (points, layers + 2, 4), q (points, nodes)."""
    A = 4 * math.pi * (rows[:, :, 1] - rows[:, :1, 1])
    im = rows[:, :, 2]
    B = 4 * math.pi * torch.where(im < 0, -im, im)
    B = torch.cat([torch.zeros_like(B[:, :1]), B[:, 1:]], 1)
    k0 = 0.25 * q * q
    L = rows.shape[1] - 2
    below = _root(k0 - A[:, -1:], B[:, -1:])
    P = torch.ones_like(below)
    T = torch.zeros_like(below)
    for j in range(L, -1, -1):
        here = _root(k0 - A[:, j:j + 1], B[:, j:j + 1]) if j else torch.complex(0.5 * q, torch.zeros_like(q))
        step = torch.complex(A[:, j + 1] - A[:, j], B[:, j + 1] - B[:, j])[:, None]
        r = step / (here + below) ** 2 * torch.exp(-2 * rows[:, j + 1, 3, None] ** 2 * here * below)
        P, T = P + r * T, r * P + T
        if j:
            T = T * torch.exp(-2j * here * rows[:, j, 0, None])
        below = here
    r = T / P
    return r.real ** 2 + r.imag ** 2


def _evaluate(c, h, rows, scale, bkg, seeds=None, grad=True):
    """Per item logL (or the seeded sum), the packed curve, and the gradients in the layout of loglik_grad."""
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    f = lambda v: torch.as_tensor(v, dtype=torch.float64, device=dev)  # noqa: E731
    rows, scale, bkg = f(rows), f(scale), f(bkg)
    Q, r_obs, r_err = f(h["Q"]), f(h["r_obs"]), f(h["r_err"])
    t, w = (f(v) for v in _rule())
    n, layers, of = h["of"].size, np.diff(h["row_off"]) - 2, h["of"]
    counts = np.diff(h["q_off"])[of]
    out_off = np.concatenate([[0], np.cumsum(counts)])
    logL, R = torch.zeros(n, dtype=torch.float64, device=dev), torch.zeros(int(out_off[-1]), dtype=torch.float64, device=dev)
    g_rows, g_inst = torch.zeros_like(rows), torch.zeros(n, 2, dtype=torch.float64, device=dev)
    smeared = h["smear"][of] > 0
    for L, K in sorted({(int(a), bool(b)) for a, b in zip(layers, smeared)}):
        items = np.flatnonzero((layers == L) & (smeared == K))
        own_rows = torch.as_tensor(h["row_off"][items][:, None] + np.arange(L + 2), device=dev)
        p_rows, p_scale, p_bkg = (v.detach().clone().requires_grad_(grad) for v in (rows[own_rows], scale[items], bkg[items]))
        who = np.repeat(np.arange(items.size), counts[items])
        nth = np.arange(who.size) - np.repeat(np.cumsum(counts[items]) - counts[items], counts[items])
        point = torch.as_tensor(h["q_off"][of[items]][who] + nth, device=dev)
        place = torch.as_tensor(out_off[items][who] + nth, device=dev)
        width = f(h["smear"][of[items]][who])
        who = torch.as_tensor(who, device=dev)
        most = max(1, int(1.5e7 / ((L + 1) * (NODES if K else 1))))
        for a in range(0, who.numel(), most):
            i, x = who[a:a + most], point[a:a + most]
            q = Q[x, None]
            if K:
                q = q + width[a:a + most, None] * q / 2.3548200450309493 * t
            with torch.set_grad_enabled(grad):
                v = _curve(p_rows[i], q)
                v = p_scale[i] * ((v * w).sum(1) if K else v[:, 0]) + p_bkg[i]
                if seeds is not None:
                    ll = f(seeds)[place[a:a + most]] * v
                else:
                    ll = -0.5 * ((v - r_obs[x]) / r_err[x]) ** 2 - torch.log(r_err[x]) - 0.5 * math.log(2 * math.pi)
                if grad:
                    ll.sum().backward()
            R[place[a:a + most]] = v.detach()
            logL.index_add_(0, torch.as_tensor(items, device=dev)[i], ll.detach())
        if grad:
            g_rows[own_rows.reshape(-1)] = p_rows.grad.reshape(-1, 4)
            g_inst[torch.as_tensor(items, device=dev)] = torch.stack([p_scale.grad, p_bkg.grad], 1)
    return logL, R, g_rows, g_inst


def exact(c, seed):
    h = host_values(c, seed)
    kind = c["kind"]
    p = (h["rows"], h["scale"], h["bkg"])
    if kind in ("value", "curves"):
        logL, R, _, _ = _evaluate(c, h, *p, grad=False)
        return logL if kind == "value" else R
    if kind == "vjp":
        n = int(np.diff(h["q_off"])[h["of"]].sum())
        seeds = np.random.default_rng([int(seed), 4]).standard_normal(n)
        _, R, g_rows, g_inst = _evaluate(c, h, *p, seeds=seeds)
        return R, g_rows, g_inst[:, 0], g_inst[:, 1]
    if kind == "vi":
        mu, omega, mask, eps = vi_args(c, h, seed)
        s = np.log1p(np.exp(omega))
        at = np.where(mask, mu + s * eps, mu)
        logL, _, g_rows, g_inst = _evaluate(c, h, at[:, :-2].reshape(-1, 4), at[:, -2], at[:, -1])
        g = torch.cat([g_rows.reshape(c["items"], -1), g_inst], 1).cpu().numpy()
        slope = 1 / (1 + np.exp(-omega))
        elbo = logL.mean().cpu().numpy() + np.sum(np.log(s[mask != 0]))
        return np.array([elbo]), np.where(mask, g.mean(0), 0.0), np.where(mask, (g * eps).mean(0) * slope + slope / s, 0.0), logL
    if kind == "leapfrog":
        if steps(c) > 1e9:  # over 20 seconds
            return None
        g_rows, g_inst = (t.cpu().numpy() for t in _evaluate(c, h, *p)[2:])
        m_rows, m_inst = momenta(h, seed)
        moves = np.ones_like(h["rows"])
        moves[h["row_off"][:-1]] = (0, 1, 0, 0)
        moves[h["row_off"][1:] - 1, 0] = 0
        m_rows, m_inst = m_rows + 0.5 * DT * g_rows, m_inst + 0.5 * DT * g_inst
        rows = h["rows"] + DT * moves * np.square(UNITS) * m_rows
        inst = np.stack([h["scale"], h["bkg"]], 1) + DT * np.array((1.0, 1e-14)) * m_inst
        logL, _, g_rows, g_inst = _evaluate(c, h, rows, inst[:, 0], inst[:, 1])
        gr, gi = g_rows.cpu().numpy(), g_inst.cpu().numpy()
        return rows, inst[:, 0], inst[:, 1], m_rows + 0.5 * DT * gr, m_inst + 0.5 * DT * gi, logL, g_rows, g_inst
    logL, _, g_rows, g_inst = _evaluate(c, h, *p)
    if kind == "autograd":
        return logL, g_rows, g_inst[:, 0], g_inst[:, 1]
    if kind == "cofit":
        first, src = tie_map(h)
        v = torch.cat([g_rows.reshape(-1), g_inst.reshape(-1)]).cpu().numpy()
        return logL, np.add.reduceat(v[src], first[:-1])
    return logL, g_rows, g_inst
