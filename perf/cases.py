"""What the library is timed on: filter + smoother, marginal likelihood and
discrete-state passes over the sizes that its users and its own workloads have.

A case is a dict of plain values:
  kind   "cv"         one constant-velocity track (nx = 4, ny = 2): pks.filter_smooth
         "small"      one sequence of a generic model with nx, ny <= 4: pks.filter, then pks.smooth
         "cv_plan"    many uneven tracks, one model each, packed into one captured pks.Plan
         "cv_loglik"  many uneven tracks, one model each: pks.filter_batched + pks.loglik_batched
         "irregular"  one constant-velocity track sampled at irregular times (time-varying model)
         "random"     one sequence of a random stable model with nx >= 5: pks.filter_smooth
         "random_plan"   packed uneven sequences of one random stable model, captured pks.Plan
         "random_eager"  the same through pks.filter_batched and pks.smooth_batched
         "hmm"        one sequence of a discrete-state model: pks.hmm_filter_smooth
  prec   "fp64" or "mixed" (float32 storage)
  nx, ny, T            sizes of one sequence (K states for "hmm")
  B, lo, hi            packed sequences: their number and the range of their lengths

Every case keeps what a program that calls in a loop keeps: the device model,
the workspace and the output buffers.
"""
import numpy as np
import torch

from paper_1905_13002_amd import workloads as wl


def listed():
    return [
        # the smallest call: a short track, all latency
        {"name": "cv_1k_fp64", "kind": "cv", "prec": "fp64", "nx": 4, "ny": 2, "T": 1024},
        # the benchmark workload
        {"name": "cv_1m_fp64", "kind": "cv", "prec": "fp64", "nx": 4, "ny": 2, "T": 1 << 20},
        # the same in float32 storage, at a length that fills no tile
        {"name": "cv_1m_mixed", "kind": "cv", "prec": "mixed", "nx": 4, "ny": 2, "T": 1000003},
        # a local linear trend, filtered first and smoothed later
        {"name": "small_nx2_fp64", "kind": "small", "prec": "fp64", "nx": 2, "ny": 1, "T": 100003},
        # a batch of uneven tracks replayed as one captured pass
        {"name": "cv_plan_mixed", "kind": "cv_plan", "prec": "mixed", "nx": 4, "ny": 2, "B": 1024, "lo": 256, "hi": 16384},
        # likelihoods of many tracks under their own parameters
        {"name": "cv_loglik_fp64", "kind": "cv_loglik", "prec": "fp64", "nx": 4, "ny": 2, "B": 300, "lo": 64, "hi": 4096},
        # a model that changes at every step
        {"name": "irregular_1m_fp64", "kind": "irregular", "prec": "fp64", "nx": 4, "ny": 2, "T": 1 << 20},
        # a state of the largest size that stays in registers
        {"name": "random_nx16_fp64", "kind": "random", "prec": "fp64", "nx": 16, "ny": 8, "T": 1 << 16},
        # an ordinary mid-size state, odd length
        {"name": "random_nx6_mixed", "kind": "random", "prec": "mixed", "nx": 6, "ny": 3, "T": 20011},
        # the largest state, uneven sequences replayed as one captured pass
        {"name": "random_nx64_plan_fp64", "kind": "random_plan", "prec": "fp64", "nx": 64, "ny": 32, "B": 16, "lo": 512, "hi": 8192},
        # a large state through the separate batched calls
        {"name": "random_nx24_mixed", "kind": "random_eager", "prec": "mixed", "nx": 24, "ny": 10, "B": 40, "lo": 100, "hi": 2000},
        # the discrete-state pass
        {"name": "hmm_64_fp64", "kind": "hmm", "prec": "fp64", "nx": 64, "ny": 1, "T": 1 << 16},
    ]


def _spread(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["cv", "cv", "small", "cv_plan", "cv_loglik", "irregular", "random", "random_plan",
                       "random_eager", "hmm"])
    prec = rng.choice(["fp64", "mixed"])
    c = {"kind": kind, "prec": prec, "nx": 4, "ny": 2}
    if kind in ("cv", "irregular"):
        c["T"] = _spread(rng, 1000, 1 << 20)
    elif kind == "small":
        c.update(nx=rng.randint(1, 4), ny=rng.randint(1, 4), T=_spread(rng, 1000, 200000))
    elif kind in ("cv_plan", "cv_loglik"):
        hi = _spread(rng, 1024, 16384)
        c.update(B=_spread(rng, 16, 1024), lo=hi // 64, hi=hi)
    elif kind == "random":
        nx = rng.randint(5, 16)
        c.update(nx=nx, ny=rng.randint(1, nx), T=_spread(rng, 2000, 1 << 16))
    elif kind in ("random_plan", "random_eager"):
        nx = _spread(rng, 5, 64)
        hi = _spread(rng, 512, 8192)
        most = max(2, min(64, (16 * 8192 * 64) // (hi * nx)))    # no larger than the largest listed case
        c.update(nx=nx, ny=rng.randint(1, min(nx, 32)), B=_spread(rng, 2, most), lo=max(1, hi // 16), hi=hi)
    else:
        c.update(prec="fp64", nx=_spread(rng, 2, 64), ny=1, T=_spread(rng, 1000, 1 << 16))
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _offsets(case):
    """Packed sequences: the lengths belong to the case, not to the seed."""
    n = np.random.default_rng([case["B"], case["lo"], case["hi"]]).integers(case["lo"], case["hi"], size=case["B"],
                                                                            endpoint=True)
    return np.concatenate([[0], np.cumsum(n)]).astype(np.int64)


def _tracks(offsets, q, r, rng):
    """Constant-velocity measurements of packed sequences (velocity a random walk, position its sum)."""
    total, B = int(offsets[-1]), len(offsets) - 1
    seq = np.repeat(np.arange(B), np.diff(offsets))
    dt = 0.1
    z = rng.standard_normal((total, 2, 2))
    qv = np.sqrt(q[seq] * dt)[:, None] * z[:, 0]
    qp = 0.5 * dt * qv + np.sqrt(q[seq] * dt ** 3 / 12)[:, None] * z[:, 1]

    def within(a):          # running sums that start again with every sequence
        s = np.cumsum(a, axis=0)
        before = np.vstack([np.zeros((1, 2)), s])[offsets[:-1]]
        return s - before[seq]

    v0 = rng.standard_normal((B, 2))
    v = v0[seq] + within(qv)
    pos = rng.standard_normal((B, 2))[seq] + within(dt * (v - qv) + qp)
    return pos + np.sqrt(r[seq])[:, None] * rng.standard_normal((total, 2))


def _simulate(model, offsets, rng):
    """Packed sequences of one model, all of them stepped together."""
    n = np.diff(offsets)
    B, nx = len(n), model.nx
    LQ, LR, L0 = (np.linalg.cholesky(X) for X in (model.Q, model.R, model.P0))
    u = 0.0 if model.u is None else model.u
    d = 0.0 if model.d is None else model.d
    x = model.m0 + rng.standard_normal((B, nx)) @ L0.T
    X = np.empty((int(offsets[-1]), nx))
    noise = rng.standard_normal((int(offsets[-1]), nx)) @ LQ.T
    FT = np.ascontiguousarray(model.F.T)
    order = np.argsort(-n, kind="stable")            # the sequences still running come first
    x, at = x[order], offsets[:-1][order]
    for k in range(int(n.max())):
        a = int(np.count_nonzero(n > k))
        x = x[:a] @ FT + u + noise[at[:a] + k]
        X[at[:a] + k] = x
    return X @ model.H.T + d + rng.standard_normal((X.shape[0], model.ny)) @ LR.T


def _inputs(case, seed):
    """(model, offsets, y, one model per sequence?, time-varying?) as float64 numpy arrays."""
    rng = np.random.default_rng([seed, 20])
    kind = case["kind"]
    if kind == "cv":
        y, _ = wl.simulate_cv(1.0, 0.25, case["T"], rng)
        return wl.cv_model(1.0, 0.25), None, y, False, False
    if kind == "irregular":
        dts = rng.uniform(0.05, 0.15, size=case["T"])
        y, _ = wl.simulate_cv_tv(dts, 1.0, 0.25, rng)
        return wl.cv_model_tv(dts, 1.0, 0.25), None, y, False, True
    if kind in ("cv_plan", "cv_loglik"):
        offsets = _offsets(case)
        q, r = rng.uniform(0.1, 10.0, size=case["B"]), rng.uniform(0.01, 1.0, size=case["B"])
        each = [wl.cv_model(q[b], r[b]) for b in range(case["B"])]
        model = wl.Model(*(np.stack([getattr(m, f) for m in each]) for f in ("F", "Q", "H", "R", "m0", "P0")))
        return model, offsets, _tracks(offsets, q, r, rng), True, False
    if kind == "small":
        model, offsets = wl.random_small_model(case["nx"], case["ny"], rng), np.array([0, case["T"]])
        return model, None, _simulate(model, offsets, rng), False, False
    model = wl.random_stable_model(case["nx"], case["ny"], rng, radius=0.99, with_offsets=True)
    if kind == "random":
        return model, None, _simulate(model, np.array([0, case["T"]]), rng), False, False
    offsets = _offsets(case)
    return model, offsets, _simulate(model, offsets, rng), False, False


def _hmm_inputs(case, seed):
    rng = np.random.default_rng([seed, 21])
    Pi, p0 = wl.hmm_model(case["nx"], rng)
    return Pi, p0, wl.hmm_simulate(Pi, p0, case["T"], rng)[0]


def prepare(case, seed):
    from paper_1905_13002_amd import pks
    if case["kind"] == "hmm":
        Pi, p0, L = _hmm_inputs(case, seed)
        K, T = case["nx"], case["T"]
        new = lambda *s: torch.empty(s, dtype=torch.float64, device="cuda")
        return {"kind": "hmm", "model": pks.hmm_to_device(Pi, p0), "L": torch.as_tensor(L).cuda(),
                "ws": pks.hmm_workspace(K, T), "out": (new(T, K), new(T), new(T, K))}
    model, offsets, y, each, tv = _inputs(case, seed)
    prec, nx, total = case["prec"], case["nx"], len(y)
    rt = torch.float64 if prec == "fp64" else torch.float32
    s = {"kind": case["kind"], "prec": prec, "model": pks.to_device(model, per_sequence=each, time_varying=tv),
         "y": torch.as_tensor(y).to("cuda", rt)}
    if offsets is not None:
        s["offsets"] = torch.as_tensor(offsets).cuda()
    if case["kind"].endswith("_plan"):
        s["plan"] = pks.Plan(s["model"], s["y"], s["offsets"], prec)
        return s
    s["ws"] = pks.workspace(nx, case["ny"], total, 1 if offsets is None else case["B"], prec, time_varying=tv)
    new = lambda: (torch.empty((total, nx), dtype=rt, device="cuda"), torch.empty((total, nx, nx), dtype=rt, device="cuda"))
    s["filtered"] = new()
    if case["kind"] != "cv_loglik":
        s["smoothed"] = new()
    return s


def run(s):
    from paper_1905_13002_amd import pks
    kind = s["kind"]
    if kind == "hmm":
        return pks.hmm_filter_smooth(s["model"], s["L"], ws=s["ws"], out=s["out"])
    if "plan" in s:
        return s["plan"].launch()
    model, y, prec, ws = s["model"], s["y"], s["prec"], s["ws"]
    if kind == "cv_loglik":
        m, P = pks.filter_batched(model, s["offsets"], y, prec, ws=ws, out=s["filtered"])
        ll, total = pks.loglik_batched(model, s["offsets"], y, m, P, prec, ws=ws)
        return m, P, ll, total
    if kind == "random_eager":
        m, P = pks.filter_batched(model, s["offsets"], y, prec, ws=ws, out=s["filtered"])
        ms, Ps = pks.smooth_batched(model, s["offsets"], m, P, prec, ws=ws, out=s["smoothed"])
        return m, P, ms, Ps
    if kind == "small":
        m, P = pks.filter(model, y, prec, ws=ws, out=s["filtered"])
        ms, Ps = pks.smooth(model, m, P, prec, ws=ws, out=s["smoothed"])
        return m, P, ms, Ps
    return pks.filter_smooth(model, y, prec, ws=ws, out=s["filtered"] + s["smoothed"])


def work(case):
    """Inputs read once, outputs written once; flops of the sequential recursions."""
    n, q = case["nx"], case["ny"]
    if case["kind"] == "hmm":
        return {"bytes": 8 * (case["T"] * (3 * n + 1) + n * n + n), "flops": case["T"] * (2 * n * n + 4 * n * n + 8 * n)}
    T = case["T"] if "T" in case else int(_offsets(case)[-1])
    r = 8 if case["prec"] == "fp64" else 4
    each = case["B"] if case["kind"] in ("cv_plan", "cv_loglik") else 1
    rows = T if case["kind"] == "irregular" else each
    model = 8 * (rows * (2 * n * n + n * q + q * q) + each * (n * n + n))
    predict_update = 4 * n ** 3 + 2 * n * n + 4 * n * n * q + 2 * n * q * q + q ** 3 // 3 + 4 * n * q
    smooth = n ** 3 // 3 + 2 * n ** 3 + 4 * n ** 3 + 4 * n * n
    if case["kind"] == "cv_loglik":
        return {"bytes": T * (r * (q + n + n * n) + 8) + model + 8 * each,
                "flops": T * (predict_update + 4 * n * n * q + 2 * n * q * q)}
    return {"bytes": T * r * (q + 2 * (n + n * n)) + model, "flops": T * (predict_update + smooth)}


# ---------------------------------------------------------------------------
# the same results in 64 bits: elements of the filter and of the smoother
# combined by recursive doubling in plain torch
# ---------------------------------------------------------------------------
def _mm(X, Y):
    if max(X.shape[-2:] + Y.shape[-2:]) <= 8:
        return (X.unsqueeze(-1) * Y.unsqueeze(-3)).sum(-2)
    return torch.matmul(X.contiguous(), Y.contiguous())


def _mv(X, v):
    return (X * v.unsqueeze(-2)).sum(-1)


def _t(X):
    return X.transpose(-1, -2)


def _sym(X):
    return 0.5 * (X + _t(X))


def _inv(M):
    """Batched Gauss-Jordan inverse and one Newton step."""
    n = M.shape[-1]
    W = M.clone()
    for k in range(n):
        row = W[..., k, :].clone()
        p = 1.0 / row[..., k]
        row *= p.unsqueeze(-1)
        row[..., k] = p
        col = W[..., :, k].clone()
        col[..., k] = 0.0
        W[..., :, k] = 0.0
        W[..., k, :] = 0.0
        W -= col.unsqueeze(-1) * row.unsqueeze(-2)
        W[..., k, :] = row
    I = torch.eye(n, dtype=M.dtype, device=M.device)
    return W + _mm(W, I - _mm(M, W))


def _kalman(F, u, Q, H, d, R, m, P, y):
    """One prediction and update from (m, P), every step at once."""
    mp, Pp = _mv(F, m) + u, _sym(_mm(_mm(F, P), _t(F))) + Q
    S = _sym(_mm(_mm(H, Pp), _t(H))) + R
    K = _mm(_mm(Pp, _t(H)), _inv(S))
    v = y - _mv(H, mp) - d
    return mp + _mv(K, v), _sym(Pp - _mm(_mm(K, S), _t(K))), v, S


def _exact_filter(rows, m0, P0, first, longest, y):
    F, u, Q, H, d, R = rows
    n = F.shape[-1]
    S = _sym(_mm(_mm(H, Q), _t(H))) + R
    Si = _sym(_inv(S))
    K = _mm(_mm(Q, _t(H)), Si)
    HF = _mm(H, F)
    W = _mm(_t(HF), Si)
    v = y - _mv(H, u.expand(y.shape[0], n)) - d
    A, b, C = F - _mm(K, HF), u + _mv(K, v), _sym(Q - _mm(_mm(K, S), _t(K)))
    eta, J = _mv(W, v), _sym(_mm(W, HF))
    m1, P1, v1, S1 = _kalman(F[first], u[first], Q[first], H[first], d[first], R[first], m0, P0, y[first])
    A, J, C = A.clone(), J.clone(), C.clone()
    A[first], b[first], C[first], eta[first], J[first] = 0.0, m1, P1, 0.0, 0.0
    I = torch.eye(n, dtype=y.dtype, device=y.device)
    step = 1
    while step < longest:
        Ai, bi, Ci, ei, Ji = (x[:-step] for x in (A, b, C, eta, J))
        Aj, bj, Cj, ej, Jj = (x[step:] for x in (A, b, C, eta, J))
        X = _inv(I + _mm(Ci, Jj))
        AX = _mm(Aj, X)
        XA = _mm(X, Ai)
        new = (_mm(AX, Ai), _mv(AX, bi + _mv(Ci, ej)) + bj, _sym(_mm(_mm(AX, Ci), _t(Aj))) + Cj,
               _mv(_t(XA), ej - _mv(Jj, bi)) + ei, _sym(_mm(_t(XA), _mm(Jj, Ai))) + Ji)
        A, b, C, eta, J = (torch.cat([x[:step], z]) for x, z in zip((A, b, C, eta, J), new))
        step *= 2
    # one prediction and update from the step before
    mb, Pb = torch.cat([b[:1], b[:-1]]), torch.cat([C[:1], C[:-1]])
    mb[first], Pb[first] = m0, P0
    return _kalman(F, u, Q, H, d, R, mb, Pb, y)


def _exact_smoother(rows, m, P, last, longest):
    F, u, Q = (torch.cat([x[1:], x[:1]]) for x in rows[:3])     # the transition out of a step
    FP = _mm(F, P)
    E = _t(_mm(_inv(_sym(_mm(FP, _t(F))) + Q), FP)).contiguous()
    g, L = m - _mv(E, _mv(F, m) + u), _sym(P - _mm(E, FP))
    E[last], g[last], L[last] = 0.0, m[last], P[last]
    step = 1
    while step < longest:
        Ei, gi, Li = (x[:-step] for x in (E, g, L))
        Ej, gj, Lj = (x[step:] for x in (E, g, L))
        new = (_mm(Ei, Ej), _mv(Ei, gj) + gi, _sym(_mm(_mm(Ei, Lj), _t(Ei))) + Li)
        E, g, L = (torch.cat([z, x[-step:]]) for x, z in zip((E, g, L), new))
        step *= 2
    return g, L


def _exact_hmm(case, seed):
    Pi, p0, L = _hmm_inputs(case, seed)
    T, K = L.shape
    alpha, logp, gamma, run_ = np.empty((T, K)), np.empty(T), np.empty((T, K)), 0.0
    w = np.exp(L - L.max(axis=1, keepdims=True))
    top = L.max(axis=1)
    a = p0
    for k in range(T):
        a = (a @ Pi) * w[k]
        s = a.sum()
        a = a / s
        alpha[k] = a
        run_ += np.log(s) + top[k]
        logp[k] = run_
    g = gamma[T - 1] = alpha[T - 1]
    for k in range(T - 2, -1, -1):
        pred = alpha[k] @ Pi
        g = gamma[k] = alpha[k] * (Pi @ np.divide(g, pred, out=np.zeros(K), where=pred > 0))
    return alpha, logp, gamma


def exact(case, seed):
    if case["kind"] == "hmm":
        return _exact_hmm(case, seed)
    model, offsets, y, each, tv = _inputs(case, seed)
    if case["prec"] != "fp64":
        y = y.astype(np.float32).astype(np.float64)
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    cv = lambda a: torch.as_tensor(np.ascontiguousarray(a)).to(dev)
    T, n, q = len(y), case["nx"], case["ny"]
    off = np.array([0, T]) if offsets is None else offsets
    full = off[:-1][np.diff(off) > 0]
    first, last = cv(full), cv(off[1:][np.diff(off) > 0] - 1)
    longest = int(np.diff(off).max())
    u = np.zeros(model.F.shape[:-1]) if model.u is None else model.u
    d = np.zeros(model.H.shape[:-1]) if model.d is None else model.d
    rows = [cv(a) for a in (model.F, u, model.Q, model.H, d, model.R)]
    if each:
        seq = cv(np.repeat(np.arange(len(off) - 1), np.diff(off)))
        rows = [a[seq] for a in rows]
    elif not tv:
        rows = [a.expand((T,) + a.shape) for a in rows]
    m0, P0 = cv(model.m0), cv(model.P0)
    if each:
        m0, P0 = m0[seq[first]], P0[seq[first]]
    m, P, v, S = _exact_filter(rows, m0, P0, first, longest, cv(y))
    if case["kind"] == "cv_loglik":
        # of the 2 x 2 innovation covariance
        det = S[:, 0, 0] * S[:, 1, 1] - S[:, 0, 1] * S[:, 1, 0]
        ll = -0.5 * (q * np.log(2 * np.pi) + torch.log(det) + (v * _mv(_inv(S), v)).sum(-1))
        return m, P, ll, torch.zeros(case["B"], dtype=torch.float64, device=dev).index_add_(0, seq, ll)
    return (m, P) + _exact_smoother(rows, m, P, last, longest)
