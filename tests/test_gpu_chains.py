"""Time-varying models, and packed sequences with a model each, by overlapped
chains (csrc/chains.hip): the path taken
(a word of the workspace's status block), every step against the oracle at the
parity bars, for every size that takes the path, lengths around the edges of
chains and groups of steps, packed sequences shorter and longer than a chain,
the filter alone; models that do not forget and failing factorisations go to
the general scan."""
import numpy as np
import pytest

import oracle
from paper_1905_13002_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-9, "mixed": 1e-4}
CTL = 16          # word of the status block: 1 if the chains have done the work
SHORT = {"fp64": 1 << 18, "mixed": 1 << 19}


@pytest.fixture(scope="module")
def pks():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13002_amd import pks as mod
    return mod


def varying(nx, ny, T, seed, offsets_too=True):
    """Rows of a few random models, mixed over the steps."""
    rng = np.random.default_rng(seed)
    some = [wl.random_small_model(nx, ny, rng) for _ in range(5)]
    pick = rng.integers(0, 5, size=T)
    row = lambda f: np.stack([getattr(m, f) for m in some])[pick]
    u, d = (row("u"), row("d")) if offsets_too and some[0].u is not None else (None, None)
    return wl.Model(row("F"), row("Q"), row("H"), row("R"), some[0].m0, some[0].P0, u, d), rng.standard_normal((T, ny))


def dev(y, precision):
    return torch.as_tensor(np.ascontiguousarray(y)).to("cuda", torch.float64 if precision == "fp64" else torch.float32)


def run(pks, model, y, precision):
    dm, yd = pks.to_device(model, time_varying=True), dev(y, precision)
    ws = pks.workspace(model.m0.shape[-1], y.shape[1], len(y), 1, precision, time_varying=True)
    out = pks.filter_smooth(dm, yd, precision, ws=ws)
    torch.cuda.synchronize()
    return out, int(ws[:256].cpu().numpy().view(np.int32)[CTL]), dm, yd, ws


def check(model, y, out, precision):
    yy = y if precision == "fp64" else y.astype(np.float32).astype(np.float64)
    ref = oracle.kf_rts_tv(model.F, model.Q, model.H, model.R, model.m0, model.P0, yy, u=model.u, d=model.d)
    for k, v in zip(("m", "P", "ms", "Ps"), out):
        e = wl.max_rel_err(v.double().cpu().numpy(), ref[k], "rms" if precision == "mixed" else "none")
        assert e <= TOL[precision], (k, e)


@pytest.mark.parametrize("nx,ny,extra,precision", [(3, 1, 0, "fp64"), (3, 2, 1, "fp64"), (3, 3, 77, "mixed"),
                                                   (4, 1, 66, "fp64"), (4, 2, 3, "mixed"), (4, 3, 4098, "fp64"),
                                                   (4, 4, 5, "fp64")])
def test_sizes(pks, nx, ny, extra, precision):
    model, y = varying(nx, ny, SHORT[precision] + extra, seed=10 * nx + ny)
    out, ctl, dm, yd, ws = run(pks, model, y, precision)
    assert ctl == 1
    check(model, y, out, precision)
    P = out[1].cpu()
    assert torch.equal(P, P.transpose(1, 2))
    m, P = pks.filter(dm, yd, precision, ws=ws)
    assert torch.equal(m, out[0]) and torch.equal(P, out[1])


def test_packed_sequences(pks):
    """Lengths of one step up to many chains, an empty one, a prior each."""
    lengths = [1, 63, 64, 65, 0, 191, 257, 4097, 100000, 2, 130000, 40000]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    T, B = int(offsets[-1]), len(lengths)
    assert T >= SHORT["fp64"]
    model, y = varying(4, 2, T, seed=3)
    rng = np.random.default_rng(4)
    model.m0 = rng.standard_normal((B, 4))
    model.P0 = np.stack([np.eye(4) * s for s in rng.uniform(0.5, 2.0, size=B)])
    dm = pks.to_device(model, time_varying=True, per_sequence=True)
    off = torch.as_tensor(offsets).cuda()
    plan = pks.Plan(dm, dev(y, "fp64"), off, "fp64")
    for _ in range(3):
        out = plan.launch()
        torch.cuda.synchronize()
        assert int(plan.ws[:256].cpu().numpy().view(np.int32)[CTL]) == 1
    for b, (s, e) in enumerate(zip(offsets[:-1], offsets[1:])):
        if s == e:
            continue
        r = lambda a: None if a is None else a[s:e]
        ref = oracle.kf_rts_tv(r(model.F), r(model.Q), r(model.H), r(model.R), model.m0[b], model.P0[b], y[s:e],
                               u=r(model.u), d=r(model.d))
        for k, v in zip(("m", "P", "ms", "Ps"), out):
            assert wl.max_rel_err(v[s:e].cpu().numpy(), ref[k]) <= TOL["fp64"], (b, k)


def test_models_that_do_not_forget(pks):
    """A constant state seen through large noise: the gains fall like 1 / k."""
    T = SHORT["fp64"]
    tile = lambda a: np.broadcast_to(a, (T,) + a.shape).copy()
    model = wl.Model(tile(np.eye(4)), tile(1e-12 * np.eye(4)), tile(np.eye(2, 4)), tile(1e2 * np.eye(2)),
                     np.zeros(4), np.eye(4))
    y = np.random.default_rng(5).standard_normal((T, 2))
    out, ctl, _, _, _ = run(pks, model, y, "fp64")
    assert ctl == 0
    ref = oracle.kf_rts_tv(model.F, model.Q, model.H, model.R, model.m0, model.P0, y)
    for k, v in zip(("P", "Ps"), (out[1], out[3])):
        assert wl.max_rel_err(v.cpu().numpy(), ref[k]) <= TOL["fp64"], k


def test_failing_factorisation_is_flagged(pks):
    model, y = varying(4, 2, SHORT["fp64"], seed=6)
    model.R[200001] = -50.0 * np.eye(2)
    out, ctl, _, _, ws = run(pks, model, y, "fp64")
    assert ctl == 0
    ok, first = pks.read_numeric_status(ws)
    assert not ok and first == 0


# ---------------------------------------------------------------------------
# one time-invariant model per sequence
# ---------------------------------------------------------------------------
def each(nx, ny, lengths, seed, model=None):
    rng = np.random.default_rng(seed)
    def draw():                                  # forgets fast enough: noise in every direction, all of it seen
        m = wl.random_small_model(nx, ny, rng)
        return wl.Model(0.8 * m.F, m.Q, m.H, m.R, m.m0, m.P0, m.u, m.d)
    models = [(model or draw)() for _ in lengths]
    row = lambda f: None if getattr(models[0], f) is None else np.stack([getattr(m, f) for m in models])
    packed = wl.Model(*(row(f) for f in ("F", "Q", "H", "R", "m0", "P0", "u", "d")))
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    return models, packed, offsets, rng.standard_normal((int(offsets[-1]), ny))


def run_each(pks, packed, offsets, y, precision):
    dm, yd, off = pks.to_device(packed, per_sequence=True), dev(y, precision), torch.as_tensor(offsets).cuda()
    plan = pks.Plan(dm, yd, off, precision)
    for _ in range(3):
        out = plan.launch()
        torch.cuda.synchronize()
    return out, int(plan.ws[:256].cpu().numpy().view(np.int32)[CTL]), dm, yd, off


LENGTHS = [1, 15, 0, 16, 17, 300, 1041, 2, 4097, 131072, 33001, 70000]


@pytest.mark.parametrize("nx,ny,precision", [(3, 1, "fp64"), (3, 3, "mixed"), (4, 1, "mixed"), (4, 2, "fp64"),
                                             (4, 3, "fp64"), (4, 4, "mixed")])
def test_each_its_model(pks, nx, ny, precision):
    """Sequences of one step, of less than a head, of many chains, an empty one."""
    lengths = LENGTHS + [600003 if precision == "fp64" else 1400003]
    models, packed, offsets, y = each(nx, ny, lengths, seed=100 * nx + ny)
    out, ctl, dm, yd, off = run_each(pks, packed, offsets, y, precision)
    assert ctl == 1
    yy = y if precision == "fp64" else y.astype(np.float32).astype(np.float64)
    for b, (s, e) in enumerate(zip(offsets[:-1], offsets[1:])):
        if s == e:
            continue
        mo = models[b]
        ref = oracle.kf_rts(mo.F, mo.Q, mo.H, mo.R, mo.m0, mo.P0, yy[s:e], u=mo.u, d=mo.d)
        for k, v in zip(("m", "P", "ms", "Ps"), out):
            err = wl.max_rel_err(v[s:e].double().cpu().numpy(), ref[k], "rms" if precision == "mixed" else "none")
            assert err <= TOL[precision], (b, k, err)
    m, P = pks.filter_batched(dm, off, yd, precision)
    assert torch.equal(m, out[0]) and torch.equal(P, out[1])


@pytest.mark.parametrize("q", [0.0, 1e-9])
def test_each_its_model_that_settles_late(pks, q):
    """One model of a constant (nearly constant) state among them: the general scan."""
    lengths = [200000, 3000, 300000, 400000]
    models, packed, offsets, y = each(4, 2, lengths, seed=9)
    packed.F[1], packed.Q[1] = np.eye(4), q * np.eye(4)
    out, ctl, _, _, _ = run_each(pks, packed, offsets, y, "fp64")
    assert ctl == 0
    mo, (s, e) = models[3], offsets[3:5]
    ref = oracle.kf_rts(mo.F, mo.Q, mo.H, mo.R, mo.m0, mo.P0, y[s:e], u=mo.u, d=mo.d)
    for k, v in zip(("m", "P", "ms", "Ps"), out):
        assert wl.max_rel_err(v[s:e].cpu().numpy(), ref[k]) <= TOL["fp64"], k
