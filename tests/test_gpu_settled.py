"""Time-invariant models whose covariances settle (csrc/steady*.hip): the path
taken (a word of the workspace's status block), every step against the oracle
at the parity bars, over state and measurement sizes, lengths
around the edges of chains and blocks, packed sequences shorter and longer than
the head, and models that do not settle, which the general scan takes."""
import json

import numpy as np
import pytest
import torch

import oracle
from paper_1905_13002_amd import workloads as wl

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-9, "mixed": 1e-4}
CTL = 16          # word of the status block: length of the head, 0 if the model has not settled


@pytest.fixture(scope="module")
def pks():
    from paper_1905_13002_amd import pks as p
    return p


def run(pks, model, y, precision, offsets=None):
    """(outputs, length of the head) of the combined call, or of a plan for packed sequences."""
    dt = torch.float64 if precision == "fp64" else torch.float32
    dm = pks.to_device(model)
    yd = torch.as_tensor(np.ascontiguousarray(y)).to("cuda", dt)
    if offsets is None:
        ws = pks.workspace(model.nx, model.ny, len(y), 1, precision)
        out = pks.filter_smooth(dm, yd, precision, ws=ws)
    else:
        plan = pks.Plan(dm, yd, torch.as_tensor(offsets).cuda(), precision)
        out, ws = plan.launch(), plan.ws
    torch.cuda.synchronize()
    head = int(ws[:256].cpu().numpy().view(np.int32)[CTL])
    return {k: v.double().cpu().numpy() for k, v in zip(("m", "P", "ms", "Ps"), out)}, head


def against_oracle(out, model, y, precision, offsets=None):
    y = y if precision == "fp64" else y.astype(np.float32).astype(np.float64)
    args = (model.F, model.Q, model.H, model.R, model.m0, model.P0, y)
    ref = (oracle.kf_rts(*args, u=model.u, d=model.d) if offsets is None else
           oracle.kf_rts_batched(*args, offsets, u=model.u, d=model.d, per_sequence=False))
    floor = "rms" if precision == "mixed" else "none"
    for k in ("m", "P", "ms", "Ps"):
        e = wl.max_rel_err(out[k], ref[k], floor)
        assert e <= TOL[precision], (k, e)


@pytest.mark.parametrize("nx,ny,T", [(3, 1, 466101), (4, 2, 196609), (4, 4, 196700), (4, 16, 262143), (5, 5, 8192), (7, 2, 9001), (8, 8, 12345), (9, 4, 8255), (12, 16, 8200), (13, 5, 16384),
                                     (16, 16, 8193), (16, 3, 20011),
                                     (17, 32, 8200), (24, 10, 9001), (33, 5, 8192), (48, 48, 8193), (64, 32, 8209), (64, 64, 8192)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_sizes(pks, nx, ny, T, precision):
    rng = np.random.default_rng(100 * nx + ny)
    model = wl.random_stable_model(nx, ny, rng, radius=0.9, with_offsets=True)
    w = wl.single_sequence(model, T, seed=nx)
    out, head = run(pks, model, w.y, precision)
    assert head > 0
    against_oracle(out, model, w.y, precision)
    for k in ("P", "Ps"):
        assert np.array_equal(out[k], np.swapaxes(out[k], 1, 2))
    assert np.array_equal(out["ms"][-1], out["m"][-1]) and np.array_equal(out["Ps"][-1], out["P"][-1])


@pytest.mark.parametrize("nx,ny,long", [(4, 2, 200000), (6, 6, 20000), (16, 5, 20000), (20, 6, 20000), (50, 20, 20000)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_packed(pks, nx, ny, long, precision):
    """Sequences of 0 and 1 steps, up to, at and beyond the head, between the
    head and twice the head, and at the edges of a chain and of a block."""
    rng = np.random.default_rng(7 * nx)
    model = wl.random_stable_model(nx, ny, rng, radius=0.9, with_offsets=True)
    probe = wl.single_sequence(model, long, seed=1)
    head = run(pks, model, probe.y, precision)[1]
    assert head > 0
    lengths = [0, 1, head - 1, head, head + 1, 2 * head - 1, 2 * head, 0, head + 16, head + 1024, head + 1025, 30000, 5, long]
    offsets = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    y = np.concatenate([wl.simulate(model, n, rng)[0] for n in lengths])
    out, got = run(pks, model, y, precision, offsets)
    assert got == head
    against_oracle(out, model, y, precision, offsets)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_filter_alone(pks, precision):
    """The filter alone gives the combined call's filtered moments."""
    rng = np.random.default_rng(3)
    model = wl.random_stable_model(6, 3, rng, radius=0.9)
    y = torch.as_tensor(wl.single_sequence(model, 9000, seed=2).y).to(
        "cuda", torch.float64 if precision == "fp64" else torch.float32)
    dm = pks.to_device(model)
    m, P = pks.filter(dm, y, precision)
    both = pks.filter_smooth(dm, y, precision)
    assert torch.equal(m, both[0]) and torch.equal(P, both[1])


def slow_model(nx):
    """A random walk with little noise: thousands of steps to settle."""
    return wl.Model(np.eye(nx), 1e-8 * np.eye(nx), np.eye(nx), np.eye(nx), np.ones(nx), np.eye(nx))


@pytest.mark.parametrize("model,T", [(slow_model(4), 100000), (slow_model(6), 9000), (slow_model(20), 8192),
                                     (wl.Model(np.eye(3), np.zeros((3, 3)), np.eye(3)[:2], 0.5 * np.eye(2), np.zeros(3),
                                               np.eye(3)), 240000)])
def test_models_that_do_not_settle(pks, model, T):
    """FP64 (float32 cannot hold P + Q at Q = 1e-4 P to the mixed bar)."""
    y = np.random.default_rng(5).standard_normal((T, model.ny))
    out, head = run(pks, model, y, "fp64")
    assert head == 0
    against_oracle(out, model, y, "fp64")


@pytest.mark.parametrize("ept,ept1", [(4, 0), (8, 2), (16, 1)])
def test_general_scan_configurations(pks, tmp_path, monkeypatch, ept, ept1):
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({"nx4_ny4_fp64_T16_B0": [ept, ept1]}))
    monkeypatch.setenv("PKS_TUNE_CACHE", str(cache))
    model, y = slow_model(4), np.random.default_rng(6).standard_normal((100001, 4))
    out, head = run(pks, model, y, "fp64")
    assert head == 0
    against_oracle(out, model, y, "fp64")


@pytest.mark.parametrize("nx", [4, 9, 20])
def test_priors(pks, nx):
    """A known start (P0 = 0) and one far above the settled covariance (the
    oracle's own update P - K S K^T loses |P0|^2 of the rounding: 6e-6 at 1e6 I
    against extended precision, 1e-12 at 100 I)."""
    rng = np.random.default_rng(11)
    model = wl.random_stable_model(nx, 3, rng, radius=0.9, with_offsets=True)
    y = wl.single_sequence(model, 100000, seed=4).y
    for P0 in (np.zeros((nx, nx)), 100.0 * np.eye(nx)):
        mo = wl.Model(model.F, model.Q, model.H, model.R, model.m0, P0, model.u, model.d)
        out, head = run(pks, mo, y, "fp64")
        assert head > 0
        against_oracle(out, mo, y, "fp64")


def test_nan_and_failed_models(pks):
    rng = np.random.default_rng(12)
    model = wl.random_stable_model(6, 2, rng, radius=0.9)
    y = wl.single_sequence(model, 9000, seed=5).y.copy()
    y[5000, 1] = np.nan
    out, head = run(pks, model, y, "fp64")
    assert head > 0
    assert np.isfinite(out["m"][:5000]).all() and np.isnan(out["m"][5000:]).all()
    assert np.isnan(out["ms"]).all() and np.isfinite(out["P"]).all() and np.isfinite(out["Ps"]).all()
    bad = wl.Model(model.F, model.Q, model.H, -10.0 * np.eye(2), model.m0, model.P0)
    ws = pks.workspace(6, 2, 9000)
    m, _ = pks.filter(pks.to_device(bad), torch.as_tensor(y).cuda(), "fp64", ws=ws)
    assert pks.read_numeric_status(ws) == (False, 0) and torch.isnan(m).all()


# ---------------------------------------------------------------------------
# the smoother alone (nx > 16) of covariances that are the filter's own
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("nx,ny,lengths,precision", [(17, 5, [9000], "fp64"), (24, 10, [3000, 1, 700, 5001], "mixed"),
                                                     (33, 20, [8193], "mixed"), (64, 32, [2000, 6400], "fp64")])
def test_smoother_alone(pks, nx, ny, lengths, precision):
    rng = np.random.default_rng(nx)
    model = wl.random_stable_model(nx, ny, rng, radius=0.9, with_offsets=True)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    T = int(off[-1])
    y = rng.standard_normal((T, ny))
    dt = torch.float64 if precision == "fp64" else torch.float32
    dm, yd, offd = pks.to_device(model), torch.as_tensor(y).to("cuda", dt), torch.as_tensor(off).cuda()
    ws = pks.workspace(nx, ny, T, len(lengths), precision)
    word = lambda: int(ws[:256].cpu().numpy().view(np.int32)[CTL])
    m, P = pks.filter_batched(dm, offd, yd, precision, ws=ws)
    ms, Ps = pks.smooth_batched(dm, offd, m, P, precision, ws=ws)
    torch.cuda.synchronize()
    assert word() > 0
    yy = y if precision == "fp64" else y.astype(np.float32).astype(np.float64)
    for s, e in zip(off[:-1], off[1:]):
        ref = oracle.kf_rts(model.F, model.Q, model.H, model.R, model.m0, model.P0, yy[s:e], u=model.u, d=model.d)
        for k, v in zip(("ms", "Ps"), (ms, Ps)):
            err = wl.max_rel_err(v[s:e].double().cpu().numpy(), ref[k], "rms" if precision == "mixed" else "none")
            assert err <= TOL[precision], (s, k, err)
    # covariances that are not the filter's, by one bit of one entry early or late: the general kernels
    for row in (1, T - 400):
        Q = P.clone()
        Q[row, 1, 1] *= 1 + 2 * torch.finfo(dt).eps
        m2, P2 = pks.smooth_batched(dm, offd, m, Q, precision, ws=ws)
        torch.cuda.synchronize()
        assert word() == 0
        assert (P2 - Ps).abs().max() <= TOL[precision] * Ps.abs().max()
        assert (m2 - ms).abs().max() <= TOL[precision] * ms.abs().max()


@pytest.mark.parametrize("nx,lengths", [(6, [8192]), (16, [10007]), (9, [3001, 1, 2000, 0, 6000]), (16, [1024] * 9)])
def test_general_scan_behind_a_failed_attempt(pks, nx, lengths):
    """4 < nx <= 16, covariances that do not settle: scan levels of four."""
    rng = np.random.default_rng(nx)
    model = wl.random_stable_model(nx, nx // 2, rng)
    model = wl.Model(np.eye(nx), 1e-4 * np.eye(nx), model.H, model.R, model.m0, model.P0)
    off = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)
    y = rng.standard_normal((int(off[-1]), nx // 2))
    out, head = run(pks, model, y, "fp64", off if len(lengths) > 1 else None)
    assert head == 0
    for s, e in zip(off[:-1], off[1:]):
        if s < e:
            against_oracle({k: v[s:e] for k, v in out.items()}, model, y[s:e], "fp64")
