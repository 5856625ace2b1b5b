"""Short sequences of nx = 3, 4 with one and two steps a thread: lengths around
waves, workgroups and the ends of the two ranges, against the oracle at the
parity bars; the workspace never shrinks as the length grows, so one sized for
a longer sequence is still taken."""
import numpy as np
import pytest

import oracle
from paper_1905_13002_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-9, "mixed": 1e-4}


@pytest.fixture(scope="module")
def pks():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13002_amd import pks as mod
    return mod


@pytest.mark.parametrize("nx,ny,T", [(4, 2, 1), (4, 1, 2), (4, 2, 63), (3, 2, 64), (4, 4, 65), (3, 3, 256), (4, 2, 257),
                                     (4, 3, 4099), (3, 1, 32768), (4, 2, 32769), (3, 2, 65537), (4, 1, 65536)])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_lengths(pks, nx, ny, T, precision):
    rng = np.random.default_rng(1000 * nx + T)
    model = wl.random_small_model(nx, ny, rng)
    y = rng.standard_normal((T, ny))
    dt = torch.float64 if precision == "fp64" else torch.float32
    dm, yd = pks.to_device(model), torch.as_tensor(y).to("cuda", dt)
    ws = pks.workspace(nx, ny, T, 1, precision)
    out = pks.filter_smooth(dm, yd, precision, ws=ws)
    torch.cuda.synchronize()
    yy = y if precision == "fp64" else y.astype(np.float32).astype(np.float64)
    ref = oracle.kf_rts(model.F, model.Q, model.H, model.R, model.m0, model.P0, yy, u=model.u, d=model.d)
    for k, v in zip(("m", "P", "ms", "Ps"), out):
        e = wl.max_rel_err(v.double().cpu().numpy(), ref[k], "rms" if precision == "mixed" else "none")
        assert e <= TOL[precision], (k, e)
    m, P = pks.filter(dm, yd, precision, ws=ws)
    ms, Ps = pks.smooth(dm, m, P, precision, ws=ws)
    torch.cuda.synchronize()
    for k, v in zip(("m", "P", "ms", "Ps"), (m, P, ms, Ps)):
        e = wl.max_rel_err(v.double().cpu().numpy(), ref[k], "rms" if precision == "mixed" else "none")
        assert e <= TOL[precision], (k, e)


@pytest.mark.parametrize("nx", [2, 3, 4])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_workspace_grows_with_the_length(pks, nx, precision):
    T = sorted(set([1, 100, 300000] + [b + d for b in (1 << 14, 1 << 15, 1 << 16, 98304, 1 << 17, 1 << 18) for d in (-1, 0, 1)]))
    need = [pks.lib.pks_workspace_bytes(nx, min(nx, 2), t, 1, pks._prec(precision)) for t in T]
    assert all(a <= b for a, b in zip(need, need[1:]))
    rng = np.random.default_rng(nx)
    model = wl.random_small_model(nx, 2, rng)
    ws = pks.workspace(nx, 2, 32769, 1, precision)
    dt = torch.float64 if precision == "fp64" else torch.float32
    pks.filter_smooth(pks.to_device(model), torch.zeros((32768, 2), dtype=dt, device="cuda"), precision, ws=ws)
    torch.cuda.synchronize()


@pytest.mark.parametrize("nx,ny", [(1, 1), (2, 1), (2, 2), (3, 2), (4, 2), (4, 4)])
def test_strongly_correlated_noise(pks, nx, ny):
    """I + C J far from symmetric: its leading entries can be small or negative,
    where the top level's elimination (pivots on the diagonal) has to notice."""
    for seed in range(6):
        rng = np.random.default_rng([nx, ny, seed])
        B, D = rng.standard_normal((nx, nx)), 10.0 ** rng.uniform(-1.5, 1.5, size=nx)
        F = rng.standard_normal((nx, nx))
        F *= 0.95 / np.abs(np.linalg.eigvals(F)).max()
        Q = B @ np.diag(D) @ B.T
        H, Rr = rng.standard_normal((ny, nx)), rng.standard_normal((ny, ny))
        model = wl.Model(F, 0.5 * (Q + Q.T) + 1e-3 * np.eye(nx), H, Rr @ Rr.T + 0.05 * np.eye(ny),
                         rng.standard_normal(nx), np.eye(nx))
        T = 20011
        y = 10.0 * rng.standard_normal((T, ny))
        out = pks.filter_smooth(pks.to_device(model), torch.as_tensor(y).cuda(), "fp64")
        torch.cuda.synchronize()
        ref = oracle.kf_rts(model.F, model.Q, model.H, model.R, model.m0, model.P0, y)
        for k, v in zip(("m", "P", "ms", "Ps"), out):
            e = wl.max_rel_err(v.cpu().numpy(), ref[k], "rms")
            assert e <= TOL["fp64"], (seed, k, e)
