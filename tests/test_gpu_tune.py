"""pks_autotune times the general scan, which its configuration is for, and not the
paths that stand before it; short sequences of nx = 3, 4 are tuned over one and two
steps a thread as well."""
import json

import numpy as np
import pytest

import oracle
from paper_1905_13002_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pks():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13002_amd import pks as mod
    return mod


@pytest.mark.parametrize("nx,ny,B,T", [(4, 2, 1, 300000), (6, 3, 1, 10000), (16, 8, 4, 20000), (24, 24, 2, 9000)])
def test_the_general_scan_is_timed(pks, tmp_path, nx, ny, B, T):
    pks.profile_start()
    pks.autotune(nx, ny, B, T, "fp64", str(tmp_path / "tune.json"))
    names = set(pks.profile_stop())
    assert any("filter_reduce" in n for n in names), names
    assert not any(n.startswith(("k_st_", "k_stl_", "k_chain_")) for n in names), names


@pytest.mark.parametrize("nx", [3, 4])
def test_short_sequences(pks, tmp_path, monkeypatch, nx):
    """T = 1000, FP64: 82, 74 and 68 us with 4, 2 and 1 steps a thread at nx = 4."""
    T, cache = 1000, tmp_path / "tune.json"
    pks.autotune(nx, 2, 1, T, "fp64", str(cache))
    ept, ept1 = json.loads(cache.read_text())["nx%d_ny2_fp64_T9_B0" % nx][:2]
    assert ept in (1, 2)
    monkeypatch.setenv("PKS_TUNE_CACHE", str(cache))
    check(pks, nx, T)


@pytest.mark.parametrize("nx,T,config", [(4, 900, [1, 0]), (4, 100000, [2, 1]), (4, 40000, [1, 0]), (3, 120000, [2, 0]),
                                         (2, 900, [1, 0])])
def test_cached_configurations(pks, tmp_path, monkeypatch, nx, T, config):
    """Entries that fit are used; those with more threads than the workspace holds, or
    at nx = 2, are passed over."""
    cache = tmp_path / "tune.json"
    cache.write_text(json.dumps({"nx%d_ny2_fp64_T%d_B0" % (nx, T.bit_length() - 1): config}))
    monkeypatch.setenv("PKS_TUNE_CACHE", str(cache))
    check(pks, nx, T)


def check(pks, nx, T):
    rng = np.random.default_rng(T)
    model, y = wl.random_small_model(nx, 2, rng), rng.standard_normal((T, 2))
    out = pks.filter_smooth(pks.to_device(model), torch.as_tensor(y).cuda(), "fp64")
    torch.cuda.synchronize()
    ref = oracle.kf_rts(model.F, model.Q, model.H, model.R, model.m0, model.P0, y, u=model.u, d=model.d)
    for k, v in zip(("m", "P", "ms", "Ps"), out):
        assert wl.max_rel_err(v.cpu().numpy(), ref[k]) <= 1e-9, k
