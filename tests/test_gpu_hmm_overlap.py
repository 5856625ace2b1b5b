"""Discrete-state filter and smoother by overlapped blocks (csrc/hmm.hip): the
path taken (the flags in the last 256 bytes of the workspace: filter, smoother),
every step against the sequential oracle at the absolute bar of the parity
tests, for every padded state count, around the shortest lengths that take the
path and with ragged last blocks; chains that do not forget, and steps without
weight, go to the block-element scan."""
import numpy as np
import pytest

import oracle
from paper_1905_13002_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
TOL = 1e-9


@pytest.fixture(scope="module")
def pks():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1905_13002_amd import pks as mod
    return mod


def flags(ws):
    return [int(v) for v in ws[-256:].cpu().numpy().view(np.int32)[:2]]


def errors(ref, alpha, logp, gamma):
    cum, mag = np.cumsum(ref["ll"]), np.cumsum(np.abs(ref["ll"]))
    e = [np.max(np.abs(alpha.cpu().numpy() - ref["alpha"])),
         np.max(np.abs(logp.cpu().numpy() - cum) / np.maximum(1.0, mag))]
    return e if gamma is None else e + [np.max(np.abs(gamma.cpu().numpy() - ref["gamma"]))]


@pytest.mark.parametrize("K,T,sparse", [(64, 4096, False), (64, 4099, True), (49, 33001, False), (48, 8192, False),
                                        (33, 8193, False), (32, 32773, False), (17, 40002, False),
                                        (16, 65536, False), (3, 65569, False)])
def test_overlapped_blocks(pks, K, T, sparse):
    w = wl.hmm_workload(K=K, T=T, seed=31, sparse=sparse)
    dm, L = pks.hmm_to_device(w.Pi, w.p0), torch.as_tensor(w.L).cuda()
    ref = oracle.hmm_fb(w.Pi, w.p0, w.L)
    ws = pks.hmm_workspace(K, T)
    out = pks.hmm_filter_smooth(dm, L, ws=ws)
    torch.cuda.synchronize()
    assert flags(ws) == [1, 1]
    assert max(errors(ref, *out)) <= TOL
    # apart: bitwise what the combined call gives
    alpha, logp, _ = pks.hmm_filter_smooth(dm, L, smooth=False)
    gamma = pks.hmm_smooth(dm, alpha)
    for a, b in zip((alpha, logp, gamma), out):
        assert torch.equal(a, b)


@pytest.mark.parametrize("K,T", [(64, 4100), (20, 32768)])
def test_chains_that_do_not_forget(pks, K, T):
    """A cyclic permutation, nearly uninformative data, any start."""
    rng = np.random.default_rng(K)
    Pi, p0, L = np.roll(np.eye(K), 1, axis=1), rng.dirichlet(np.ones(K)), 1e-3 * rng.normal(size=(T, K))
    ws = pks.hmm_workspace(K, T)
    out = pks.hmm_filter_smooth(pks.hmm_to_device(Pi, p0), torch.as_tensor(L).cuda(), ws=ws)
    torch.cuda.synchronize()
    assert flags(ws) == [0, 0]
    assert max(errors(oracle.hmm_fb(Pi, p0, L), *out)) <= TOL


@pytest.mark.parametrize("at", [0, 100, 4094])
def test_steps_without_weight(pks, at):
    """A step that no state explains: up to it the filter is the oracle's."""
    w = wl.hmm_workload(K=64, T=4096, seed=5)
    L = w.L.copy()
    L[at] = -np.inf
    ws = pks.hmm_workspace(64, 4096)
    alpha, logp, _ = pks.hmm_filter_smooth(pks.hmm_to_device(w.Pi, w.p0), torch.as_tensor(L).cuda(), ws=ws)
    torch.cuda.synchronize()
    assert flags(ws) == [0, 0]
    if at:
        ref = oracle.hmm_fb(w.Pi, w.p0, w.L[:at])
        assert np.max(np.abs(alpha.cpu().numpy()[:at] - ref["alpha"])) <= TOL
