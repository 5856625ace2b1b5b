"""pks_autotune times the general scan, which its configuration is for, and not the
paths that stand before it."""
import pytest

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
