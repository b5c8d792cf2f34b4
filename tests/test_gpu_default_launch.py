"""The launch shapes a handle takes without tuning, on fields of the sizes where
the rule changes: bit for bit the oracle-checked kernels' results over runs of
every length up to 13 (so that every rest of a run shorter than the depth
occurs), and the column kernel on plane counts around its planes per thread."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ace():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2312_07010_amd import ace as A
    A.lib()
    return A


def _args(M, bc, dt, kappa=0.1):
    d = len(M)
    N = [m + (-2, 1, 0)[bc] for m in M]
    dx = 1.0 / N[-1]
    return d, N, [0.0] * d, [n * dx for n in N], math.sqrt(kappa / dt) * dx, dt, bc


@pytest.mark.parametrize("fex", [0, 1])
@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [(45, 45), (45, 46), (300, 301), (60, 2000), (40, 41, 43), (110, 100, 90), (20, 330, 300),
                               (200, 60, 70)])
def test_default_launch(ace, orc, M, bc, fex):
    args = _args(M, bc, 2e-3)
    s, r, p = ace.Solver(*args), ace.Solver(*args), orc.Problem(*args)
    r.set_kernel(ace.ACE_KERNEL_MARCH if len(M) == 3 else ace.ACE_KERNEL_DIRECT)
    if fex:
        s.set_scheme(ace.ACE_SCHEME_FEX)
        r.set_scheme(ace.ACE_SCHEME_FEX)
    phi = np.random.default_rng(len(M) * 100 + bc).uniform(-1, 1, s.shape)
    s.set_phi0(phi)
    r.set_phi0(phi)
    for n in (1, 2, 3, 5, 7, 11, 13):
        s.step(n)
        r.step(n)
        assert np.array_equal(s.get_phi(), r.get_phi()), (n, s.get_kernel())
    Es, ms = s.run_monitored(7, 3)
    Er, mr = r.run_monitored(7, 3)
    np.testing.assert_allclose(Es, Er, rtol=1e-13)
    assert np.array_equal(ms, mr)
    assert np.array_equal(s.get_phi(), r.get_phi())
    if not fex:
        s.set_phi0(phi)
        s.step(2)
        np.testing.assert_allclose(s.get_phi(), p.run(phi, 2)[0], rtol=0, atol=1e-14)
    s.close()
    r.close()


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [(3, 3, 3), (4, 5, 7), (5, 17, 15), (7, 16, 16), (8, 64, 65), (9, 400, 330), (33, 129, 130)])
def test_column_kernel(ace, M, bc):
    args = _args(M, bc, 0.01)
    s, r = ace.Solver(*args), ace.Solver(*args)
    s.set_kernel(ace.ACE_KERNEL_DIRECT)
    r.set_kernel(ace.ACE_KERNEL_MARCH)
    phi = np.random.default_rng(bc).uniform(-1.3, 1.3, s.shape)  # (some roots beyond 1)
    s.set_phi0(phi)
    r.set_phi0(phi)
    Es, ms = s.run_monitored(4, 1)
    Er, mr = r.run_monitored(4, 1)
    assert np.array_equal(s.get_phi(), r.get_phi())
    np.testing.assert_allclose(Es, Er, rtol=1e-13)
    assert np.array_equal(ms, mr)
    s.close()
    r.close()


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [(6, 5, 7), (30, 47, 61), (21, 81, 113)])
def test_deep_region(ace, M, bc, tmp_path, monkeypatch):
    """The four-step kernel on 48-row regions, which only the library's own
    choice takes (here through a tuning record)."""
    cache = tmp_path / "tune"
    cache.write_text('{"d": 3, "bc": %d, "M": [%d, %d, %d], "kernel": 4, "zchunk": 8, "depth2": 5, "tb3": 6, '
                     '"tb2": -1, "ms_per_step": 0.01}\n' % (bc, *M))
    args = _args(M, bc, 5e-4)
    r = ace.Solver(*args)
    monkeypatch.setenv("ACE_AUTOTUNE_CACHE", str(cache))
    s = ace.Solver(*args)
    assert s.get_region3d() == (4, 48, 3)
    with pytest.raises(ace.AceError):
        r.set_region3d(4, 48, 3)
    r.set_kernel(ace.ACE_KERNEL_DIRECT)
    phi = np.random.default_rng(bc + 7).uniform(-1.2, 1.2, s.shape)
    s.set_phi0(phi)
    r.set_phi0(phi)
    Es, ms = s.run_monitored(11, 4)
    Er, mr = r.run_monitored(11, 4)
    assert np.array_equal(s.get_phi(), r.get_phi())
    np.testing.assert_allclose(Es, Er, rtol=1e-13)
    assert np.array_equal(ms, mr)
    s.close()
    r.close()
