"""The 1D register-segment kernels against the one-step kernel (bit for bit) and
the oracle, at sizes around one, two and several segments of every nodes-per-
lane and on grids smaller than a segment's ring, with monitors, values beyond
1, NaN margins and every scheme."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [3, 5, 8, 31, 64, 65, 97, 128, 255, 257, 400, 513, 900, 1500, 2999, 5000, 8000, 8001, 30011, 70000, 250001]


@pytest.fixture(scope="module")
def ace():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2312_07010_amd import ace as A
    A.lib()
    return A


def _args(M, bc, dt):
    N = M + (-2, 1, 0)[bc]
    return 1, [N], [0.0], [1.0], math.sqrt(0.2 / dt) / N, dt, bc


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", SIZES)
def test_segments_equal_one_step_kernel(ace, orc, M, bc):
    import torch
    dt = (2e-3, 0.2, 0.6)[(M + bc) % 3]
    args = _args(M, bc, dt)
    p, r = orc.Problem(*args), ace.Solver(*args)
    r.set_kernel(ace.ACE_KERNEL_DIRECT)
    phi = np.random.default_rng(M + bc).uniform(-1.2, 1.2, r.shape)
    r.set_phi0(phi)
    Er, mr = r.run_monitored(75, 10)
    ref = r.get_phi()
    if M < 3000:
        want, _, _ = p.run(phi, 75)
        np.testing.assert_allclose(ref, want, rtol=0, atol=1e-12)
    for kernel in (ace.ACE_KERNEL_AUTO, ace.ACE_KERNEL_TBLOCK, ace.ACE_KERNEL_RESIDENT):
        s = ace.Solver(*args)
        guard = 512
        big = [torch.full((M + 2 * guard,), float("nan"), dtype=torch.float64, device="cuda") for _ in range(2)]
        s.bind_fields(big[0][guard:guard + M], big[1][guard:guard + M])
        s.set_kernel(kernel)
        s.set_phi0(phi)
        E, m = s.run_monitored(75, 10)
        assert np.array_equal(s.get_phi(), ref), kernel
        np.testing.assert_allclose(E, Er, rtol=1e-13)
        assert np.array_equal(m, mr)
        s.set_phi0(phi)
        for n in (1, 33, 41):
            s.step(n)
        assert np.array_equal(s.get_phi(), ref), kernel
        for t in big:
            assert bool(torch.isnan(t[:guard]).all()) and bool(torch.isnan(t[guard + M:]).all())
        s.close()
    r.close()


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [64, 700, 20011])
def test_segments_explicit_scheme_and_graphs(ace, M, bc):
    args = _args(M, bc, 1e-3)
    s, r = ace.Solver(*args), ace.Solver(*args)
    phi = np.random.default_rng(M).uniform(-1, 1, s.shape)
    for x in (s, r):
        x.set_scheme(ace.ACE_SCHEME_FEX)
        x.set_phi0(phi)
    r.set_kernel(ace.ACE_KERNEL_DIRECT)
    s.set_graph_launches(2)
    for n in (500, 501):
        s.step(n)
        r.step(n)
        assert np.array_equal(s.get_phi(), r.get_phi())
    s.close()
    r.close()
