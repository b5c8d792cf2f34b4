"""The root's variants at the time steps where the host changes from one to the
next (the polynomials' degrees, the polynomials with a Newton step, Newton
steps alone): the one-thread-per-node kernel's root within 1 ulp of the
oracle's root of the kernel's own xi, and the LDS-resident kernel (whose
variant is compiled in) equal to it bit for bit, 0 and +-1 kept exactly."""
import math
from fractions import Fraction

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 400


@pytest.fixture(scope="module")
def ace():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    from paper_2312_07010_amd import ace as A
    A.lib()
    return A


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def _xi(p, lo, hi, kappa, h):
    t = _fma(kappa, _fma(-2.0, p, lo + hi), p)
    return _fma(-h, _fma(p, p * p, -p), t)


@pytest.mark.parametrize("dt", [4.9e-4, 6e-4, 1.9e-3, 2.4e-3, 0.0099, 0.013, 0.02, 0.026, 0.049, 0.06, 0.29, 0.34,
                                0.44, 0.5])
def test_root_variant_edges(ace, orc, dt):
    eps = math.sqrt(0.01 / dt) / N
    s = ace.Solver(1, [N], [0.0], [1.0], eps, dt, "P")
    kappa, h = s.params["kappa"], s.params["h"]
    rng = np.random.default_rng(int(dt * 1e5))
    phi = np.concatenate([rng.uniform(-1, 1, N - 200), rng.uniform(-1e-3, 1e-3, 50),
                          np.full(10, 0.0), np.full(10, 1.0), np.full(10, -1.0),
                          1 - 1e-3 * rng.uniform(0, 1, 60), 1e-200 * rng.uniform(-1, 1, 60)])
    s.set_kernel(ace.ACE_KERNEL_DIRECT)
    s.set_phi0(phi)
    s.step(1)
    got = s.get_phi()
    for i in range(N):
        xi = _xi(float(phi[i]), float(phi[i - 1]), float(phi[(i + 1) % N]), kappa, h)
        r = float(orc.root(xi, h)[0])
        assert abs(float(got[i]) - r) <= np.spacing(abs(r)), (dt, i, xi, float(got[i]), r)
    for v, at in ((0.0, 255), (1.0, 265), (-1.0, 275)):
        assert got[at] == v  # equal neighbours: the step keeps 0 and +-1
    s.set_kernel(ace.ACE_KERNEL_RESIDENT)
    s.set_phi0(phi)
    s.step(1)
    assert np.array_equal(s.get_phi(), got)
    s.close()
