"""The reverse sweep on 2D register regions (one launch holding the transposed
steps of a segment and the recompute of the one before) and by 3D columns: at
sizes around a region's tiles and a column's planes, segments shorter and
longer than a launch and not dividing the steps, against the oracle; in 2D
also against the one-node-per-thread sweep, dL/dphi0 bit for bit."""
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


def _args(M, bc, dt):
    d = len(M)
    N = [m + (-2, 1, 0)[bc] for m in M]
    dx = 1.0 / N[-1]
    return d, N, [0.0] * d, [n * dx for n in N], math.sqrt(0.15 / d / dt) * dx, dt, bc


def _run(ace, orc, M, bc, steps, ckpt, dt, bitwise):
    args = _args(M, bc, dt)
    s, p = ace.Solver(*args), orc.Problem(*args)
    rng = np.random.default_rng(sum(M) + bc)
    phi0 = rng.uniform(-0.6, 0.6, p.shape)
    lam = rng.uniform(-0.5, 0.5, p.shape)
    g_or, _, ge_or = p.adjoint(phi0, steps, lam)
    scale = np.abs(g_or).max()
    kernels = [ace.ACE_KERNEL_TBLOCK, ace.ACE_KERNEL_DIRECT] if bitwise else [ace.ACE_KERNEL_AUTO]
    grads = []
    for k in kernels:
        s.set_kernel(k)
        g, ge = s.adjoint(phi0, steps, ckpt, lam)
        np.testing.assert_allclose(g, g_or, rtol=0, atol=1e-12 * scale)
        assert ge == pytest.approx(ge_or, rel=1e-10, abs=1e-13)
        np.testing.assert_allclose(s.get_phi(), p.run(phi0, steps)[0], rtol=0, atol=1e-13)
        grads.append(g)
    assert all(np.array_equal(g, grads[0]) for g in grads)
    s.close()


@pytest.mark.parametrize("steps,ckpt", [(1, 1), (2, 5), (23, 1), (23, 3), (24, 8), (29, 13), (45, 40)])
@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [(47, 46), (100, 65), (9, 301), (150, 17)])
def test_regions(ace, orc, M, bc, steps, ckpt):
    _run(ace, orc, M, bc, steps, ckpt, (2e-3, 0.02, 0.2)[(bc + ckpt) % 3], True)


@pytest.mark.parametrize("bc", [0, 1, 2])
def test_regions_of_64_rows(ace, orc, bc):
    _run(ace, orc, (330, 517), bc, 21, 10, 1e-3, True)


@pytest.mark.parametrize("steps,ckpt", [(1, 1), (11, 4), (12, 30)])
@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [(3, 3, 3), (5, 33, 17), (9, 64, 65), (34, 70, 90)])
def test_columns(ace, orc, M, bc, steps, ckpt):
    _run(ace, orc, M, bc, steps, ckpt, (5e-4, 0.02, 0.2)[(bc + ckpt) % 3], False)
