"""dL/d(eps^2) of a uniform field: Lambda phi is 0 at every state, so with no
walls (or reflecting ones) the gradient is 0, not a rounding residue, on every
way of sweeping."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


@pytest.mark.parametrize("bc", [0, 2])
@pytest.mark.parametrize("M,sweep", [((700,), None), ((60, 70), None), ((60, 70), (64, 4)), ((60, 70), (32, 2)),
                                     ((60, 70), (0, 0)), ((130, 190), None), ((40, 37, 50), None)])
def test_uniform_field_has_no_gradient(M, sweep, bc):
    from paper_2312_07010_amd import ace
    dt, d = 1e-3, len(M)
    s = ace.Solver(d, [m + (-2, 1, 0)[bc] for m in M], [0.0] * d, [float(m + (-2, 1, 0)[bc]) for m in M],
                   math.sqrt(0.1 / dt), dt, bc)
    if sweep is not None:
        s.set_kernel(ace.ACE_KERNEL_TBLOCK, 3)
        s.set_region2d(*sweep)
    lam = np.random.default_rng(1).uniform(-1, 1, s.shape)
    for p in (0.25, -0.75):  # (sums of six of these are exact, so each state stays uniform with Lambda phi = 0)
        s.forward_ckpt(np.full(s.shape, p), 21, 5)
        dphi, deps2 = s.backward(lam)
        assert deps2 == 0.0
        assert np.isfinite(dphi).all() and dphi.any()
    s.close()
