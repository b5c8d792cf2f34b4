"""The largest 1D field that one workgroup's segments hold (16 wavefronts of 240
output nodes) and the sizes around it, chosen LDS-resident, against the one-step
kernel bit for bit."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", [3839, 3840, 3841, 4064])
def test_edge(M, bc):
    from paper_2312_07010_amd import ace
    N = M + (-2, 1, 0)[bc]
    args = (1, [N], [0.0], [1.0], math.sqrt(0.2 / 2e-3) / N, 2e-3, bc)
    phi = np.random.default_rng(M).uniform(-1, 1, M)
    out = []
    for kernel in (ace.ACE_KERNEL_DIRECT, ace.ACE_KERNEL_RESIDENT):
        s = ace.Solver(*args)
        s.set_kernel(kernel)
        s.set_phi0(phi)
        E, mx = s.run_monitored(61, 20)
        out.append((s.get_phi(), E, mx))
        s.close()
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][2], out[1][2])
    np.testing.assert_allclose(out[0][1], out[1][1], rtol=1e-13)
