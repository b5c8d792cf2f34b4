"""The phase volume and the energy where the volume goes from one workgroup to many
(32768 nodes) and where its loop of eight loads per thread ends."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


@pytest.mark.parametrize("M", [(1024,), (8191,), (8193,), (32767,), (32768,), (32769,), (182, 180), (181, 181), (182, 181), (32, 32, 32),
                               (33, 32, 32)])
def test_edge(M):
    from paper_2312_07010_amd import ace
    d = len(M)
    s = ace.Solver(d, list(M), [0.0] * d, [float(m) for m in M], 5.0, 1e-3, 2)
    phi = np.random.default_rng(7).uniform(-1, 1, s.shape)
    s.set_phi0(phi)
    # (n terms in [0, 1], each rounded twice, then sums of at most n / 1024 + 20 additions in a chain)
    n = phi.size
    want = math.fsum((0.5 * (1 + phi)).ravel())
    for _ in range(2):
        assert abs(s.phase_volume() - want) <= (n / 1024 + 25) * 2.0 ** -53 * n
    s.close()
