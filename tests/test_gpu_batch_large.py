"""Batched 1D instances at and past the size whose indices 32 bits hold (2^30
nodes, 8.6 GB each): windows at the ends, at the middle and around node 2^30
against the oracle on each window, whose own boundary cannot reach the nodes
compared in so few steps."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")

STEPS, W, KEEP = 5, 600, 300  # an odd count of one-step launches ends in the second arena


@pytest.mark.timeout(600)
@pytest.mark.parametrize("M,bc", [(2 ** 30 - 2, "HN"), (2 ** 30 + 2, "HN"), (2 ** 30, "HD"), (2 ** 31, "P")])
def test_1d_instance_past_32_bit_indices(orc, M, bc):
    import torch
    from paper_2312_07010_amd import ace
    N = M + {"HN": -2, "HD": 1, "P": 0}[bc]
    dt, kappa = 0.01, 0.2
    eps = (kappa / dt) ** 0.5  # dx = 1

    def problem(n, b):
        cells = n + {"HN": -2, "HD": 1, "P": 0}[b]
        return orc.Problem(1, [cells], [0.0], [float(cells)], eps, dt, b)

    small = (1, [300], [0.0], [300.0], eps, dt, "HN")
    b = ace.Batch([small, (1, [N], [0.0], [float(N)], eps, dt, bc), small])
    assert b.totals[1] == M
    lead = b.totals[0]
    torch.manual_seed(3)
    field = torch.empty(sum(b.totals), dtype=torch.float64, device="cuda").uniform_(-0.9, 0.9)
    start = field.clone()
    L = ace.lib()
    assert L.ace_batch_set_all(b._h, ctypes.c_void_p(field.data_ptr()), ace.ACE_DEVICE) == 0
    b.step(STEPS)
    assert L.ace_batch_get_all(b._h, ctypes.c_void_p(field.data_ptr()), ace.ACE_DEVICE) == 0
    torch.cuda.synchronize()

    def window(t, a, n):
        return t[lead + a:lead + a + n].cpu().numpy()

    def check(x0, b_, lo, hi, got):
        want, _, _ = problem(len(x0), b_).run(x0, STEPS)
        np.testing.assert_allclose(got, want[lo:hi], rtol=0, atol=1e-14)

    for a in (M // 2 - 111, min(2 ** 30, M - W) - W // 2):
        check(window(start, a, W), "HN", 150, 450, window(field, a + 150, 300))
    if bc == "P":
        ends = np.concatenate([window(start, M - W // 2, W // 2), window(start, 0, W // 2)])
        got = np.concatenate([window(field, M - 150, 150), window(field, 0, 150)])
        check(ends, "HN", 150, 450, got)
    else:
        check(window(start, 0, W), bc, 0, KEEP, window(field, 0, KEEP))
        check(window(start, M - W, W), bc, W - KEEP, W, window(field, M - KEEP, KEEP))
    for i, a in ((0, 0), (2, lead + M)):  # its neighbours in the arena
        x0 = start[a:a + lead].cpu().numpy()
        want, _, _ = orc.Problem(*small).run(x0, STEPS)
        np.testing.assert_allclose(field[a:a + lead].cpu().numpy(), want, rtol=0, atol=1e-14)
    b.close()
    del field, start
    torch.cuda.empty_cache()
