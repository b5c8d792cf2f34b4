"""Fields with an axis of one node whose regions are more workgroups than one
launch holds: the default run and a batch, against the oracle on windows at the
ends, in the middle and around the first workgroup past a launch."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

DT, KAPPA = 0.01, 0.1
EPS = (KAPPA / DT) ** 0.5  # dx = 1


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


def _check(orc, start, field, n, steps, at):
    W, keep = 400, 200
    for a in at:
        a = max(0, min(a, n - W))
        x0 = start[a:a + W].cpu().numpy()
        want, _, _ = orc.Problem(2, [W + 1, 2], [0.0, 0.0], [W + 1.0, 2.0], EPS, DT, "HD").run(x0.reshape(W, 1), steps)
        lo, hi = (0 if a == 0 else (W - keep) // 2), (W if a == n - W else (W + keep) // 2)
        np.testing.assert_allclose(field[a + lo:a + hi].cpu().numpy(), want.ravel()[lo:hi], rtol=0, atol=1e-14)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("M", [(60_000_000, 1), (1, 200_000_000)])
def test_default_run(orc, M):
    import torch
    from paper_2312_07010_amd import ace
    n = max(M)
    s = ace.Solver(2, [m + 1 for m in M], [0.0, 0.0], [m + 1.0 for m in M], EPS, DT, "HD")
    start = torch.empty(n, dtype=torch.float64, device="cuda").uniform_(-0.9, 0.9)
    field = start.clone()
    s.set_phi0(field.view(M))
    s.step(23)
    s.get_phi(field.view(M))
    _check(orc, start, field, n, 23, (0, n // 2, n))
    s.close()


@pytest.mark.timeout(600)
def test_batch(orc):
    import torch
    from paper_2312_07010_amd import ace
    n, steps = 260_000_000, 16
    b = ace.Batch([(2, [n + 1, 2], [0.0, 0.0], [n + 1.0, 2.0], EPS, DT, "HD")])
    start = torch.empty(n, dtype=torch.float64, device="cuda").uniform_(-0.9, 0.9)
    field = start.clone()
    L = ace.lib()
    assert L.ace_batch_set_all(b._h, ctypes.c_void_p(field.data_ptr()), ace.ACE_DEVICE) == 0
    b.set_depth(8)  # 48 rows of output per region
    b.step(steps)
    assert L.ace_batch_get_all(b._h, ctypes.c_void_p(field.data_ptr()), ace.ACE_DEVICE) == 0
    torch.cuda.synchronize()
    first = (2 ** 32 - 1) // 1024 * 48
    assert first < n
    _check(orc, start, field, n, steps, (0, first - 200, n // 2, n))
    b.close()
