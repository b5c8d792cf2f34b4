"""Checkpointed runs whose segments hold many launches: gradients with graph replay
between the launches that read and write checkpoints equal those without."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


@pytest.mark.parametrize("M,bc", [((9000,), 0), ((130, 90), 2), ((24, 31, 20), 1)])
@pytest.mark.parametrize("steps,every", [(400, 100), (385, 97), (64, 64)])
def test_gradients_equal(M, bc, steps, every):
    from paper_2312_07010_amd import ace
    d = len(M)
    N = [m + (-2, 1, 0)[bc] for m in M]
    s = ace.Solver(d, N, [0.0] * d, [float(n) for n in N], 10.0, 1e-3, bc)
    rng = np.random.default_rng(steps)
    phi, lam = rng.uniform(-0.9, 0.9, s.shape), rng.uniform(-1, 1, s.shape)
    got = []
    for graphs in (0, 2, 8):
        s.set_graph_launches(graphs)
        for rep in range(3):  # (replays after the first, with the sweep's eager work between)
            s.forward_ckpt(phi, steps, every)
            assert s.step_count == steps
            end = s.get_phi()
            got.append((end, *s.backward(lam)))
    for end, dphi, deps2 in got[1:]:
        assert np.array_equal(end, got[0][0]) and np.array_equal(dphi, got[0][1]) and deps2 == got[0][2]
    s.close()
