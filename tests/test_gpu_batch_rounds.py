"""The batch's rounds: step counts that make an odd number of one-step rounds,
uneven rounds and more than one graph, on 1D and 2D instances around the sizes
of a segment (192 outputs) and a region, bit for bit single-instance runs; and
the whole-batch copies on the device and the host, and the chunked monitor."""
import ctypes
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _insts():
    out = []
    rng = np.random.default_rng(3)
    for d, sizes in ((1, (3, 64, 191, 193, 385, 8001, 20000)), (2, (3, 7, 47, 49, 65, 130))):
        for N in sizes:
            for bc in (0, 1, 2):
                dt = float(rng.choice([5e-4, 0.01, 0.2, 0.6]))
                eps = math.sqrt(0.3 * (1 - dt) / (2 * d) / dt) / N
                out.append((d, [N] * d, [0.0] * d, [1.0] * d, eps, dt, bc))
    return out


@pytest.mark.parametrize("graphs", [True, False])
def test_rounds_equal_single_runs(graphs):
    from paper_2312_07010_amd import ace
    insts = _insts()
    b = ace.Batch(insts)
    b.set_graphs(graphs)
    rng = np.random.default_rng(4)
    phi0 = [rng.uniform(-1.1, 1.1, shp) for shp in b.shapes]
    steps = (1, 2, 5, 33, 2100)
    b.set_all(phi0)
    got = []
    for n in steps:
        b.step(n)
        got.append(b.get_all())
    b.set_depth(1)
    b.set_all(phi0)
    b.step(3)
    odd = b.get_all()
    E, mx = b.monitor()
    for i, inst in enumerate(insts):
        s = ace.Solver(*inst)
        s.set_phi0(phi0[i])
        for n, g in zip(steps, got):
            s.step(n)
            assert np.array_equal(s.get_phi(), g[i]), (n, inst)
        s.set_phi0(phi0[i])
        s.step(3)
        assert np.array_equal(s.get_phi(), odd[i]), inst
        assert E[i] == pytest.approx(s.energy(), rel=1e-13)
        assert mx[i] == s.maxnorm()
        s.close()
    b.close()


def test_whole_batch_copies():
    import torch
    from paper_2312_07010_amd import ace
    b = ace.Batch(_insts())
    n = sum(b.totals)
    f = torch.rand(n, dtype=torch.float64, device="cuda") - 0.5
    out = torch.empty_like(f)
    assert ace.lib().ace_batch_set_all(b._h, ctypes.c_void_p(f.data_ptr()), ace.ACE_DEVICE) == 0
    assert ace.lib().ace_batch_get_all(b._h, ctypes.c_void_p(out.data_ptr()), ace.ACE_DEVICE) == 0
    torch.cuda.synchronize()
    assert torch.equal(out, f)
    host = np.concatenate([x.ravel() for x in b.get_all()])
    assert np.array_equal(host, f.cpu().numpy())
    for i in (0, 5, len(b.totals) - 1):
        assert np.array_equal(b.get_phi(i).ravel(), host[sum(b.totals[:i]):sum(b.totals[:i + 1])])
    bad = [np.zeros(s) for s in b.shapes]
    bad[3].flat[0] = np.inf
    with pytest.raises(ace.AceError) as e:
        b.set_all(bad)
    assert e.value.code == ace.ACE_E_NONFINITE
    assert np.array_equal(b.get_phi(0).ravel(), host[:b.totals[0]])  # nothing changed
    b.close()
