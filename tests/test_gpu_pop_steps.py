"""The carried population form over several steps in one call (whose inner steps
write phi alone) against one-step calls of the fused form, which writes and
reads every population at every step: populations and phi bit for bit, on the
column kernel's fields (around its planes per thread) and past 20 million nodes
on the tiled march; and phi right after the populations are set."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SMALL = [(3, 3), (5, 70), (47, 65), (700, 301), (3, 3, 3), (5, 4, 7), (9, 40, 33), (34, 29, 33), (130, 17, 70)]


def _pair(M, bc, dt):
    import torch
    from paper_2312_07010_amd import ace
    d = len(M)
    N = [m + (-2, 1, 0)[bc] for m in M]
    dx = 1.0 / N[-1]
    args = (d, N, [0.0] * d, [n * dx for n in N], math.sqrt(0.05 / dt) * dx, dt, bc)
    a, b = ace.Pop(*args), ace.Pop(*args)
    b.set_kernel(ace.ACE_POP_FUSED)
    gen = torch.Generator(device="cuda").manual_seed(1)
    phi = torch.rand(M, dtype=torch.float64, device="cuda", generator=gen) * 2.2 - 1.1
    return torch, a, b, phi


def _check(torch, a, b, phi, counts):
    a.set_phi0(phi)
    b.set_phi0(phi)
    out = torch.empty_like(phi)
    f = torch.empty((a.q,) + a.shape, dtype=torch.float64, device="cuda")
    g = torch.empty_like(f)
    p = torch.empty_like(phi)
    assert torch.equal(a.get_phi(out), b.get_phi(p))
    for n in counts:
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert torch.equal(a.get_populations(f), b.get_populations(g)), n
        assert torch.equal(a.get_phi(out), b.get_phi(p)), n
    a.set_populations(g)
    assert torch.equal(a.get_phi(out), p)
    a.step(2)
    b.step(2)
    assert torch.equal(a.get_populations(f), b.get_populations(g))
    a.close()
    b.close()


@pytest.mark.parametrize("bc", [0, 1, 2])
@pytest.mark.parametrize("M", SMALL)
def test_carried_steps(M, bc):
    _check(*_pair(M, bc, (5e-4, 0.02, 0.2)[(bc + len(M)) % 3]), (1, 2, 5))


@pytest.mark.parametrize("M,bc", [((301, 260, 270), 2), ((290, 270, 261), 1), ((4700, 4600), 0)])
def test_carried_steps_past_the_caches(M, bc):
    _check(*_pair(M, bc, 5e-4), (3,))
