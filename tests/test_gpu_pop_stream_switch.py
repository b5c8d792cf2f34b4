"""A population handle alternating between two streams, with enough work queued on
the one it leaves that it is still running, equals the same run on one stream."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


@pytest.mark.parametrize("kernel", ["AUTO", "SPLIT"])
def test_switch(kernel):
    import torch
    from paper_2312_07010_amd import ace
    args = (3, [180, 170, 190], [0.0] * 3, [180.0, 170.0, 190.0], 7.0, 1e-3, 2)
    ref, sw = ace.Pop(*args), ace.Pop(*args)
    phi0 = torch.empty(args[1], dtype=torch.float64, device="cuda").uniform_(-0.9, 0.9)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for p in (ref, sw):
        p.set_kernel(getattr(ace, "ACE_POP_" + kernel))
        p.set_phi0(phi0)
    for rep in range(6):
        with torch.cuda.stream(streams[rep % 2]):
            sw.use_torch_stream()
            sw.step(30)
        ref.step(30)
    torch.cuda.synchronize()
    assert np.array_equal(sw.get_phi(), ref.get_phi())
    ref.close()
    sw.close()
