"""A handle that steps inside a caller's capture and leaves the capturing stream
before the capture ends: the graph holds the steps, and its replays, with eager
work between them, equal eager runs."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")


def test_leave_the_stream_before_the_capture_ends():
    import torch
    from paper_2312_07010_amd import ace
    args = (2, [120, 90], [0, 0], [120.0, 90.0], 10.0, 1e-3, 0)
    s, r = ace.Solver(*args), ace.Solver(*args)
    phi0 = np.random.default_rng(5).uniform(-0.9, 0.9, s.shape)
    for x in (s, r):
        x.set_kernel(ace.ACE_KERNEL_DIRECT)
        x.set_phi0(phi0)
        x.step(2)  # (the kernel is loaded before the capture)
    torch.cuda.synchronize()
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=a, capture_error_mode="thread_local"):
        s.set_stream(a.cuda_stream)
        s.step(4)  # an even count: the field ends in the buffer it began in
        s.set_stream(b.cuda_stream)
    with torch.cuda.stream(b):
        for rep in range(3):
            g.replay()
            torch.cuda.synchronize()
            r.step(4)
            assert np.array_equal(s.get_phi(), r.get_phi()), rep
            s.step(2)  # eager, on the stream it moved to
            r.step(2)
            torch.cuda.synchronize()
    s.close()
    r.close()
