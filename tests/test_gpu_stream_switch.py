"""Switching a handle between streams waits for the old one also where no graph
was captured: short direct launches alternating between two streams equal the
same run on one stream."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", [0, 32])
def test_switch_without_graphs(graphs):
    import torch
    from paper_2312_07010_amd import ace
    args = (2, [700, 700], [0, 0], [1, 1], 0.002, 1e-3, 0)
    ref, sw = ace.Solver(*args), ace.Solver(*args)
    phi0 = np.random.default_rng(5).uniform(-0.9, 0.9, ref.shape)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for s in (ref, sw):
        s.set_graph_launches(graphs)
        s.set_phi0(phi0)
    for rep in range(6):
        with torch.cuda.stream(streams[rep % 2]):
            sw.use_torch_stream()
            sw.step(40)
        ref.step(40)
    torch.cuda.synchronize()
    assert np.array_equal(sw.get_phi(), ref.get_phi())
    ref.close()
    sw.close()


def test_batch_switch_without_graphs():
    import torch
    from paper_2312_07010_amd import ace
    insts = [(1, [300], [0.0], [1.0], 0.02, 1e-3, "P"), (2, [300, 300], [0.0, 0.0], [1.0, 1.0], 0.005, 1e-3, "HN")]
    b1, b2 = ace.Batch(insts), ace.Batch(insts)
    fields = [np.random.default_rng(7 + i).uniform(-0.9, 0.9, shp) for i, shp in enumerate(b1.shapes)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for b in (b1, b2):
        b.set_graphs(False)
        b.set_all(fields)
    for rep in range(4):
        with torch.cuda.stream(streams[rep % 2]):
            b2.use_torch_stream()
            b2.step(30)
        b1.step(30)
    torch.cuda.synchronize()
    for i in range(len(insts)):
        assert np.array_equal(b1.get_phi(i), b2.get_phi(i))
    b1.close()
    b2.close()
