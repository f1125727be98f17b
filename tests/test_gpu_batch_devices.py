"""A batch of lattices and graphs created and swept on streams of a device that
is not the current one: the graphs' second stream, which belongs to the
device that was current, is left out.  Bitwise the chains swept on their own.
Needs two devices.
"""
import numpy as np
import pytest

from paper_1702_05518_amd import inputs

pytestmark = pytest.mark.gpu


def chains(G, device, stream):
    y = inputs.image_observations(70, 65, 0.2, 1)[1]
    a = G.Chain(G.Graph(lattice=(70, 65, 8), device=device, stream=stream), y, seed=3,
                stream=stream)
    pts, rp, cl = inputs.delaunay_graph(900, data_seed=2)
    color, k = G.greedy_coloring(rp, cl)
    g = G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.95, device=device,
                stream=stream)
    return [a, G.Chain(g, inputs.smooth_field(pts), seed=3, stream=stream)]


@pytest.mark.parametrize("batch_current", [0, 1])
def test_streams_of_another_device(batch_current):
    import torch

    if torch.cuda.device_count() < 2:
        pytest.skip("one device")
    from paper_1702_05518_amd import gmrf as G

    with torch.cuda.device(1):
        stream = torch.cuda.Stream()
        alone, together = chains(G, "cuda:1", stream), chains(G, "cuda:1", stream)
        for c in alone:
            c.sweep(12, stream=stream)
    with torch.cuda.device(batch_current):
        batch = G.Batch(together, stream=stream)
    with torch.cuda.device(0):
        batch.sweep(12, stream=stream)
    with torch.cuda.device(1):
        stream.synchronize()
        for a, b in zip(alone, together):
            xa, xb = a.get_state(stream=stream), b.get_state(stream=stream)
            assert np.array_equal(xa[0], xb[0]) and xa[1:] == xb[1:]
