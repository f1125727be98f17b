"""Batches of lattices and graphs, whose graphs run on a second stream within a
call: call lengths around the line from which they do and around the groups
of unit variates (128 sweeps), plain and captured, on a stream of the
caller's, with work queued right behind the call.  Bitwise the chains swept
on their own.
"""
import numpy as np
import pytest

from paper_1702_05518_amd import inputs

pytestmark = pytest.mark.gpu


def chains(G, seed):
    out = []
    for i, (rows, cols, st) in enumerate([(40, 70, 4), (65, 64, 8), (130, 33, 4)]):
        y = inputs.image_observations(rows, cols, 0.2, seed + i)[1]
        out.append(G.Chain(G.Graph(lattice=(rows, cols, st)), y, precision=G.FP64, seed=seed,
                           instance=i, intercept=i == 1))
    for i, (n, shape) in enumerate([(700, 1), (1500, 0), (2500, 1)]):
        pts, rp, cl = inputs.delaunay_graph(n, data_seed=seed)
        color, k = G.greedy_coloring(rp, cl)
        y = inputs.smooth_field(pts) + 0.1 * np.random.default_rng(i).standard_normal(n)
        ch = G.Chain(G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.95), y,
                     precision=G.FP64, seed=seed, instance=10 + i)
        ch.set_tile(shape)
        out.append(ch)
    return out


@pytest.mark.parametrize("capture", [False, True])
@pytest.mark.parametrize("sweeps", [5, 6, 128, 129, 257])
def test_mixed_batch(sweeps, capture):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf as G

    alone, together = chains(G, 3), chains(G, 3)
    for c in alone + together:      # lattice shapes that a batch also takes
        if c.tile[0] == 2:
            c.set_tile(0)
    batch = G.Batch(together)
    n = sum(c.n for c in together)
    mean = torch.empty(n, dtype=torch.float64, device="cuda")
    var = torch.empty_like(mean)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    for c in alone:
        c.sweep(sweeps)
        c.sweep(sweeps)
    for _ in range(2):
        batch.sweep(sweeps, capture=capture, stream=stream)
        at = 0
        for c in together:          # queued behind the call, before any synchronisation
            c.posterior_stats_device(mean[at:at + c.n], var[at:at + c.n], stream=stream)
            at += c.n
    torch.cuda.synchronize()
    at = 0
    for a, b in zip(alone, together):
        xa, ta, la, na = a.get_state()
        xb, tb, lb, nb = b.get_state()
        assert np.array_equal(xa, xb) and (ta, la, na) == (tb, lb, nb)
        ma, va, _ = a.posterior_stats()
        assert np.array_equal(ma, mean[at:at + a.n].cpu().numpy())
        assert np.array_equal(va, var[at:at + a.n].cpu().numpy())
        at += a.n
