"""The Polya-Gamma terms drawn through lists: both chunk lengths, trials around
the edges of a chunk and of a wavefront's run, and tilts on both sides of the
line between the two left methods (|c| = 3.125), against the CPU oracle.

FP64 within 1e-12 relative: the uniforms and the decisions are the oracle's,
and a site's psi is a sum of positive terms.
"""
import numpy as np
import pytest

from paper_1702_05518_amd import inputs

pytestmark = pytest.mark.gpu

RTOL64 = 1e-12


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


@pytest.mark.parametrize("tilt", [0.0, 1.5, 3.125, 6.0, 40.0])
@pytest.mark.parametrize("extra", [0, 1100])     # below and above 2^20 terms in total
def test_chunk_edges_and_tilts(orc, extra, tilt):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf as G

    n = 1000
    _, row_ptr, col = inputs.delaunay_graph(n, data_seed=3)
    color, k = G.greedy_coloring(row_ptr, col)
    edges = [0, 1, 2, 3, 4, 7, 8, 9, 15, 16, 17, 127, 128, 129, 511, 512, 513, 1]
    trials = np.array([edges[i % len(edges)] for i in range(n)], dtype=np.int32)
    trials[n // 2:] += extra * 2
    assert (int(trials.sum()) >= 1 << 20) == (extra > 0)
    rng = np.random.default_rng(7)
    y = rng.binomial(trials, 0.5).astype(np.float64)
    g = G.Graph(row_ptr=row_ptr, col_idx=col, color=color, num_colors=k, rho=0.95)
    kw = dict(seed=17, instance=2, intercept=True, beta0_var=100.0, trials=trials)
    ch = G.Chain(g, y, precision=G.FP64, **kw)
    oc = orc.Chain(row_ptr, col, color, y, rho=0.95, **kw)
    x0 = rng.choice([-1.0, 1.0], n) * tilt + 0.2 * rng.standard_normal(n)
    ch.set_state(x0, 1.5, 1.0, 4)
    oc.set_state(x0, 1.5, 1.0, 4, beta0=0.0)
    for _ in range(2):
        ch.sweep(1)
        oc.sweeps(1)
        x, tau, _, _ = ch.get_state()
        assert rel(x, oc.x) <= RTOL64
        assert rel(tau, oc.tau) <= RTOL64 and abs(ch.beta0 - oc.beta0) <= RTOL64
