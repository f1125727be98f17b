"""The trials that a binomial chain takes in all: what fits with at most
2^31 - 257 chunks of four Polya-Gamma terms, whatever chunks the kernel
takes.  The footprint decides it from the counts alone, so no memory is used.
"""
import numpy as np
import pytest

from paper_1702_05518_amd import inputs

pytestmark = pytest.mark.gpu

LIMIT = 2 ** 31 - 1 - 256           # chunks of four


@pytest.fixture(scope="module")
def G():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf

    gmrf.lib()
    return gmrf


def footprint(G, trials):
    rp, cl = inputs.path_graph(len(trials))
    color, k = G.greedy_coloring(rp, cl)
    g = G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k)
    t = np.array(trials, dtype=np.int32)
    return G.lib().gmrf_binomial_footprint(g.handle, G.FP64, G._p(t, G.C.c_int32))


def spread(total, sites=5):
    """total trials over the sites, all but the last a multiple of four."""
    each = min(total // sites // 4 * 4, 2 ** 31 - 4)
    return [each] * (sites - 1) + [total - each * (sites - 1)]


# 2^20: chunks of two below, of eight from there on; 4.29e9: what chunks of
# two could hold; 4 LIMIT: the most
@pytest.mark.parametrize("total", [2 ** 20 - 1, 2 ** 20, 2 * LIMIT - 8, 2 * LIMIT + 8,
                                   3 * LIMIT, 4 * LIMIT])
def test_accepted(G, total):
    trials = spread(total)
    chunk = 2 if total < 2 ** 20 else 8
    nc = sum(-(-m // chunk) for m in trials)
    al = lambda b: (b + 255) // 256 * 256
    # a site index and a sum per chunk (one of each without trials)
    assert footprint(G, trials) - footprint(G, [0] * 5) == al(4 * nc) + al(8 * nc) - 2 * 256


@pytest.mark.parametrize("total", [4 * LIMIT + 1, 5 * LIMIT, 8 * LIMIT])
def test_refused(G, total):
    trials = spread(total, 9)
    assert footprint(G, trials) == 0
    assert "too many trials" in G.last_error()
