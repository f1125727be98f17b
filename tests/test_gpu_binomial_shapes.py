"""Launch shapes of a binomial chain: what a chain reports is what it runs,
setting that again changes nothing, every shape that fits can be set and set
back, and the chunked shape is refused where its tables or terms are missing.
Exact between chains of one shape; shapes agree to rounding (1e-12 relative
after two FP64 sweeps).
"""
import numpy as np
import pytest

from paper_1702_05518_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf

    gmrf.lib()
    return gmrf


def chain(G, rp, cl, f64=True, trials=None):
    n = len(rp) - 1
    color, k = G.greedy_coloring(rp, cl)
    g = G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.95)
    rng = np.random.default_rng(n)
    if trials is None:
        trials = rng.integers(0, 30, n).astype(np.int32)
    y = rng.binomial(trials, 0.4).astype(np.float64)
    return G.Chain(g, y, precision=G.FP64 if f64 else G.FP32_ACC64, seed=5, intercept=True,
                   beta0_var=50.0, trials=trials)


def result(ch):
    return ch.get_state()[0], ch.beta0, *ch.last_reductions()


def same(a, b):
    ra, rb = result(a), result(b)
    return np.array_equal(ra[0], rb[0]) and ra[1:] == rb[1:]


@pytest.mark.parametrize("f64", [True, False])
@pytest.mark.parametrize("n", [300, 2500])
def test_set_again_and_set_back(G, n, f64):
    _, rp, cl = inputs.delaunay_graph(n, data_seed=6)
    a, b, c = (chain(G, rp, cl, f64) for _ in range(3))
    assert a.tile == (1, 0, 0, 256)
    a.set_tile(a.tile[0])                       # what it runs
    a.sweep(3)
    b.sweep(3)
    assert same(a, b)
    for shape, threads in ((0, 256), (2, 512), (1, 256)):
        b.set_tile(shape)
        assert b.tile == (shape, 0, 0, threads)
        x = a.get_state()[0]
        for ch in (a, b, c):                    # the field stays where it is
            ch.set_state(x, 2.0, 1.0, 7 + shape)
            ch.set_intercept(0.1)
        c.set_tile(shape)                       # and when the shape changes
        for ch in (a, b, c):
            ch.sweep(1)
            ch.sweep(1, capture=True)
        assert same(b, c)
        if f64:
            assert np.max(np.abs(a.get_state()[0] - b.get_state()[0])) <= \
                1e-12 * np.max(np.abs(a.get_state()[0]))
    assert same(a, b)                           # shape 1 again


def test_refused(G):
    _, rp, cl = inputs.delaunay_graph(300, data_seed=6)
    no_trials = chain(G, rp, cl, trials=np.zeros(300, dtype=np.int32))
    i, j = np.triu_indices(33, 1)
    many_colors = chain(G, *inputs.edges_to_csr(33, i, j))
    for ch in (no_trials, many_colors):
        shape = ch.tile[0]
        assert shape != 1
        with pytest.raises(G.GmrfError):
            ch.set_tile(1)
        assert ch.tile[0] == shape
        ch.sweep(1)
        assert np.isfinite(ch.get_state()[0]).all()
