"""gmrf_set_state without a field (x NULL: keep the current one) at sweep
indices of the same and the other parity, for every shape whose field
alternates between the two state buffers and for those whose field stays in
one.  Exact: the field kept is the one that was there, and the sweeps that
follow are those of a chain that is given the same field.
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


def graph(G, kind):
    if kind == "lattice":
        return G.Graph(lattice=(70, 65, 8))
    _, rp, cl = inputs.delaunay_graph(1500, data_seed=3)
    color, k = G.greedy_coloring(rp, cl)
    return G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.95)


@pytest.mark.parametrize("f64", [True, False])
@pytest.mark.parametrize("kind,shape", [("lattice", 0), ("lattice", 1), ("graph", 0),
                                        ("graph", 1), ("graph", 2)])
def test_field_is_kept(G, kind, shape, f64):
    prec = G.FP64 if f64 else G.FP32_ACC64
    g = graph(G, kind)
    rng = np.random.default_rng(g.n)
    y = rng.standard_normal(g.n)
    x0 = rng.standard_normal(g.n).astype(np.float32).astype(np.float64)
    a = G.Chain(g, y, precision=prec, seed=2, x0=x0)      # a new chain, and one mid-run
    b = G.Chain(g, y, precision=prec, seed=2)
    a.set_tile(shape)
    b.set_tile(shape)
    for start in (3, 8, 10, 11):
        x = a.get_state()[0]
        a.set_state(None, 1.5, 2.0, start)
        got = a.get_state()
        assert np.array_equal(got[0], x) and got[1:] == (1.5, 2.0, start)
        b.set_state(x, 1.5, 2.0, start)
        a.sweep(2)
        b.sweep(2)
        assert np.array_equal(a.get_state()[0], b.get_state()[0])
