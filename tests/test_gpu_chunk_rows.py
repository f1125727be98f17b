"""The chunked sweep's row groups: sites of every degree around the edges of
a group of four neighbours and of the twelve read in one round (0 .. 17, 33,
300), on graphs with more sites of a color than a block has threads (trees:
two colors) and with fewer than one chunk.  FP64 field, accumulators and
precisions within 1e-12 relative of the oracle, FP32 within 1e-4 (the FP32
chains' criterion), over calls that end sweeps inside the next kernel."""
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


def rel(a, b):
    return float(np.max(np.abs(np.asarray(a) - np.asarray(b))) / np.max(np.abs(b)))


def stars(degrees, chain):
    """A star of each degree, its center joined to the next star's center if
    chain; ids shuffled so that neighbours of one site lie far apart."""
    ei, ej, centers, n = [], [], [], 0
    for d in degrees:
        centers.append(n)
        links = min(d, 2) if chain else 0
        leaves = d - links if chain else d
        ei += [n] * leaves
        ej += list(range(n + 1, n + 1 + leaves))
        n += 1 + leaves
    if chain:
        ei += centers[:-1]
        ej += centers[1:]
    perm = np.random.default_rng(3).permutation(n)
    return inputs.edges_to_csr(n, perm[np.array(ei, dtype=np.int64)],
                               perm[np.array(ej, dtype=np.int64)])


GRAPHS = {
    "degrees": lambda: stars([d for d in range(18) for _ in range(3)] + [33, 300], False),
    "chained": lambda: stars(list(range(3, 18)) * 30, True),
    "tiny": lambda: stars([5], False),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("intercept", [False, True])
@pytest.mark.parametrize("name", sorted(GRAPHS))
def test_rows_of_every_degree(G, orc, name, intercept, prec):
    p = G.FP64 if prec == "fp64" else G.FP32_ACC64
    rp, cl = GRAPHS[name]()
    n = len(rp) - 1
    color, k = G.greedy_coloring(rp, cl)
    y = np.sin(np.arange(n) * 0.7) + 0.1 * np.random.default_rng(1).standard_normal(n)
    kw = dict(seed=8, instance=3, burn_in=2, intercept=intercept)
    ch = G.Chain(G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.9), y,
                 precision=p, **kw)
    assert ch.tile[0] == 1
    oc = orc.Chain(rp, cl, color, y, rho=0.9, **kw)
    for calls in (1, 7, 4):
        ch.sweep(calls)
    oc.sweeps(12)
    tol = 1e-12 if prec == "fp64" else 1e-4
    x, tau, lam, _ = ch.get_state()
    s1, s2, nacc = ch.get_accumulators()
    assert nacc == 10
    assert rel(x, oc.x) <= tol and rel(s1, oc.s1) <= tol and rel(s2, oc.s2) <= tol
    assert rel(tau, oc.tau) <= tol and rel(lam, oc.lam) <= tol
