"""The binomial model's color passes as one chunked launch, what a new chain
runs: chunk edges (512 owned sites), hubs (more than twelve and more than 64
neighbours), sites without trials or neighbours, both precisions, captured
and plain sweeps, and a shape set between sweeps, against the CPU oracle.

FP64 within 1e-12 relative (sums of the same terms in another order); FP32,
one sweep from a common state, within 64 rounding errors of the field's size
(a neighbour sum and five roundings per color, at most eight colors deep).
"""
import numpy as np
import pytest

from paper_1702_05518_amd import inputs

pytestmark = pytest.mark.gpu

RTOL64 = 1e-12


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return float(np.max(np.abs(a - b)) / max(np.max(np.abs(b)), 1e-300))


def graph(kind):
    if kind == "wheel":                 # a hub of 700 neighbours on a ring
        ring = np.arange(1, 701)
        return inputs.edges_to_csr(701, np.r_[np.zeros(700, dtype=np.int64), ring],
                                   np.r_[ring, np.roll(ring, -1)])
    if kind == "stars":                 # hubs of 13, 64 and 65 neighbours, two lone sites
        ei, ej, n = [], [], 0
        for m in (13, 64, 65):
            ei += [n] * m
            ej += list(range(n + 1, n + 1 + m))
            n += m + 1
        return inputs.edges_to_csr(n + 2, np.array(ei), np.array(ej))
    return inputs.delaunay_graph(int(kind), data_seed=6)[1:]


def pair(orc, kind, f64, intercept):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf as G

    rp, cl = graph(kind)
    n = len(rp) - 1
    color, k = G.greedy_coloring(rp, cl)
    rng = np.random.default_rng(n)
    trials = rng.integers(1, 40, n).astype(np.int32)
    trials[np.flatnonzero(np.diff(rp) > 0)[::7]] = 0
    y = rng.binomial(trials, 0.4).astype(np.float64)
    kw = dict(seed=5, instance=1, intercept=intercept, beta0_var=50.0 if intercept else 0.0,
              trials=trials, burn_in=5)
    g = G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.95)
    ch = G.Chain(g, y, precision=G.FP64 if f64 else G.FP32_ACC64, **kw)
    oc = orc.Chain(rp, cl, color, y, rho=0.95, **kw)
    x0 = (0.5 * rng.standard_normal(n)).astype(np.float32).astype(np.float64)
    ch.set_state(x0, 2.0, 1.0, 3)
    oc.set_state(x0, 2.0, 1.0, 3, beta0=0.0)
    return ch, oc


@pytest.mark.parametrize("intercept", [True, False])
@pytest.mark.parametrize("kind", ["511", "513", "1500", "wheel", "stars"])
def test_sweeps(orc, kind, intercept):
    ch, oc = pair(orc, kind, True, intercept)
    for step in range(4):
        if step == 3:
            ch.set_tile(0)              # the same field goes on in another shape
        ch.sweep(3, capture=step == 1)
        oc.sweeps(3)
        x, tau, _, _ = ch.get_state()
        q, spsi = ch.last_reductions()
        assert rel(x, oc.x) <= RTOL64
        assert rel(tau, oc.tau) <= RTOL64 and abs(ch.beta0 - oc.beta0) <= RTOL64
        assert rel(q, oc.q) <= RTOL64 and rel(spsi, oc.sse) <= RTOL64
    m, v, _ = ch.posterior_stats()
    om, ov = oc.stats()
    assert rel(m, om) <= RTOL64 and rel(v, ov) <= 1e-9


@pytest.mark.parametrize("kind", ["513", "wheel", "stars"])
def test_fp32_sweep(orc, kind):
    ch, oc = pair(orc, kind, False, True)
    ch.sweep(1)
    oc.sweeps(1)
    x, _, _, _ = ch.get_state()
    assert np.max(np.abs(x - oc.x)) <= 64 * 2.0 ** -24 * max(1.0, np.max(np.abs(oc.x)))
