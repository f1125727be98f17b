"""The lattice tile kernels at the edges of their tiles and groups: lattices
one site either side of whole tiles and of their halos, single rows and
columns, odd widths (unaligned pairs), both stencils, both tile shapes, with
and without the intercept and the paired random-number contract; calls whose
sweep counts cut the groups of deferred accumulation anywhere, across the
burn-in boundary.

However a run is cut into calls, the field, the accumulators and the
precisions are the same bits (each accumulator takes the same additions in
the same order).  FP64 agrees with the oracle to 1e-12 relative per field
(the bound of one instruction sequence against another over a few sweeps),
FP32 to 1e-4, the criterion of the FP32 chains."""
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


CASES = [
    # rows, cols, stencil, shape, intercept, rng_version
    (1, 1, 4, 1, False, 1), (1, 70, 8, 0, True, 1), (67, 1, 4, 0, False, 1),
    (2, 3, 8, 1, True, 1), (64, 64, 8, 0, False, 1), (65, 63, 8, 0, True, 1),
    (66, 68, 8, 0, False, 2), (67, 131, 4, 0, True, 1), (130, 132, 8, 0, False, 2),
    (194, 203, 8, 0, True, 1), (195, 196, 4, 0, False, 2), (194, 197, 4, 0, True, 1),
    (32, 33, 8, 1, True, 1), (98, 101, 8, 1, False, 1), (99, 100, 4, 1, True, 2),
    (97, 99, 4, 1, False, 1),
]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("rows,cols,st,shape,intercept,rng", CASES)
def test_tiles_and_groups(G, orc, rows, cols, st, shape, intercept, rng, prec):
    p = G.FP64 if prec == "fp64" else G.FP32_ACC64
    wl = inputs.lattice_workload(rows, cols, st, data_seed=rows + cols)
    kw = dict(seed=rows * cols, burn_in=4, intercept=intercept, rng_version=rng)
    g = G.Graph(lattice=(rows, cols, st))
    runs = [[1] * 14, [14], [2, 7, 5], [3, 11]]
    out = []
    for calls in runs:
        ch = G.Chain(g, wl["y"], precision=p, **kw)
        ch.set_tile(shape)
        for i, k in enumerate(calls):
            ch.sweep(k, capture=len(calls) == 3 and i == 1)
        x, tau, lam, sw = ch.get_state()
        s1, s2, nacc = ch.get_accumulators()
        assert sw == 14 and nacc == 10
        out.append((x, s1, s2, tau, lam, ch.beta0))
    for other in out[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(out[0], other))
    oc = orc.Chain(wl["row_ptr"], wl["col"], wl["color"], wl["y"], **kw)
    oc.sweeps(14)
    tol = 1e-12 if prec == "fp64" else 1e-4
    x, s1, s2, tau, lam, b0 = out[0]
    assert rel(x, oc.x) <= tol and rel(s1, oc.s1) <= tol and rel(s2, oc.s2) <= tol
    assert rel(tau, oc.tau) <= tol and rel(lam, oc.lam) <= tol
    if intercept:
        assert rel(b0, oc.beta0) <= tol
