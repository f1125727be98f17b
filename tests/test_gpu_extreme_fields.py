"""Fields beyond 1e154, whose squares overflow, under the intrinsic prior: q is
a sum over edges alone, so q and tau stay finite, in every lattice shape and
in batches.  Against the CPU oracle.

Neighbours differ by 1e-6 of the field, so a difference of two values within
a few roundings of the oracle's is within 8 x 2^-53 / 1e-6 of its difference,
and q within twice that: 2e-9.
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


@pytest.mark.parametrize("rows,cols,stencil,shape", [
    (50, 50, 8, 2), (50, 50, 8, 0), (64, 64, 4, 2), (140, 200, 8, 0), (140, 200, 8, 1),
    (140, 200, 4, 0), (50, 50, 8, None)])
def test_intrinsic_field_near_the_largest_square(G, orc, rows, cols, stencil, shape):
    wl = inputs.lattice_workload(rows, cols, stencil, data_seed=3)
    rng = np.random.default_rng(rows + cols)
    n = rows * cols
    y = 2e154 * (1.0 + 1e-6 * rng.standard_normal(n))
    x0 = 2e154 * (1.0 + 1e-6 * rng.standard_normal(n))
    ch = G.Chain(G.Graph(lattice=(rows, cols, stencil)), y, precision=G.FP64, seed=4, x0=x0)
    oc = orc.Chain(wl["row_ptr"], wl["col"], wl["color"], y, seed=4)
    oc.set_state(x0, 1.0, 1.0, 0)
    if shape is None:
        G.Batch([ch]).sweep(1)
    else:
        ch.set_tile(shape)
        ch.sweep(1)
    oc.sweeps(1)
    q, sse = ch.last_reductions()
    _, tau, lam, _ = ch.get_state()
    assert np.isfinite(oc.q) and abs(q - oc.q) <= 2e-9 * oc.q
    assert abs(sse - oc.sse) <= 2e-9 * oc.sse
    assert abs(tau - oc.tau) <= 2e-9 * oc.tau and abs(lam - oc.lam) <= 2e-9 * oc.lam
