"""State reads on a thread whose last HIP error is the caller's own: they give
what they read, and leave the error to the caller.  More such reads than
there are pinned slots, so that none may keep its slot.
"""
import ctypes as C

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

INVALID_DEVICE = 101


@pytest.fixture(scope="module")
def G():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf

    gmrf.lib()
    return gmrf


@pytest.fixture
def hip():
    with open("/proc/self/maps") as f:
        paths = {ln.split()[-1] for ln in f if "libamdhip64" in ln}
    assert len(paths) == 1
    L = C.CDLL(paths.pop())
    yield L
    L.hipGetLastError()


@pytest.mark.parametrize("sites", [(48, 40), (300, 300)])
def test_reads_beside_the_callers_error(G, hip, sites):
    rng = np.random.default_rng(7)
    g = G.Graph(lattice=(*sites, 8))
    x0 = rng.standard_normal(g.n)
    ch = G.Chain(g, rng.standard_normal(g.n), precision=G.FP64, seed=1, x0=x0, intercept=True,
                 beta0=0.25)
    assert hip.hipSetDevice(1 << 20) == INVALID_DEVICE
    for _ in range(10):
        assert hip.hipPeekAtLastError() == INVALID_DEVICE
        x, tau, lam, sw = ch.get_state()
        assert np.array_equal(x, x0) and (tau, lam, sw) == (1.0, 1.0, 0)
        assert ch.beta0 == 0.25
        assert ch.last_reductions() == (0.0, 0.0)
    assert hip.hipGetLastError() == INVALID_DEVICE
