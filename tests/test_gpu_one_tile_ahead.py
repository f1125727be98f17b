"""Site normals drawn ahead into memory of any size: the workspace's own, a
buffer of one sweep's, of seven sweeps', of all.  Exact: the chains agree bit
for bit with each other and with the tile kernel, and nothing beyond the
buffer is written.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_05518_amd import gmrf

    gmrf.lib()
    return gmrf


def lend(G, ch, nbytes):
    import torch

    buf = torch.full((nbytes + 4096,), 0xAB, dtype=torch.uint8, device="cuda")
    G._check(G.lib().gmrf_chain_set_ahead(ch.handle, G.C.c_void_p(buf.data_ptr()), nbytes))
    return buf


def result(ch):
    x, tau, lam, sw = ch.get_state()
    s1, s2, n = ch.get_accumulators()
    return np.concatenate([x, s1, s2, [tau, lam, sw, n, ch.beta0, *ch.last_reductions()]])


@pytest.mark.parametrize("rows,cols,stencil,f64,b0,rng", [
    (1, 1, 8, True, False, 1), (1, 63, 4, True, True, 1), (3, 3, 8, False, False, 1),
    (50, 49, 8, True, True, 1), (63, 64, 4, False, False, 2), (64, 64, 8, True, False, 2),
    (64, 64, 4, False, True, 1), (7, 64, 8, True, False, 1)])
def test_any_memory(G, rows, cols, stencil, f64, b0, rng):
    prec = G.FP64 if f64 else G.FP32_ACC64
    g = G.Graph(lattice=(rows, cols, stencil), rho=0.9)
    y = np.random.default_rng(rows).standard_normal(g.n)
    kw = dict(precision=prec, seed=3, intercept=b0, burn_in=2, rng_version=rng)
    each = 4 * (8 if f64 else 4) * ((rows + 1) // 2) * ((cols + 1) // 2)
    full = G.Chain(g, y, **kw)
    own, tiles = G.Chain(g, y, ahead=False, **kw), G.Chain(g, y, **kw)
    tiles.set_tile(0)
    chains, bufs = [own, tiles], []
    for nbytes in (0, each - 1, each, 7 * each + 3, 200 * each):
        ch = G.Chain(g, y, ahead=False, **kw)
        bufs.append((nbytes, lend(G, ch, nbytes)))
        chains.append(ch)
    for nsweeps, capture in ((1, False), (131, False), (9, True), (9, True)):
        full.sweep(nsweeps, capture=capture)
        want = result(full)
        for ch in chains:
            ch.sweep(nsweeps, capture=capture)
            assert np.array_equal(result(ch), want)
    for nbytes, buf in bufs:
        assert (buf[nbytes:] == 0xAB).all()


def test_buffers_change_under_captured_sweeps(G):
    g = G.Graph(lattice=(40, 48, 8))
    y = np.random.default_rng(1).standard_normal(g.n)
    a, b = G.Chain(g, y, seed=9), G.Chain(g, y, seed=9, ahead=False)
    bufs = []
    for i, nbytes in enumerate((0, 5 * 8 * g.n, 3 * 8 * g.n, 0)):
        if i == 3:
            G._check(G.lib().gmrf_chain_set_ahead(b.handle, None, 0))
        else:
            bufs.append(lend(G, b, nbytes))
        a.sweep(12, capture=True)
        b.sweep(12, capture=True)
        assert np.array_equal(result(a), result(b))
        m, v, _ = a.posterior_stats()           # the statistics area between calls
        bm, bv, _ = b.posterior_stats()
        assert np.array_equal(m, bm) and np.array_equal(v, bv)
    with pytest.raises(G.GmrfError):            # not at a multiple of 256 bytes
        G._check(G.lib().gmrf_chain_set_ahead(b.handle, G.C.c_void_p(bufs[0].data_ptr() + 8), 64))
