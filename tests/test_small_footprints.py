"""Workspaces of lattices within one tile (no GPU needed): in proportion to
their sites, the memory for normals drawn ahead beside them and by their own
quads, and jobs admitted by them.
"""
import ctypes as C

import numpy as np
import pytest

from paper_1702_05518_amd import gmrf, serve


class HostLattice:
    """A lattice graph handle; a lattice needs no device memory."""

    def __init__(self, rows, cols, st=8):
        d = gmrf._Desc(lattice=(rows, cols, st))
        self.handle, self.n = C.c_void_p(), rows * cols
        assert gmrf.lib().gmrf_graph_create(C.byref(d.desc), None, 0, None,
                                            C.byref(self.handle)) == gmrf.OK

    def __del__(self):
        gmrf.lib().gmrf_graph_destroy(self.handle)


SIZES = [(1, 1), (1, 63), (3, 3), (16, 16), (50, 50), (63, 64), (64, 64), (64, 65), (200, 90)]


@pytest.mark.parametrize("rows,cols", SIZES)
@pytest.mark.parametrize("prec,real", [(gmrf.FP64, 8), (gmrf.FP32_ACC64, 4)])
def test_footprint_is_proportional(rows, cols, prec, real):
    L = gmrf.lib()
    one, g = HostLattice(1, 1), HostLattice(rows, cols)
    more = L.gmrf_chain_footprint(g.handle, prec) - L.gmrf_chain_footprint(one.handle, prec)
    # x twice and y, S1 and S2, the statistics area, and six doubles per
    # 32 x 32 tile, each area rounded up to 256 bytes
    tiles = -(-rows // 32) * -(-cols // 32)
    assert 0 <= more <= (3 * real + 32) * g.n + 48 * tiles + 7 * 256
    assert L.gmrf_chain_footprint(one.handle, prec) <= 16 << 10


@pytest.mark.parametrize("rows,cols", SIZES)
@pytest.mark.parametrize("prec,real", [(gmrf.FP64, 8), (gmrf.FP32_ACC64, 4)])
def test_ahead_bytes(rows, cols, prec, real):
    g = HostLattice(rows, cols)
    quads = (rows + 1) // 2 * ((cols + 1) // 2) if max(rows, cols) <= 64 else 0
    assert gmrf.lib().gmrf_chain_ahead_bytes(g.handle, prec) == 128 * 4 * real * quads
    # the statistics area holds at least one sweep's
    assert 4 * real * quads <= (16 * g.n + 255) // 256 * 256


def test_ahead_arguments():
    L = gmrf.lib()
    assert L.gmrf_chain_ahead_bytes(None, gmrf.FP64) == 0
    assert L.gmrf_chain_ahead_bytes(HostLattice(4, 4).handle, 7) == 0
    assert L.gmrf_chain_set_ahead(None, None, 0) == gmrf.E_INVALID_ARG


def test_admission():
    """Thirty 50 x 50 FP64 jobs fit in 5 MB."""
    g = HostLattice(50, 50)
    budget = 5 << 20
    assert 30 * serve.chain_bytes(g, gmrf.FP64) <= budget
    server = serve.Server(budget_bytes=200_000)
    server.submit(serve.Job(0, g, np.zeros(g.n), seed=1, instance=0, precision=gmrf.FP64))
    assert len(server.waiting) == 1
