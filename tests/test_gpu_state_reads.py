"""Reads of a chain's state: fields just inside and just beyond what the pinned
read holds, both state buffers of a chain, graphs (a permuted layout), and
more threads and streams at once than there are pinned slots.  Exact: a read
moves bytes.
"""
import threading

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


def check(G, graph, prec, seed, stream=None, rounds=3):
    rng = np.random.default_rng(seed)
    x0 = rng.standard_normal(graph.n)
    if prec == G.FP32_ACC64:
        x0 = x0.astype(np.float32).astype(np.float64)
    ch = G.Chain(graph, rng.standard_normal(graph.n), precision=prec, seed=seed, stream=stream)
    for start in (0, 1, 2):
        ch.set_state(x0, 1.5, 2.5, start, stream=stream)
        x, tau, lam, sw = ch.get_state(stream=stream)
        assert np.array_equal(x, x0) and (tau, lam, sw) == (1.5, 2.5, start)
    zero = np.zeros(graph.n)
    for i in range(rounds):
        ch.set_accumulators(zero, zero, 0, stream=stream)
        ch.sweep(1, stream=stream)
        x, _, _, sw = ch.get_state(stream=stream)
        assert sw == 3 + i
        assert np.array_equal(x, ch.get_accumulators(stream=stream)[0])


# (256 KiB less the state block) / 8 = 32746 FP64 sites, / 4 = 65492 FP32 sites
@pytest.mark.parametrize("rows,cols,f64", [(1, 2, True), (48, 40, True), (14, 2339, True),
                                           (143, 229, True), (28, 2339, False), (3, 21831, False),
                                           (300, 300, True)])
def test_lattice_reads(G, rows, cols, f64):
    check(G, G.Graph(lattice=(rows, cols, 4)), G.FP64 if f64 else G.FP32_ACC64, rows + cols)


@pytest.mark.parametrize("n", [300, 40000])
@pytest.mark.parametrize("shape", [0, 1])
def test_graph_reads(G, n, shape):
    _, rp, cl = inputs.delaunay_graph(n, data_seed=2)
    color, k = G.greedy_coloring(rp, cl)
    g = G.Graph(row_ptr=rp, col_idx=cl, color=color, num_colors=k, rho=0.95)
    rng = np.random.default_rng(n)
    ch = G.Chain(g, rng.standard_normal(n), precision=G.FP64)
    ch.set_tile(shape)
    x0 = rng.standard_normal(n)
    ch.set_state(x0, 1.0, 1.0, 5)
    assert np.array_equal(ch.get_state()[0], x0)
    for _ in range(2):
        ch.set_accumulators(np.zeros(n), np.zeros(n), 0)
        ch.sweep(1)
        assert np.array_equal(ch.get_state()[0], ch.get_accumulators()[0])


def test_reads_of_many_threads(G):
    import torch

    errors = []
    device = torch.cuda.current_device()

    def work(i):
        try:
            torch.cuda.set_device(device)
            s = torch.cuda.Stream()
            check(G, G.Graph(lattice=(60 + i, 71, 8)), G.FP64, i, stream=s, rounds=12)
        except BaseException as e:      # reported by the main thread
            errors.append((i, e))

    threads = [threading.Thread(target=work, args=(i,)) for i in range(12)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
