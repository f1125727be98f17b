"""Sanitizer build (CPU only) of the graph builder under
tests/sanitize/chunk_rows_check.cpp: the row heads, neighbour groups and LDS
sizes that the chunked sweep kernel reads, on graphs whose rows end at every
place of a group, of degree 0 and 1, with hubs, and of many chunks.
"""
import os
import subprocess

import numpy as np

from paper_1702_05518_amd import inputs
from test_sanitizers import CSRC, ROOT, SAN, colored, runtime, write_graphs


def test_chunk_rows_under_sanitizers(tmp_path):
    runtime("libasan.so")
    exe = str(tmp_path / "chunk_rows_check")
    subprocess.run(["g++", "-std=c++17", *SAN, "-D__HIP_PLATFORM_AMD__",
                    "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-I", "/opt/rocm/include",
                    os.path.join(ROOT, "tests", "sanitize", "chunk_rows_check.cpp"),
                    os.path.join(CSRC, "graph_host.cpp"), "-o", exe], check=True)
    pairs = np.arange(0, 4000, 2)                    # degree 1 throughout
    stars = [[], [], 0]                              # hubs of 1 .. 17 neighbours
    for m in range(1, 18):
        stars[0] += [stars[2]] * m
        stars[1] += list(range(stars[2] + 1, stars[2] + 1 + m))
        stars[2] += m + 1
    few = np.array([0, 1]), np.array([1, 2])         # sites 3 .. 699 isolated
    graphs = [colored(*inputs.delaunay_graph(3000, data_seed=2)[1:]),
              colored(*inputs.delaunay_graph(60000, data_seed=9)[1:], rho=0.95),
              colored(*inputs.lattice_csr(40, 30, 8)),
              colored(*inputs.edges_to_csr(4000, pairs, pairs + 1)),
              colored(*inputs.edges_to_csr(stars[2], np.array(stars[0]), np.array(stars[1]))),
              colored(*inputs.edges_to_csr(700, *few), rho=0.5),
              colored(*inputs.edges_to_csr(301, np.zeros(300, np.int64), np.arange(1, 301))),
              colored(*inputs.path_graph(1100))]
    data = str(tmp_path / "graphs.bin")
    write_graphs(data, graphs)
    env = dict(os.environ, ASAN_OPTIONS="detect_leaks=1",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    r = subprocess.run([exe, data], capture_output=True, text=True, env=env, timeout=600)
    assert r.returncode == 0, r.stdout + r.stderr
    assert f"checked {len(graphs)} graphs, {len(graphs)} with chunk tables" in r.stdout
