// chunk_rows_check.cpp -- host-only check of the tables that the chunked sweep
// kernel reads (row heads, neighbour groups, LDS sizes), built with
// AddressSanitizer and UndefinedBehaviorSanitizer by
// tests/test_sanitize_chunk_rows.py.  Reads the graph files of
// graph_check.cpp.  Exit status 0 when every check holds; the first failed
// check is printed.
#include <algorithm>
#include <cstdio>
#include <fstream>
#include <vector>

#include "internal.hpp"

using namespace gmrf;

#define CHECK(cond)                                                                  \
    do {                                                                             \
        if (!(cond)) {                                                               \
            std::fprintf(stderr, "graph %d: check failed: %s (line %d)\n", gi, #cond, \
                         __LINE__);                                                  \
            return 1;                                                                \
        }                                                                            \
    } while (0)

static int check_rows(int gi, const HostGraph &g)
{
    const int32_t k = g.k;
    CHECK((int32_t)g.ch_head.size() == g.nchunks + 1 && (int32_t)g.ch_grp.size() == g.nchunks + 1);
    CHECK(g.ch_head[0] == 0 && g.ch_grp[0] == 0);
    CHECK(g.ch_head.back() == (int32_t)g.loc_head.size());
    CHECK(4 * (size_t)g.ch_grp.back() == g.loc_grp.size());
    int64_t lds4 = 0, lds8 = 0;
    for (int32_t b = 0; b < g.nchunks; ++b) {
        const int32_t l0 = g.ch_loc[b], nloc = g.ch_loc[b + 1] - l0;
        const int32_t nr = g.ch_meta[(size_t)b * (3 * k + 1) + k];
        const int32_t h0 = g.ch_head[b], nhead = g.ch_head[b + 1] - h0;
        const int32_t g0 = g.ch_grp[b], ngrp = g.ch_grp[b + 1] - g0;
        // whole 16-byte vectors, the last heads 0
        CHECK(h0 % 4 == 0 && g0 % 2 == 0 && nhead == (nr + 3) / 4 * 4);
        for (int32_t i = nr; i < nhead; ++i)
            CHECK(g.loc_head[h0 + i] == 0);
        const uint16_t *grp = g.loc_grp.data() + 4 * (size_t)g0;
        const int32_t fill = 4 * nloc;      // the slot past the staged sites
        CHECK(fill <= 65535);
        for (int j = 0; j < 4; ++j)         // group 0: no neighbours
            CHECK(grp[j] == fill);
        int32_t next = 1;                   // groups follow each other in row order
        for (int32_t s = 0; s < nr; ++s) {
            const int32_t u = g.loc_site[l0 + s];
            const int32_t deg = (int32_t)(g.loc_head[h0 + s] & 0xffffu);
            CHECK(deg == g.row_ptr[u + 1] - g.row_ptr[u]);
            CHECK((int32_t)(g.loc_head[h0 + s] >> 16) == next);
            for (int32_t e = 0; e < (deg + 3) / 4 * 4; ++e) {
                CHECK(next + e / 4 < ngrp);
                const int32_t w = grp[4 * next + e];
                if (e >= deg) {
                    CHECK(w == fill);
                    continue;
                }
                CHECK(w % 4 == 0 && w < fill);
                CHECK(g.loc_site[l0 + w / 4] == g.col[g.row_ptr[u] + e]);   // same order
            }
            next += (deg + 3) / 4;
        }
        CHECK(ngrp == (next + 1) / 2 * 2);
        for (int32_t i = 4 * next; i < 4 * ngrp; ++i)
            CHECK(grp[i] == fill);
        lds4 = std::max(lds4, sweep_lds_bytes(nloc, nr, ngrp, 4));
        lds8 = std::max(lds8, sweep_lds_bytes(nloc, nr, ngrp, 8));
    }
    // the launch reserves the largest image
    CHECK(lds4 == g.max_lds4 && lds8 == g.max_lds8 && lds8 <= kFusedLaunchLds);
    // at least the bytes that the caps bound, at most half as much again (and
    // what rounding and group 0 add)
    CHECK(g.max_lds4 >= g.max_image4 && g.max_lds4 <= g.max_image4 * 3 / 2 + 64);
    CHECK(g.max_lds8 >= g.max_image8 && g.max_lds8 <= g.max_image8 * 3 / 2 + 64);
    return 0;
}

int main(int argc, char **argv)
{
    if (argc != 2) {
        std::fprintf(stderr, "usage: chunk_rows_check FILE\n");
        return 2;
    }
    std::ifstream f(argv[1], std::ios::binary);
    int gi = 0, chunked = 0, rc = 0;
    for (;; ++gi) {
        int64_t n = 0, nnz = 0;
        int32_t k = 0;
        double rho = 1.0;
        if (!f.read((char *)&n, 8))
            break;
        f.read((char *)&nnz, 8);
        f.read((char *)&k, 4);
        f.read((char *)&rho, 8);
        std::vector<int64_t> rp(n + 1);
        std::vector<int32_t> cl(nnz), color(n);
        f.read((char *)rp.data(), 8 * (n + 1));
        f.read((char *)cl.data(), 4 * nnz);
        f.read((char *)color.data(), 4 * n);
        if (!f)
            return 2;
        gmrf_graph_desc d{};
        d.n = n;
        d.row_ptr = rp.data();
        d.col_idx = cl.data();
        d.color = color.data();
        d.num_colors = k;
        d.rho = rho;
        HostGraph g;
        CHECK(build_host_graph(&d, &g) == GMRF_OK);
        if (!g.chunks_ok)
            continue;
        ++chunked;
        const size_t bytes = graph_device_bytes(g);
        drop_chunk_rows(&g);                // nothing below, and no upload, needs them
        CHECK(g.loc_row.capacity() == 0 && g.loc_adj.capacity() == 0);
        CHECK(graph_device_bytes(g) == bytes);
        rc |= check_rows(gi, g);
    }
    std::printf("checked %d graphs, %d with chunk tables\n", gi, chunked);
    return rc;
}
