// Host-logic checks of how the streaming kernels are dealt to blocks; argv[1]
// names the check.  Prints what is wrong and exits non-zero on failure.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include "layouts.h"
using namespace sllbm;

static int fail(const char *what, const int n[3], int p)
{
    std::printf("%s: %d x %d x %d cells, p = %d\n", what, n[0], n[1], n[2], p);
    return 1;
}

// every grid of up to 60 million nodes has a launch of the streaming by departure
// cell, with less than 2^32 threads along each grid dimension
static int run_grids()
{
    const int sides[] = {1, 2, 3, 7, 16, 61, 200, 611, 900, 3000};
    for (int p = 3; p <= 6; ++p)
        for (int a : sides)
            for (int b : sides)
                for (int c : sides) {
                    const int n[3] = {a, b, c};
                    if (static_cast<int64_t>(a) * b * c * p * p * p > 60000000) continue;
                    for (size_t elem : {sizeof(float), sizeof(double)}) {
                        unsigned runs = 0;
                        const MappedRuns r = mapped_runs(p, n, elem);
                        if (!mapped_run_grid(r, n, runs)) return fail("no launch", n, p);
                        if (runs != static_cast<int64_t>(r.nx) * b * c || static_cast<int64_t>(runs) * 256 >> 32)
                            return fail("grid", n, p);
                    }
                }
    return 0;
}

static bool covers(int parts, int size, int n) { return parts * size >= n && (parts - 1) * size < n; }

static Geometry geometry(const int n[3], int p)
{
    Geometry g{};
    g.p = p;
    g.nodes = 1;
    for (int a = 0; a < 3; ++a) {
        g.nel[a] = n[a];
        g.N[a] = n[a] * p;
        g.nodes *= g.N[a];
    }
    return g;
}

// blocks cover every cell once, along each axis, with no block of them empty
static int layouts()
{
    const int sides[] = {1, 2, 3, 5, 8, 13, 32, 43, 64, 65, 86, 129, 256, 257, 512, 513, 2400};
    for (int p = 1; p <= 6; ++p)
        for (int a : sides)
            for (int b : sides) {
                for (int c : {1, 2, 12, 33, 70, 900}) {
                    const int n[3] = {a, b, c};
                    const Geometry g = geometry(n, p);
                    for (int t = 0; t < 2; ++t)
                        for (size_t elem : {sizeof(float), sizeof(double)}) {
                            const ZLayout l = z_layout(g, t == 1, elem);
                            const bool whole = l.ntx == 1;
                            if (!covers(l.ntx, l.txc, a) || !covers(l.nty, l.tyc, b) || !covers(l.nchunk, l.zcells, c))
                                return fail("cells", n, p);
                            if (l.nt > std::max(ZNT, l.tyc == 1 && whole ? z_row(p) : 0) || l.nt % 64 || l.cx * l.tyc > l.nt || l.nt - 64 >= l.cx * l.tyc)
                                return fail("threads", n, p);
                            if (l.cx != (whole ? g.N[0] : l.txc * p + (t ? p : 1)) || (g.N[0] <= ZNT && !whole))
                                return fail("columns", n, p);
                            const int64_t blocks = static_cast<int64_t>(l.ntx) * l.nty * l.nchunk;
                            if (l.blocks != (90 * blocks >> 31 ? 0 : blocks)) return fail("blocks", n, p);
                            if (l.zcells > (t ? zt_max_cells(p, elem) : z_max_cells(p))) return fail("march", n, p);
                        }
                }
                const int n[3] = {a, b, 1};
                Geometry g = geometry(n, p);
                g.nodes = static_cast<int64_t>(g.N[0]) * g.N[1];
                const YLayout l = y_layout(g);
                if (l.nc != (b == 1 ? 1 : y_cells(p))) return fail("cells per lane (2-D)", n, p);
                const int groups = (b + l.nc - 1) / l.nc;
                if (!covers(l.ntx, l.txc, a) || !covers(l.nty, l.tyg, groups)) return fail("cells (2-D)", n, p);
                if (l.nt > YNT || l.nt % 64 || l.cx * l.tyg > l.nt) return fail("threads (2-D)", n, p);
                if (l.cx != (l.ntx == 1 ? g.N[0] : l.txc * p + 1)) return fail("columns (2-D)", n, p);
                if (l.blocks != static_cast<unsigned>(l.ntx * l.nty)) return fail("blocks (2-D)", n, p);
            }
    return 0;
}

// a block's LDS holds no more columns than its threads round up to: at least four
// waves per SIMD fit a CU (160 KB) at order 4, two at order 6, whatever the block
static int lds_of_block()
{
    for (int nt = 64; nt <= z_row(4); nt += 64) {
        const int n[3] = {nt, 1, 1};
        if (nt > ZNT && static_cast<size_t>(4 * 4 * z_columns(nt)) * sizeof(double) > 160 * 1024) return fail("LDS", n, 4);
        if (nt > ZNT) continue;
        if (z_columns(nt) < nt || z_columns(nt) >= 2 * nt) return fail("columns", n, 1);
        for (int p = 4; p <= 6; ++p) {
            const int blocks = 160 * 1024 / static_cast<int>(p * p * z_columns(nt) * sizeof(double));
            if (blocks * nt / 256 < (p == 4 ? 4 : p == 5 ? 3 : 2) - (nt == 192 ? 1 : 0)) return fail("waves", n, p);
        }
    }
    return 0;
}

// non-temporal stores only where no two blocks share a cache line of an output row
static int nontemporal_rows()
{
    bool seen = false;
    for (int p = 1; p <= 6; ++p)
        for (int a : {16, 32, 48, 64, 72, 80, 96, 128, 256, 512, 1024})
            for (int b : {4, 32, 64}) {
                const int n[3] = {a, b, 64};
                const Geometry g = geometry(n, p);
                for (int t = 0; t < 2; ++t)
                    for (int elem : {4, 8}) {
                        const ZLayout l = z_layout(g, t == 1, elem);
                        const bool large = 90 * g.nodes * elem > int64_t(256) << 20;
                        if (l.nontemporal != (large && l.ntx == 1 && g.N[0] * elem % 128 == 0)) return fail("hint", n, p);
                        seen = seen || l.nontemporal;
                    }
            }
    return seen ? 0 : 1;
}

// runs cover the row of cells, fit their LDS, and are single cells before a grid has
// fewer than two blocks per CU
static int short_runs()
{
    for (int p = 3; p <= 6; ++p)
        for (int a = 1; a <= 40; ++a)
            for (int b : {1, 2, 3, 7, 16})
                for (size_t elem : {sizeof(float), sizeof(double)}) {
                    const int n[3] = {a, b, b};
                    const MappedRuns r = mapped_runs(p, n, elem);
                    if (!covers(r.nx, r.cells, a) || r.cells < 1 || r.cells > 16) return fail("cells", n, p);
                    if (r.width < r.cells * p + 1 || r.width % 2 == 0) return fail("width", n, p);
                    if (2 * (p + 1) * (p + 1) * r.width * elem > MAPPED_RUN_BYTES) return fail("LDS", n, p);
                    // (runs of equal length: a row of 5 cells has 3 or 5 of them)
                    if (r.cells > 2 && Q * r.nx * b * b < 512) return fail("blocks", n, p);
                }
    return 0;
}

int main(int argc, char **argv)
{
    if (argc == 2 && !std::strcmp(argv[1], "run_grids")) return run_grids();
    if (argc == 2 && !std::strcmp(argv[1], "layouts")) return layouts();
    if (argc == 2 && !std::strcmp(argv[1], "lds_of_block")) return lds_of_block();
    if (argc == 2 && !std::strcmp(argv[1], "nontemporal_rows")) return nontemporal_rows();
    if (argc == 2 && !std::strcmp(argv[1], "short_runs")) return short_runs();
    std::printf("unknown check\n");
    return 1;
}
