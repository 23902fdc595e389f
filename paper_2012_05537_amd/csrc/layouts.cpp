// Layouts of the streaming kernels (layouts.h).
#include "layouts.h"

#include <algorithm>

#include "nt.h"

namespace sllbm {

// Whether x rows may be blocks: a whole row has no halo, and its stores are whole
// lines.  FP64, p = 4, rows of 280 and 384 nodes (as many lanes idle as in tiles): S 542 ->
// 506 and 492 -> 416 us, S^T 637 -> 619 and 576 -> 490; 260 nodes (19 % idle against 10 %):
// S 322 -> 317, S^T 376 -> 398, in FP32 212 -> 160 and 222 -> 206.  Rows of more than 256
// nodes make few blocks of small grids: 288 x 32 x 32 S^T 113 -> 118 us, in FP32 42 -> 50,
// 384 x 16 x 16 S 24 -> 27.  Rows of more than 512 leave a CU one block (p = 4) and
// gain where the tiles break their lines (1024 x 32 x 32, p = 2, FP64: S 328 -> 288, S^T 357
// -> 308; 1024 x 40 x 40, p = 4, FP32: 287 -> 217, 337 -> 286; but 600 x 48 x 48, p = 4, FP64,
// S 399 -> 460).
static bool whole_rows(const Geometry &g, size_t elem)
{
    if (g.N[0] <= ZNT) return true;
    if (g.N[0] > z_row(g.p) || 90 * g.nodes * static_cast<int64_t>(elem) <= INFINITY_CACHE_BYTES) return false;
    return g.N[0] <= 512 || g.N[0] * elem % 128 == 0;
}

ZLayout z_layout(const Geometry &g, bool transpose, size_t elem)
{
    const int halo = transpose ? g.p : 1, max_cells = transpose ? zt_max_cells(g.p, elem) : z_max_cells(g.p);
    // the split with the fewest idle lanes
    ZLayout b{};
    double best = 0.0;
    auto consider = [&](int txc, int cx, double weight) {
        const int ntx = (g.nel[0] + txc - 1) / txc;
        for (int tyc = 1; tyc <= g.nel[1] && (tyc == 1 || cx * tyc <= ZNT); ++tyc) {
            const int nt = (cx * tyc + 63) / 64 * 64, nty = (g.nel[1] + tyc - 1) / tyc;
            const double used = weight * g.nel[1] * g.N[0] / (static_cast<double>(nt) * ntx * nty);
            if (used >= best) {
                best = used;
                b = ZLayout{cx, txc, tyc, ntx, nty, nt, 1.0f / static_cast<float>(cx), 0, 0, 0, false};
            }
        }
    };
    if (g.N[0] > ZNT)
        for (int txc = (64 - halo) / g.p; txc <= (ZNT - halo) / g.p; ++txc) consider(txc, txc * g.p + halo, 1.0);
    if (whole_rows(g, elem)) consider(g.nel[0], g.N[0], 1.12);
    // Cells along z per block: at most max_cells, fewer while the grid has fewer
    // than 1280 blocks of 256 threads, five per CU (transposed kernel, 64^3 nodes,
    // FP64: 86, 85 and 92 us with 2, 4 and 8 blocks per CU).
    constexpr int TARGET_BLOCKS = 1280;
    const int64_t tiles = static_cast<int64_t>(b.ntx) * b.nty;
    const int64_t want = (static_cast<int64_t>(TARGET_BLOCKS) * ZNT / b.nt + 90 * tiles - 1) / (90 * tiles);
    const int n = std::max(static_cast<int>(std::min<int64_t>(g.nel[2], want)), (g.nel[2] + max_cells - 1) / max_cells);
    b.zcells = (g.nel[2] + n - 1) / n;
    b.nchunk = (g.nel[2] + b.zcells - 1) / b.zcells;
    // (the grid is blocks x 90: with one dimension its threads would pass 2^32 on
    // the largest grids)
    if (90 * tiles * b.nchunk <= (int64_t(1) << 31) - 1) b.blocks = static_cast<unsigned>(tiles * b.nchunk);
    // Tiles of a split row end inside a cache line, which the next tile's block
    // completes (FP64, p = 4: 384 x 64 x 64 nodes, S 492 us, with the hint 558; 512 x
    // 64 x 64 579 and 614, S^T 704 and 715)
    const int64_t value = static_cast<int64_t>(elem);
    b.nontemporal = b.ntx == 1 && use_nontemporal(90 * g.nodes * value, g.N[0] * value);
    return b;
}

YLayout y_layout(const Geometry &g)
{
    // the split with the fewest idle lanes
    YLayout b{};
    double best = 0.0;
    // small grids need the blocks (512 x 64 nodes, p = 4, FP64, without launch overhead: 5.4
    // us in tiles and 6.4 in whole rows, 400 x 128 7.7 and 8.0; 400 x 400 rows are whole)
    const int most = g.nodes <= 65536 ? 256 : YNT;         // lanes
    const bool whole = g.N[0] <= most;
    // a tube of one cell has no second one to load (3200 x 1 cells, p = 1, FP64: 2.75 us,
    // and 3.07 with eight cells per lane; 800 x 1, p = 4: 3.58 and 3.92)
    const int nc = g.nel[1] == 1 ? 1 : y_cells(g.p), groups = (g.nel[1] + nc - 1) / nc;
    const int t0 = whole ? g.nel[0] : 63 / g.p, t1 = whole ? g.nel[0] : (most - 1) / g.p;
    for (int txc = t0; txc <= t1; ++txc) {
        const int cx = whole ? g.N[0] : txc * g.p + 1, ntx = (g.nel[0] + txc - 1) / txc;
        for (int tyg = 1; tyg <= groups && cx * tyg <= std::max(cx, 256); ++tyg) {
            const int nt = (cx * tyg + 63) / 64 * 64, nty = (groups + tyg - 1) / tyg;
            const double used = static_cast<double>(groups) * g.N[0] / (static_cast<double>(nt) * ntx * nty);
            if (used >= best) {
                best = used;
                b = YLayout{cx, txc, tyg, ntx, nty, nt, 1.0f / static_cast<float>(cx), nc, 0};
            }
        }
    }
    const int64_t blocks = static_cast<int64_t>(b.ntx) * b.nty;
    if (2 * Q2D * blocks <= (int64_t(1) << 31) - 1) b.blocks = static_cast<unsigned>(blocks);
    return b;
}

}  // namespace sllbm
