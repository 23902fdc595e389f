// Layouts of the streaming kernels (layouts.h).
#include "layouts.h"

#include <algorithm>

#include "nt.h"

namespace sllbm {

ZLayout z_layout(const Geometry &g, bool transpose, size_t elem)
{
    const int halo = transpose ? g.p : 1, max_cells = transpose ? zt_max_cells(g.p, elem) : z_max_cells(g.p);
    // the split with the fewest idle lanes
    ZLayout b{};
    double best = 0.0;
    const bool whole = g.N[0] <= ZNT;
    const int t0 = whole ? g.nel[0] : (64 - halo) / g.p, t1 = whole ? g.nel[0] : (ZNT - halo) / g.p;
    for (int txc = t0; txc <= t1; ++txc) {
        const int cx = whole ? g.N[0] : txc * g.p + halo;
        const int ntx = (g.nel[0] + txc - 1) / txc;
        for (int tyc = 1; tyc <= g.nel[1] && cx * tyc <= ZNT; ++tyc) {
            const int nt = (cx * tyc + 63) / 64 * 64, nty = (g.nel[1] + tyc - 1) / tyc;
            const double used = static_cast<double>(g.nel[1]) * g.N[0] / (static_cast<double>(nt) * ntx * nty);
            if (used >= best) {
                best = used;
                b = ZLayout{cx, txc, tyc, ntx, nty, nt, 1.0f / static_cast<float>(cx), 0, 0, 0, false};
            }
        }
    }
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
    const int most = g.nodes <= 65536 ? 256 : YNT;         // lanes; small grids need the blocks
    const bool whole = g.N[0] <= most;
    const int nc = y_cells(g.p), groups = (g.nel[1] + nc - 1) / nc;
    const int t0 = whole ? g.nel[0] : 63 / g.p, t1 = whole ? g.nel[0] : (most - 1) / g.p;
    for (int txc = t0; txc <= t1; ++txc) {
        const int cx = whole ? g.N[0] : txc * g.p + 1, ntx = (g.nel[0] + txc - 1) / txc;
        for (int tyg = 1; tyg <= groups && cx * tyg <= std::max(cx, 256); ++tyg) {
            const int nt = (cx * tyg + 63) / 64 * 64, nty = (groups + tyg - 1) / tyg;
            const double used = static_cast<double>(groups) * g.N[0] / (static_cast<double>(nt) * ntx * nty);
            if (used >= best) {
                best = used;
                b = YLayout{cx, txc, tyg, ntx, nty, nt, 1.0f / static_cast<float>(cx), 0};
            }
        }
    }
    const int64_t blocks = static_cast<int64_t>(b.ntx) * b.nty;
    if (2 * Q2D * blocks <= (int64_t(1) << 31) - 1) b.blocks = static_cast<unsigned>(blocks);
    return b;
}

}  // namespace sllbm
