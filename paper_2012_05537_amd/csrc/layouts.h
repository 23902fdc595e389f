// How the streaming kernels by source or output cell are dealt to blocks and
// lanes (host side; geometry only, laid out once per context).
#pragma once

#include <cstdint>

#include "sllbm_internal.h"

namespace sllbm {

// Three dimensions (k_stream_z, k_stream_zt).  A block holds tyc cells along y
// and cx columns of each.  While x rows are blocks (whole_rows), cx = N_x: the
// periodic row is complete and lane x writes output column x.  Longer rows are
// split into tiles of txc cells; a tile has halo columns more than it writes
// (forward: the last cell's far face; transposed: the group before the tile).
constexpr int ZNT = 256;              // most threads per block, but for one row of more nodes
struct ZLayout {
    int cx, txc, tyc, ntx, nty, nt;   // nt: threads per block
    float rcx;                        // 1 / cx
    int zcells, nchunk;               // cells along z per block, blocks along z
    unsigned blocks;                  // per plane (0: too many)
    bool nontemporal;                 // output stores (use_nontemporal)
};

// Cells along z per block of the forward kernel.  One source cell from order 3
// on: every load of a block is then in flight at once, and the blocks of an
// XCD cover a thin slab whose shared faces meet in its L2 (256^3 nodes, P = 4,
// FP64: 4.11 ms; marching 4, 16 or 64 cells with the next cell's rows in
// flight 4.28, 4.38 and 4.79 ms).  Cells of order 1 and 2 are too small for
// that and are marched (48 x 40 x 40 nodes, P = 2: 17.8 us with two cells, 20.8
// with one; 100 x 100 x 30, P = 1, FP32: 51 us with 30, 214 with one).
constexpr int z_max_cells(int p) { return p >= 3 ? 1 : p == 2 ? 2 : 32; }

// Of the transposed kernel: the P rows read again per block against the
// parallelism (P = 4: FP64, 256^3 nodes, 5.83, 4.98, 4.58, 4.41 and 4.37 ms with 1, 2, 4,
// 8 and 32 cells, 128^3 615 us with 4 and 8; FP32, four rows in flight, 128^3 290 us
// with 4 and 300 with 8; P = 1, 100 x 100 x 30: 93 us with 4, 41 us with 30)
constexpr int zt_max_cells(int p, size_t elem) { return p == 1 ? 32 : elem == 8 ? 8 : 4; }

// Longest row that may be a block of its own.  From order 5 on such a block's LDS
// (102 KB for 512 columns in FP64) leaves a CU one of them: 260 x 70 x 70 nodes, p = 5,
// FP64, S 364 us split and 491 whole, S^T 458 and 660.
constexpr int z_row(int p) { return p <= 4 ? 1024 : ZNT; }

// columns that the LDS of a block of nt threads holds (one P x P column per thread)
constexpr int z_columns(int nt)
{
    for (int n : {64, 128, 256, 384, 512, 768})
        if (nt <= n) return n;
    return 1024;
}

ZLayout z_layout(const Geometry &g, bool transpose, size_t elem);

// Two dimensions (k_stream_y): tyg groups of nc cells along y and cx
// columns of each per block; txc cells along x per tile (the whole row if ntx = 1)
constexpr int YNT = 512;              // most threads per block
struct YLayout {
    int cx, txc, tyg, ntx, nty, nt;
    float rcx;
    int nc;                           // source cells per lane: y_cells(p), or 1
    unsigned blocks;                  // per plane (0: too many)
};

// source cells per lane where there is more than one along y
constexpr int y_cells(int p) { return p >= 5 ? 1 : p >= 3 ? 2 : p == 2 ? 4 : 8; }

YLayout y_layout(const Geometry &g);

}  // namespace sllbm
