// Two-dimensional semi-Lagrangian streaming (Sec. II A, Eqs. (8)-(9) with
// D = 2) on a periodic mesh of equal cells, by source cell: the D2Q19
// counterpart of stream.hip.
//
// The outputs that read source cell c along an axis are P consecutive nodes,
// (c - omin - 1)*P + lstar + j, j = 0 .. P-1, with weight row (lstar + j) mod P.
// A lane takes one column (x) of NC source cells in a row along y (one, where the
// grid has no more): it loads their
// NC*P + 1 nodes (all in flight at once), interpolates along y in registers with
// the velocity's uniform weights and leaves NC*P values in LDS, from which the
// block's lanes interpolate along x, one output column each.  While N_x <= 512 a
// block holds whole periodic rows; longer rows are split into tiles of whole
// cells (N_x <= 256 up to 65536 nodes).
#include <hip/hip_runtime.h>

#include "layouts.h"
#include "rows.h"
#include "sllbm_internal.h"
#include "xcd.h"

namespace sllbm {

// Bound by HBM and, while two states fit it, the Infinity Cache: 512^2 nodes, P =
// 4, 24 us in FP64 (6.5 TB/s) and 14 us in FP32; 1024^2 115 us; 510^2 at P = 6 25 us;
// the Sod tube of 800 x 4 nodes 3.0 us (3.3 with the march).
// The march along y that this replaces (strips of 256 columns, chunks of 16
// cells, each row interpolated along x out of LDS) took 26, 17, 127 and 33 us.
template <typename S, int P, int NC>
__global__ void __launch_bounds__(YNT) k_stream_y(Geometry g, CellTables<S> tab, const S *__restrict__ in,
                                                  S *__restrict__ out, YLayout lay)
{
    constexpr int R = NC * P + 1;
    __shared__ S buf[NC * P][YNT];
    const int tid = threadIdx.x;
    const int tiles = lay.ntx * lay.nty;
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                            static_cast<int>(gridDim.x * gridDim.y)));
    const int q = L / tiles, tile = L - q * tiles;
    const int ty = tile / lay.ntx, tx = tile - ty * lay.ntx;
    const int i = q % Q2D, pop = q / Q2D;
    const int Nx = g.N[0], Ny = g.N[1];
    const int64_t N = g.nodes;
    const int omx = tab.omin[i * 3 + 0], omy = tab.omin[i * 3 + 1];
    const int lsx = tab.lstar[i * 3 + 0], lsy = tab.lstar[i * 3 + 1];
    const S *Wx = tab.w + (i * 3 + 0) * P * (P + 1);
    using CS = const __attribute__((address_space(4))) S;
    CS *Wy = (CS *)(tab.w + (i * 3 + 1) * P * (P + 1));
    const GlobalRow<S> src = plane_row(const_cast<S *>(in), static_cast<int64_t>(pop * Q2D + i) * N);
    const GlobalRow<S> dst = plane_row(out, static_cast<int64_t>(pop * Q2D + i) * N);

    // exact quotient: (tid + 1/2) / cx lies at least 1 / (2 cx) from an integer
    const int gl = static_cast<int>((static_cast<float>(tid) + 0.5f) * lay.rcx), xl = tid - gl * lay.cx;
    const int cx0 = tx * lay.txc, ncx = min(lay.txc, g.nel[0] - cx0);
    const bool whole = lay.ntx == 1;
    const int c0 = (ty * lay.tyg + gl) * NC;               // this lane's cells along y: c0 .. c0 + NC - 1
    int xs = cx0 * P + min(xl, whole ? Nx - 1 : ncx * P);
    xs -= xs >= Nx ? Nx : 0;
    S v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int y = min(c0 * P + r, Ny);                 // past the last cell: its far face again, unused
        v[r] = load_at<S>(src, plane_offset<S>((y == Ny ? 0 : y) * Nx + xs));
    }
    // output column and its taps in the block's row of columns
    int xo, cell, row;
    if (whole) {
        xo = xl;
        row = xl % P;
        cell = xl / P + wrapi(omx, g.nel[0]) + (row >= lsx ? 1 : 0);
        cell -= cell >= g.nel[0] ? g.nel[0] : 0;
        cell -= cell >= g.nel[0] ? g.nel[0] : 0;
    } else {
        cell = xl / P;
        const int j = lsx + xl % P;
        row = j % P;
        xo = wrapi((cx0 - omx - 1) * P, Nx) + cell * P + j;          // below 2 N_x + P
        xo -= xo >= Nx ? Nx : 0;
        xo -= xo >= Nx ? Nx : 0;
    }
    const bool own = gl < lay.tyg && xl < (whole ? Nx : ncx * P);
    const int b0 = own ? gl * lay.cx + cell * P : 0;
    const int bl = own && whole && cell + 1 == g.nel[0] ? gl * lay.cx : b0 + P;
    S xw[P + 1];
#pragma unroll
    for (int r = 0; r <= P; ++r) xw[r] = Wx[row * (P + 1) + r];
#pragma unroll
    for (int j = 0; j < P; ++j) {
        S w[P + 1];
#pragma unroll
        for (int m = 0; m <= P; ++m) w[m] = Wy[(lsy + j) % P * (P + 1) + m];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            S a = w[0] * v[k * P];
#pragma unroll
            for (int m = 1; m <= P; ++m) a = fma(w[m], v[k * P + m], a);
            buf[k * P + j][tid] = a;
        }
    }
    __syncthreads();
    int y = wrapi((ty * lay.tyg * NC - omy - 1) * P, Ny) + gl * NC * P + lsy;   // first output row
    y -= y >= Ny ? Ny : 0;
    y -= y >= Ny ? Ny : 0;
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        if (!own || c0 + k >= g.nel[1]) break;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const S *b = buf[k * P + j];
            S a = 0;
#pragma unroll
            for (int r = 0; r < P; ++r) a = fma(xw[r], b[b0 + r], a);
            a = fma(xw[P], b[bl], a);
            store_at<false, S>(dst, plane_offset<S>(y * Nx + xo), a);
            y = y + 1 == Ny ? 0 : y + 1;
        }
    }
}

namespace {

template <typename S, int P>
hipError_t launch_y(const Geometry &g, const CellTables<S> &t, const YLayout &lay, const S *in, S *out, hipStream_t st)
{
    if (lay.blocks == 0) return hipErrorInvalidValue;
    if (lay.nc == 1)
        hipLaunchKernelGGL((k_stream_y<S, P, 1>), dim3(lay.blocks, 2 * Q2D), dim3(lay.nt), 0, st, g, t, in, out, lay);
    else
        hipLaunchKernelGGL((k_stream_y<S, P, y_cells(P)>), dim3(lay.blocks, 2 * Q2D), dim3(lay.nt), 0, st, g, t, in, out,
                           lay);
    return hipGetLastError();
}

}  // namespace

template <typename S>
hipError_t launch_stream_2d(const Geometry &g, const CellTables<S> &t, const YLayout &lay, const S *in, S *out,
                            hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_y<S, 1>(g, t, lay, in, out, st);
    case 2: return launch_y<S, 2>(g, t, lay, in, out, st);
    case 3: return launch_y<S, 3>(g, t, lay, in, out, st);
    case 4: return launch_y<S, 4>(g, t, lay, in, out, st);
    case 5: return launch_y<S, 5>(g, t, lay, in, out, st);
    case 6: return launch_y<S, 6>(g, t, lay, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_2d<double>(const Geometry &, const CellTables<double> &, const YLayout &,
                                             const double *, double *, hipStream_t);
template hipError_t launch_stream_2d<float>(const Geometry &, const CellTables<float> &, const YLayout &,
                                             const float *, float *, hipStream_t);

}  // namespace sllbm
