// Semi-Lagrangian streaming (Sec. II A, Eqs. (8)-(9)) by source cell, and its
// transpose.
//
// For velocity i the interpolant factorises into three 1-D operators, and
// along an axis output node e*P + l reads source cell e + o_l, o_l = omin for
// l < lstar and omin + 1 otherwise.  The outputs that read source cell c thus
// form a group of P consecutive nodes, (c - omin - 1)*P + lstar + j, j =
// 0 .. P-1, read with weight row (lstar + j) mod P: each source cell of
// (P + 1)^3 nodes (faces shared with its neighbours) maps to P^3 outputs of
// its own, whatever the shift, and there is no halo beyond the shared faces.
// A lane takes one column (x) of a source cell: it loads the P + 1 nodes along
// y of each z-row, interpolates along y and z in registers with the
// velocity's uniform weights, and leaves P x P values in LDS, from which the
// block's lanes interpolate along x, one output column each.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "layouts.h"
#include "rows.h"
#include "sllbm_internal.h"
#include "xcd.h"

namespace sllbm {

template <typename S, int P, int NT>
constexpr int z_min_waves()
{
    if (NT > 512) return P == 4 && sizeof(S) == 8 ? NT / 256 : 4;      // (LDS for one block)
    return sizeof(S) == 4 ? (P <= 4 ? 5 : P == 5 ? 4 : 3) : (P <= 3 ? 5 : P == 4 ? 4 : P == 5 ? 3 : 2);
}

// Streaming, by source cell.  Bound by HBM: every value is read from it once
// (the (P+1)/P-fold y and z faces come from L1 and L2) and written once.  At
// 256^3 nodes, P = 4: 4.11 ms in FP64 and 2.07 ms in FP32 (5.9 and 5.8 TB/s,
// the rate of a copy); 64^3 71 / 29 us, 24^3 (P = 3) 7.0 us, 100^3 nodes
// at P = 5 294 us.  The march by 32 x 8 and 32 x 16 output tiles that this
// replaces read a window of P + 1 more rows and columns per tile out of LDS
// and took 5.2 / 2.9 ms, 89 / 47 us, 11.4 us and 668 us.  At order 6 in FP64 the uniform
// weights exceed the scalar registers (76 spilled into lanes of vector registers).
// NTH: non-temporal output stores (states larger than the Infinity Cache)
template <typename S, int P, bool NTH, int NT>
__global__ void __launch_bounds__(NT, (z_min_waves<S, P, NT>()))
    k_stream_z(Geometry g, CellTables<S> tab, const S *__restrict__ in, S *__restrict__ out, ZLayout lay)
{
    __shared__ S buf[P * P][NT];                           // y-z-interpolated values of a source cell, per lane
    const int tid = threadIdx.x;
    const int ntiles = lay.ntx * lay.nty;
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                                static_cast<int>(gridDim.x * gridDim.y)));
    const int q = L / (ntiles * lay.nchunk);
    const int rem = L - q * ntiles * lay.nchunk;
    const int chunk = rem / ntiles, tile = rem - chunk * ntiles;
    const int ty = tile / lay.ntx, tx = tile - ty * lay.ntx;
    const int i = q >> 1, pop = q & 1;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int64_t N = g.nodes, NP = static_cast<int64_t>(Nx) * Ny;
    const int omx = tab.omin[i * 3 + 0], omy = tab.omin[i * 3 + 1], omz = tab.omin[i * 3 + 2];
    const int lsx = tab.lstar[i * 3 + 0], lsy = tab.lstar[i * 3 + 1], lsz = tab.lstar[i * 3 + 2];
    const S *Wx = tab.w + (i * 3 + 0) * P * (P + 1);
    const S *Wy = tab.w + (i * 3 + 1) * P * (P + 1);
    const S *Wz = tab.w + (i * 3 + 2) * P * (P + 1);
    S *src = const_cast<S *>(in) + static_cast<int64_t>(pop * 45 + i) * N;
    S *dst = out + static_cast<int64_t>(pop * 45 + i) * N;

    // this lane's source column: cell cy along y, node column x.  Lanes without
    // an output of their own repeat lane 0, store included (the same value):
    // stores under a branch would make every later wait for a load a wait for
    // them.
    const int cx0 = tx * lay.txc, cy0 = ty * lay.tyc;
    // exact quotient: (tid + 1/2) / cx lies at least 1 / (2 cx) from an integer
    int cyl = static_cast<int>((static_cast<float>(tid) + 0.5f) * lay.rcx), xl = tid - cyl * lay.cx;
    const int ncx = min(lay.txc, g.nel[0] - cx0);          // cells of this tile along x
    const bool whole = lay.ntx == 1;
    const bool used = cyl < min(lay.tyc, g.nel[1] - cy0) && (whole || xl <= ncx * P);
    cyl = used ? cyl : 0;
    xl = used ? xl : 0;
    const int cy = cy0 + cyl;
    int xs = cx0 * P + xl;
    xs -= xs >= Nx ? Nx : 0;
    const uint32_t lo = plane_offset<S>(cy * P * Nx + xs);            // the cell's first row and last row
    const uint32_t le = plane_offset<S>((cy + 1 == g.nel[1] ? 0 : cy + 1) * P * Nx + xs);

    // this lane's output column and its taps in the block's row of columns
    int xo, cell;                                          // output x; source cell (of the row, or of the tile)
    S xw[P + 1];
    {
        int row;
        if (whole) {
            xo = xl;
            row = xl % P;
            cell = xl / P + wrapi(omx, g.nel[0]) + (row >= lsx ? 1 : 0);
            cell -= cell >= g.nel[0] ? g.nel[0] : 0;
            cell -= cell >= g.nel[0] ? g.nel[0] : 0;
        } else {
            cell = xl < ncx * P ? xl / P : 0;
            const int j = lsx + xl % P;
            row = j % P;
            xo = wrapi((cx0 - omx - 1) * P, Nx) + cell * P + j;     // below 2 N_x + P
            xo -= xo >= Nx ? Nx : 0;
            xo -= xo >= Nx ? Nx : 0;
        }
#pragma unroll
        for (int r = 0; r <= P; ++r) xw[r] = Wx[row * (P + 1) + r];
    }
    const int b0 = cyl * lay.cx + cell * P;                // first tap; the last one wraps in a whole row
    const int bl = whole && cell + 1 == g.nel[0] ? cyl * lay.cx : b0 + P;
    // output rows of source cell cy along y: (cy - omy - 1) P + lsy + j
    uint32_t oo[P];
    {
        int y0 = wrapi((cy0 - omy - 1) * P, Ny) + cyl * P + lsy;    // below 2 N_y + P
        y0 -= y0 >= Ny ? Ny : 0;
        y0 -= y0 >= Ny ? Ny : 0;
#pragma unroll
        for (int j = 0; j < P; ++j) oo[j] = plane_offset<S>((y0 + j - (y0 + j >= Ny ? Ny : 0)) * Nx + xo);
    }
    S wy[P][P + 1];                                        // uniform weights: output j reads with row (lsy + j) mod P
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int r = 0; r <= P; ++r) wy[j][r] = Wy[((lsy + j) % P) * (P + 1) + r];
    // z weights: from order 4 on they are fetched for each row through the
    // scalar cache (beside wy they exceed the scalar registers)
    using CS = const __attribute__((address_space(4))) S;
    CS *wzp = (CS *)Wz;
    int wzo[P];
#pragma unroll
    for (int l = 0; l < P; ++l) wzo[l] = (lsz + l) % P * (P + 1);
    auto zweights = [&](int r, S (&w)[P]) {
        if constexpr (P >= 4) asm volatile("" : "+s"(wzp));
#pragma unroll
        for (int l = 0; l < P; ++l) w[l] = wzp[wzo[l] + r];
    };

    const int zc0 = chunk * lay.zcells, zc1 = min(g.nel[2], zc0 + lay.zcells);
    auto load_row = [&](S (&v)[P + 1], int z) {
        const int64_t zo = static_cast<int64_t>(z >= Nz ? z - Nz : z) * NP;
#pragma unroll
        for (int m = 0; m < P; ++m) v[m] = load_at<S>(plane_row(src, zo + static_cast<int64_t>(m) * Nx), lo);
        v[P] = load_at<S>(plane_row(src, zo), le);
    };
    S Y[P], acc[P][P];
    auto interp_y = [&](const S (&v)[P + 1]) {
#pragma unroll
        for (int j = 0; j < P; ++j) {
            Y[j] = wy[j][0] * v[0];
#pragma unroll
            for (int m = 1; m <= P; ++m) Y[j] = fma(wy[j][m], v[m], Y[j]);
        }
    };
    auto first_row = [&] {                                 // acc of a cell from its first row
        S w[P];
        zweights(0, w);
#pragma unroll
        for (int l = 0; l < P; ++l)
#pragma unroll
            for (int j = 0; j < P; ++j) acc[l][j] = w[l] * Y[j];
    };
    S raw[P][P + 1];                                       // rows 1 .. P of the next cell, in flight
    {
        S v0[P + 1];
        load_row(v0, zc0 * P);
#pragma unroll
        for (int r = 0; r < P; ++r) load_row(raw[r], zc0 * P + 1 + r);
        interp_y(v0);
        first_row();
    }
    auto cell_step = [&](auto last, int c) {
#pragma unroll
        for (int r = 0; r < P; ++r) {
            S w[P];
            zweights(r + 1, w);
            interp_y(raw[r]);
            if constexpr (!decltype(last)::value) load_row(raw[r], (c + 1) * P + 1 + r);
#pragma unroll
            for (int l = 0; l < P; ++l)
#pragma unroll
                for (int j = 0; j < P; ++j) acc[l][j] = fma(w[l], Y[j], acc[l][j]);
        }
#pragma unroll
        for (int l = 0; l < P; ++l)
#pragma unroll
            for (int j = 0; j < P; ++j) buf[l * P + j][tid] = acc[l][j];
        if constexpr (!decltype(last)::value) first_row();
        __syncthreads();
        int z = wrapi((c - omz - 1) * P + lsz, Nz);
#pragma unroll
        for (int l = 0; l < P; ++l) {
            const GlobalRow<S> d = plane_row(dst, static_cast<int64_t>(z) * NP);
#pragma unroll
            for (int j = 0; j < P; ++j) {
                const S *b = buf[l * P + j];
                S v = 0;
#pragma unroll
                for (int r = 0; r < P; ++r) v = fma(xw[r], b[b0 + r], v);
                v = fma(xw[P], b[bl], v);
                store_at<NTH, S>(d, oo[j], v);
            }
            __builtin_amdgcn_sched_barrier(0);             // one output row's LDS reads at a time (registers)
            z = z + 1 == Nz ? 0 : z + 1;
        }
    };
    // the first cell outside the loop: entered from it, the loop's waits for a
    // row need not assume that no stores are in flight after the row's loads
    int c = zc0;
    if constexpr (z_max_cells(P) > 1) {
        if (c < zc1 - 1) {
            cell_step(std::false_type(), c);
            __syncthreads();
            for (++c; c < zc1 - 1; ++c) {
                cell_step(std::false_type(), c);
                __syncthreads();
            }
        }
    }
    cell_step(std::true_type(), c);
}

// NT: LDS columns of a block (z_columns), the fewest that hold its threads.
// A block of one wave that kept 256 columns left a CU five waves at order 4 in FP64
// (32 x 52 x 40 nodes: forward 24.9 us, transposed 34.3 us; 16.8 and 21.1 with its own
// LDS).  Strides known only at run time cost the transposed kernel registers (128^3
// FP32 299 -> 348 us).
template <int P, class Launch>
static hipError_t launch_columns(const ZLayout &lay, Launch &&launch)
{
    if (lay.blocks == 0) return hipErrorInvalidValue;
    switch (z_columns(lay.nt)) {
    case 64: launch(std::integral_constant<int, 64>()); break;
    case 128: launch(std::integral_constant<int, 128>()); break;
    case 256: launch(std::integral_constant<int, 256>()); break;
    default:
        if constexpr (z_row(P) > ZNT) {
            switch (z_columns(lay.nt)) {
            case 384: launch(std::integral_constant<int, 384>()); break;
            case 512: launch(std::integral_constant<int, 512>()); break;
            case 768: launch(std::integral_constant<int, 768>()); break;
            default: launch(std::integral_constant<int, 1024>());
            }
        } else {
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

template <typename S, int P>
static hipError_t launch_z(const Geometry &g, const CellTables<S> &t, const ZLayout &lay, const S *in, S *out,
                           hipStream_t st)
{
    return launch_columns<P>(lay, [&](auto c) {
        constexpr int NT = decltype(c)::value;
        if (NT > 512 || lay.nontemporal)                   // (such rows are whole lines of large states)
            hipLaunchKernelGGL((k_stream_z<S, P, true, NT>), dim3(lay.blocks, 90), dim3(lay.nt), 0, st, g, t, in, out, lay);
        else if constexpr (NT <= 512)
            hipLaunchKernelGGL((k_stream_z<S, P, false, NT>), dim3(lay.blocks, 90), dim3(lay.nt), 0, st, g, t, in, out, lay);
    });
}

// ---------------------------------------------------------------------------
// Transposed streaming S^T (the adjoint of Eqs. (8)-(9)), by output cell.
//
// Transposing the group rule above, node k of cell c receives
//   T[c*P + k] = sum_j W[(lstar + j) mod P][k] lam[group(c)_j]
// and node 0 also, as point P of cell c - 1,
//   + sum_j W[(lstar + j) mod P][P] lam[group(c - 1)_j],
// so a cell gathers two consecutive groups (2P inputs, starting at
// (c - omin - 2)*P + lstar) with the forward weights; this holds for any
// number of cells, wrap-around included.  A lane takes one input column of a
// cell along y, loads both groups of each z-row, gathers along y and z in
// registers and x through LDS, like the forward kernel.  Along z it marches:
// what a group adds to the next cell's node 0 stays in registers, and only a
// block's first cell reads its preceding group again.
// ---------------------------------------------------------------------------

// Rows in flight ahead of the one being processed (divides P), as registers
// allow: P = 4 in FP32 at 128^3 nodes 301, 299 and 290 us with 1, 2 and 4 rows,
// in FP64 (four rows spill) 611, 627 and 873 us; P = 6 in FP64, 96^3 nodes, 368 and
// 346 us with 1 and 2.
template <typename S, int P>
constexpr int zt_depth()
{
    return P <= 3 || (P == 4 && sizeof(S) == 4) ? P : P == 6 ? 2 : 1;
}

template <typename S, int P, int NT>
constexpr int zt_min_waves()
{
    if (NT > 512) return P == 4 && sizeof(S) == 8 ? NT / 256 : 4;      // (LDS for one block)
    return sizeof(S) == 4 ? (P <= 4 ? 5 : P == 5 ? 4 : 3) : (P <= 3 ? 5 : P == 4 ? 4 : P == 5 ? 3 : 2);
}

// Bound by HBM, behind it the reads of both groups from L1 and L2 (each value
// 2.2 to 2.5 times).  At 128^3 nodes, P = 4: 290 us in FP32 and 611 us in FP64 (5.2 and
// 4.9 TB/s), 256^3 2.3 / 4.5 ms, 24^3 (P = 3) 8.0 us, 96^3 at P = 6 346 us; the
// march by output tiles before it, with the windows in LDS, took 362 / 646 us,
// 2.83 / 5.17 ms, 11.4 us and 632 us.  Skipping the second group's LDS reads on lanes
// that are no node 0 (a branch) is 2 % slower to 2 % faster.  In FP64 the uniform weights
// of orders 4, 5 and 6 spill 6, 52 and 202 scalar registers into lanes of vector
// registers, in FP32 those of order 6 spill 26.  On a single cell (216 nodes, p = 6) the
// chain of its one wave per plane takes 10.7 us in FP64 and 8.6 in FP32, against 8.8 and
// 6.9 of the march; all its rows in flight at once do not shorten it.
// NTH: non-temporal output stores (states larger than the Infinity Cache)
template <typename S, int P, bool NTH, int NT>
__global__ void __launch_bounds__(NT, (zt_min_waves<S, P, NT>()))
    k_stream_zt(Geometry g, CellTables<S> tab, const S *__restrict__ in, S *__restrict__ out, ZLayout lay)
{
    constexpr int D = zt_depth<S, P>();
    __shared__ S buf[P * P][NT];                           // y-z-gathered values of an output cell, per lane
    const int tid = threadIdx.x;
    const int ntiles = lay.ntx * lay.nty;
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                                static_cast<int>(gridDim.x * gridDim.y)));
    const int q = L / (ntiles * lay.nchunk);
    const int rem = L - q * ntiles * lay.nchunk;
    const int chunk = rem / ntiles, tile = rem - chunk * ntiles;
    const int ty = tile / lay.ntx, tx = tile - ty * lay.ntx;
    const int i = q >> 1, pop = q & 1;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int64_t N = g.nodes, NP = static_cast<int64_t>(Nx) * Ny;
    const int omx = tab.omin[i * 3 + 0], omy = tab.omin[i * 3 + 1], omz = tab.omin[i * 3 + 2];
    const int lsx = tab.lstar[i * 3 + 0], lsy = tab.lstar[i * 3 + 1], lsz = tab.lstar[i * 3 + 2];
    using CS = const __attribute__((address_space(4))) S;
    const S *Wx = tab.w + (i * 3 + 0) * P * (P + 1);
    CS *Wy = (CS *)(tab.w + (i * 3 + 1) * P * (P + 1));
    CS *Wz = (CS *)(tab.w + (i * 3 + 2) * P * (P + 1));
    S *src = const_cast<S *>(in) + static_cast<int64_t>(pop * 45 + i) * N;
    S *dst = out + static_cast<int64_t>(pop * 45 + i) * N;

    // this lane's input column and output cell along y (surplus lanes repeat
    // lane 0, as in the forward kernel); columns are counted in group order, so
    // that column e P + j of a row is input j of the group of cell e
    const int cx0 = tx * lay.txc, cy0 = ty * lay.tyc;
    int cyl = static_cast<int>((static_cast<float>(tid) + 0.5f) * lay.rcx), xl = tid - cyl * lay.cx;
    const bool whole = lay.ntx == 1;
    const int ncx = min(lay.txc, g.nel[0] - cx0);
    const bool used = cyl < min(lay.tyc, g.nel[1] - cy0) && (whole || xl < (ncx + 1) * P);
    cyl = used ? cyl : 0;
    xl = used ? xl : 0;
    int xi = wrapi((cx0 - omx - (whole ? 1 : 2)) * P + lsx, Nx) + xl;   // a split row starts one group early
    xi -= xi >= Nx ? Nx : 0;
    // rows 0 .. 2P-1: the groups of cells cy - 1 and cy along y
    uint32_t io[2 * P];
    {
        int y0 = wrapi((cy0 - omy - 2) * P + lsy, Ny) + cyl * P;       // below 2 N_y
        y0 -= y0 >= Ny ? Ny : 0;
#pragma unroll
        for (int r = 0; r < 2 * P; ++r) {
            int y = y0 + r;
            y -= y >= Ny ? Ny : 0;
            y -= y >= Ny ? Ny : 0;                         // one cell along y: N_y = P
            io[r] = plane_offset<S>(y * Nx + xi);
        }
    }
    const int xe = whole || xl >= P ? xl : xl + P;         // the output column, counted like the input columns
    const int cell = xe / P, kx = xe - cell * P;
    const int b0 = cyl * lay.cx + cell * P;
    const int bp = cell == 0 ? cyl * lay.cx + Nx - P : b0 - P;         // cell 0: of a whole row only
    const uint32_t oo = plane_offset<S>((cy0 + cyl) * P * Nx + (whole ? xe : cx0 * P + xe - P));
    S xw[P];
#pragma unroll
    for (int j = 0; j < P; ++j) xw[j] = Wx[(lsx + j) % P * (P + 1) + kx];
    auto xp = [&](int j) { return ((CS *)Wx)[(lsx + j) % P * (P + 1) + P]; };   // (uniform)
    S wy[P][P + 1];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int k = 0; k <= P; ++k) wy[j][k] = Wy[(lsy + j) % P * (P + 1) + k];

    // input rows in march order from the group of cell zc0 - 1 on
    const int zc0 = chunk * lay.zcells, zc1 = min(g.nel[2], zc0 + lay.zcells);
    const int zb = wrapi((zc0 - omz - 2) * P + lsz, Nz);
    S raw[D][2 * P];
    auto load_row = [&](S (&v)[2 * P], int k) {            // k < N_z + P
        int z = zb + k;
        z -= z >= Nz ? Nz : 0;
        z -= z >= Nz ? Nz : 0;
        const GlobalRow<S> row = plane_row(src, static_cast<int64_t>(z) * NP);
#pragma unroll
        for (int r = 0; r < 2 * P; ++r) v[r] = load_at<S>(row, io[r]);
    };
    S Y[P], acc[P][P], carry[P];
    auto gather_y = [&](const S (&v)[2 * P]) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            Y[k] = wy[0][k] * v[P];
#pragma unroll
            for (int j = 1; j < P; ++j) Y[k] = fma(wy[j][k], v[P + j], Y[k]);
        }
#pragma unroll
        for (int j = 0; j < P; ++j) Y[0] = fma(wy[j][P], v[j], Y[0]);
    };
    // weights of row j of a group for the points k of its cell
    int wzo[P];
#pragma unroll
    for (int j = 0; j < P; ++j) wzo[j] = (lsz + j) % P * (P + 1);
    auto zweights = [&](int j, S (&w)[P + 1]) {
        if constexpr (P >= 4) asm volatile("" : "+s"(Wz));
#pragma unroll
        for (int k = 0; k <= P; ++k) w[k] = Wz[wzo[j] + k];
    };

#pragma unroll
    for (int j = 0; j < D; ++j) load_row(raw[j], j);
#pragma unroll
    for (int j = 0; j < P; ++j) {
        S w[P + 1];
        zweights(j, w);
        gather_y(raw[j % D]);
        load_row(raw[j % D], j + D);
#pragma unroll
        for (int m = 0; m < P; ++m) carry[m] = j == 0 ? w[P] * Y[m] : fma(w[P], Y[m], carry[m]);
        __builtin_amdgcn_sched_barrier(0);
    }
    auto cell_step = [&](auto last, int c) {
        constexpr bool LAST = decltype(last)::value;
        const int k0 = (c - zc0 + 1) * P;
#pragma unroll
        for (int j = 0; j < P; ++j) {
            S w[P + 1];
            zweights(j, w);
            gather_y(raw[j % D]);
            if (!LAST || j + D < P) load_row(raw[j % D], k0 + j + D);
            if (j == 0) {
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    acc[0][m] = fma(w[0], Y[m], carry[m]);
#pragma unroll
                    for (int k = 1; k < P; ++k) acc[k][m] = w[k] * Y[m];
                    carry[m] = w[P] * Y[m];
                }
            } else {
#pragma unroll
                for (int m = 0; m < P; ++m) {
#pragma unroll
                    for (int k = 0; k < P; ++k) acc[k][m] = fma(w[k], Y[m], acc[k][m]);
                    carry[m] = fma(w[P], Y[m], carry[m]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);             // D rows of loads in flight and no more (registers)
        }
#pragma unroll
        for (int k = 0; k < P; ++k)
#pragma unroll
            for (int m = 0; m < P; ++m) buf[k * P + m][tid] = acc[k][m];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < P; ++k) {
            int t0 = b0, tp = bp;
            asm volatile("" : "+v"(t0), "+v"(tp));         // LDS addresses formed here, not kept across the loop
#pragma unroll
            for (int m = 0; m < P; ++m) {
                const S *b = buf[k * P + m];
                S v = xw[0] * b[t0], e = xp(0) * b[tp];
#pragma unroll
                for (int j = 1; j < P; ++j) {
                    v = fma(xw[j], b[t0 + j], v);
                    e = fma(xp(j), b[tp + j], e);
                }
                store_at<NTH, S>(plane_row(dst, static_cast<int64_t>(c * P + k) * NP + static_cast<int64_t>(m) * Nx), oo,
                                 kx == 0 ? v + e : v);
            }
            __builtin_amdgcn_sched_barrier(0);             // one output row's LDS reads at a time (registers)
        }
    };
    // the first cell outside the loop, as in the forward kernel
    int c = zc0;
    if (c < zc1 - 1) {
        cell_step(std::false_type(), c);
        __syncthreads();
        for (++c; c < zc1 - 1; ++c) {
            cell_step(std::false_type(), c);
            __syncthreads();
        }
    }
    cell_step(std::true_type(), c);
}

template <typename S, int P>
static hipError_t launch_zt(const Geometry &g, const CellTables<S> &t, const ZLayout &lay, const S *in, S *out,
                           hipStream_t st)
{
    return launch_columns<P>(lay, [&](auto c) {
        constexpr int NT = decltype(c)::value;
        if (NT > 512 || lay.nontemporal)                   // (such rows are whole lines of large states)
            hipLaunchKernelGGL((k_stream_zt<S, P, true, NT>), dim3(lay.blocks, 90), dim3(lay.nt), 0, st, g, t, in, out, lay);
        else if constexpr (NT <= 512)
            hipLaunchKernelGGL((k_stream_zt<S, P, false, NT>), dim3(lay.blocks, 90), dim3(lay.nt), 0, st, g, t, in, out, lay);
    });
}

template <typename S>
hipError_t launch_stream_zt(const Geometry &g, const CellTables<S> &t, const ZLayout &lay, const S *in, S *out,
                           hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_zt<S, 1>(g, t, lay, in, out, st);
    case 2: return launch_zt<S, 2>(g, t, lay, in, out, st);
    case 3: return launch_zt<S, 3>(g, t, lay, in, out, st);
    case 4: return launch_zt<S, 4>(g, t, lay, in, out, st);
    case 5: return launch_zt<S, 5>(g, t, lay, in, out, st);
    case 6: return launch_zt<S, 6>(g, t, lay, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_zt<double>(const Geometry &, const CellTables<double> &, const ZLayout &, const double *,
                                           double *, hipStream_t);
template hipError_t launch_stream_zt<float>(const Geometry &, const CellTables<float> &, const ZLayout &, const float *,
                                           float *, hipStream_t);

template <typename S>
hipError_t launch_stream_z(const Geometry &g, const CellTables<S> &t, const ZLayout &lay, const S *in, S *out,
                           hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_z<S, 1>(g, t, lay, in, out, st);
    case 2: return launch_z<S, 2>(g, t, lay, in, out, st);
    case 3: return launch_z<S, 3>(g, t, lay, in, out, st);
    case 4: return launch_z<S, 4>(g, t, lay, in, out, st);
    case 5: return launch_z<S, 5>(g, t, lay, in, out, st);
    case 6: return launch_z<S, 6>(g, t, lay, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_z<double>(const Geometry &, const CellTables<double> &, const ZLayout &, const double *,
                                           double *, hipStream_t);
template hipError_t launch_stream_z<float>(const Geometry &, const CellTables<float> &, const ZLayout &, const float *,
                                           float *, hipStream_t);

}  // namespace sllbm
