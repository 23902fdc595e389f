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

#include <algorithm>
#include <type_traits>

#include "nt.h"
#include "sllbm_internal.h"
#include "xcd.h"

namespace sllbm {

namespace {

__device__ __forceinline__ int wrapi(int x, int n)
{
    int r = x % n;
    return r < 0 ? r + n : r;
}

// How an x-y plane is dealt to blocks and lanes.  A block holds tyc cells
// along y and cx columns of each.  While x rows fit a block (N_x <= ZNT),
// cx = N_x: the periodic row is complete and lane x writes output column x.
// Longer rows are split into tiles of txc cells; a tile has halo columns more
// than it writes (forward: the last cell's far face; transposed: the group
// before the tile).
struct ZLayout {
    int cx, txc, tyc, ntx, nty, nt;   // nt: threads per block
    float rcx;                        // 1 / cx
    int zcells, nchunk;               // cells along z per block, blocks along z
};

constexpr int ZNT = 256;              // most threads per block

// the split with the fewest idle lanes
ZLayout z_layout(const Geometry &g, int halo)
{
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
                b = ZLayout{cx, txc, tyc, ntx, nty, nt, 1.0f / static_cast<float>(cx), 0, 0};
            }
        }
    }
    return b;
}

// Cells along z per block: at most max_cells, fewer while the grid has fewer
// than Z_TARGET_BLOCKS blocks of 256 threads.
constexpr int Z_TARGET_BLOCKS = 1024;

// nblocks: blocks per plane (the grid is nblocks x 90: with one dimension its
// threads would pass 2^32 on the largest grids)
bool z_split(const Geometry &g, int max_cells, ZLayout &b, unsigned &nblocks)
{
    const int64_t tiles = static_cast<int64_t>(b.ntx) * b.nty;
    const int64_t want = (static_cast<int64_t>(Z_TARGET_BLOCKS) * ZNT / b.nt + 90 * tiles - 1) / (90 * tiles);
    const int n = std::max(static_cast<int>(std::min<int64_t>(g.nel[2], want)), (g.nel[2] + max_cells - 1) / max_cells);
    b.zcells = (g.nel[2] + n - 1) / n;
    b.nchunk = (g.nel[2] + b.zcells - 1) / b.zcells;
    nblocks = static_cast<unsigned>(tiles * b.nchunk);
    return 90 * tiles * b.nchunk <= (int64_t(1) << 31) - 1;
}

}  // namespace

// Byte offset of a node in an x-y plane: 32 bits suffice (the 90 planes of a
// state whose x-y plane had 4 GB would not fit the card), so that an access is
// a uniform row address plus one register per lane.
template <typename S>
__device__ __forceinline__ uint32_t plane_offset(int node)
{
    return static_cast<uint32_t>(node) * static_cast<uint32_t>(sizeof(S));
}
// A row of a plane as the compiler must see it, a uniform address that it does
// not know: otherwise it keeps plane address + offset, 64 bits per lane and
// access, across the loop.
template <typename S>
using GlobalRow = __attribute__((address_space(1))) S *;
template <typename S>
__device__ __forceinline__ GlobalRow<S> plane_row(S *base, int64_t node)
{
    GlobalRow<S> r = (GlobalRow<S>)(base + node);
    asm volatile("" : "+s"(r));
    return r;
}
template <typename S>
__device__ __forceinline__ S load_at(GlobalRow<S> row, uint32_t off)
{
    return *(GlobalRow<S>)((__attribute__((address_space(1))) char *)row + off);
}
template <bool NTH, typename S>
__device__ __forceinline__ void store_at(GlobalRow<S> row, uint32_t off, S v)
{
    GlobalRow<S> p = (GlobalRow<S>)((__attribute__((address_space(1))) char *)row + off);
    if constexpr (NTH) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Cells along z per block of the forward kernel.  One source cell from order 3
// on: every load of a block is then in flight at once, and the blocks of an
// XCD cover a thin slab whose shared faces meet in its L2 (256^3 nodes, P = 4,
// FP64: 4.11 ms; marching 4, 16 or 64 cells with the next cell's rows in
// flight 4.28, 4.38 and 4.79 ms).  Cells of order 1 and 2 are too small for
// that and are marched (48 x 40 x 40 nodes, P = 2: 17.8 us with two cells, 20.8
// with one; 100 x 100 x 30, P = 1, FP32: 51 us with 30, 214 with one).
template <int P>
constexpr int z_max_cells()
{
    return P >= 3 ? 1 : P == 2 ? 2 : 32;
}

template <typename S, int P>
constexpr int z_min_waves()
{
    return sizeof(S) == 4 ? (P <= 4 ? 5 : P == 5 ? 4 : 3) : (P <= 3 ? 5 : P == 4 ? 4 : P == 5 ? 3 : 2);
}

// Streaming, by source cell.  Bound by HBM: every value is read from it once
// (the (P+1)/P-fold y and z faces come from L1 and L2) and written once.  At
// 256^3 nodes, P = 4: 4.11 ms in FP64 and 2.07 ms in FP32 (5.9 and 5.8 TB/s,
// the rate of a copy); 64^3 71 / 29 us, 24^3 (P = 3) 7.0 us, 100^3 nodes
// at P = 5 294 us.  The march by 32 x 8 and 32 x 16 output tiles that this
// replaces read a window of P + 1 more rows and columns per tile out of LDS
// and took 5.2 / 2.9 ms, 89 / 47 us, 11.4 us and 668 us.
// NTH: non-temporal output stores (states larger than the Infinity Cache)
template <typename S, int P, bool NTH>
__global__ void __launch_bounds__(ZNT, (z_min_waves<S, P>())) k_stream_z(Geometry g, CellTables<S> tab,
                                                                        const S *__restrict__ in,
                                                                        S *__restrict__ out, ZLayout lay)
{
    __shared__ S buf[P * P][ZNT];                          // y-z-interpolated values of a source cell, per lane
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
    if constexpr (z_max_cells<P>() > 1) {
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

template <typename S, int P>
static hipError_t launch_z(const Geometry &g, const CellTables<S> &t, const S *in, S *out, hipStream_t st)
{
    ZLayout lay = z_layout(g, 1);
    unsigned nb;
    if (!z_split(g, z_max_cells<P>(), lay, nb)) return hipErrorInvalidValue;
    if (use_nontemporal(90 * g.nodes * static_cast<int64_t>(sizeof(S))))
        hipLaunchKernelGGL((k_stream_z<S, P, true>), dim3(nb, 90), dim3(lay.nt), 0, st, g, t, in, out, lay);
    else
        hipLaunchKernelGGL((k_stream_z<S, P, false>), dim3(nb, 90), dim3(lay.nt), 0, st, g, t, in, out, lay);
    return hipGetLastError();
}

namespace {

constexpr int64_t ZCHUNK_TARGET_BLOCKS = 2048;
constexpr int ZCHUNK_MIN_CELLS = 4;
constexpr int ZCHUNK_MAX_CELL_BYTES = 64;   // cells per chunk times the element size (8 x 32-node tiles)
constexpr int ZCHUNK_MAX_CELLS_LARGE = 32;  // cells per chunk with the 32 x 16-node tiles of large grids

// Number of z-chunks of a march over ntiles x-y tiles and 90 planes.  Small
// grids split the march until the grid has a few blocks per CU slot.  Every
// grid caps a chunk at max_cells cells: blocks of one plane start in
// (chunk, tile) order, so neighbouring tiles march through the same z-rows at
// nearly the same time and more of the x-y halo rows that one tile loads are
// still in L2 when its neighbours read them; blocks that marched the whole
// axis drift apart on large grids.  Each chunk re-reads P + 1 rows.
// Measured at 256^3 nodes (FP64) with 32 x 8-node tiles: reads of 1.87x the
// algorithmic bytes with whole-axis marches, 1.31x with 8-cell chunks (1.59x
// and 1.10x at 128^3), hence ZCHUNK_MAX_CELL_BYTES / elem cells (8 in FP64,
// 16 in FP32).  The 32 x 16-node tiles of large grids have half the x-y halo
// per output, and there 32-cell chunks are 2-4 % faster than 8 or 16 cells.
int z_chunks(const Geometry &g, int ntiles, int max_cells)
{
    int nchunk = 1;
    while (nchunk < g.nel[2] && static_cast<int64_t>(ntiles) * 90 * nchunk < ZCHUNK_TARGET_BLOCKS &&
           g.nel[2] / (2 * nchunk) >= ZCHUNK_MIN_CELLS)
        nchunk *= 2;
    nchunk = std::max(nchunk, (g.nel[2] + max_cells - 1) / max_cells);
    const int zcells = (g.nel[2] + nchunk - 1) / nchunk;
    return (g.nel[2] + zcells - 1) / zcells;
}

template <typename S, int V>
struct VecOf {
    typedef S T __attribute__((ext_vector_type(V)));
};
template <typename S>
struct VecOf<S, 1> {
    typedef S T;
};

template <typename VT>
__device__ __forceinline__ auto vcomp(const VT &v, int c)
{
    if constexpr (std::is_arithmetic_v<VT>) return v;
    else return v[c];
}

}  // namespace

// ---------------------------------------------------------------------------
// Transposed streaming S^T (the adjoint of Eqs. (8)-(9)), same z-march.
//
// Along an axis the forward nodes that read source cell c form a group: the
// nodes (c - omin - 1)*P + lstar + j, j = 0 .. P-1, read it with weight row
// (lstar + j) mod P.  Transposing, node k of cell c receives
//   T[c*P + k] = sum_j W[(lstar + j) mod P][k] lam[group(c)_j]
// and node 0 also, as point P of cell c - 1,
//   + sum_j W[(lstar + j) mod P][P] lam[group(c - 1)_j].
// So each output cell gathers two consecutive groups (2P inputs, starting at
// (c - omin - 2)*P + lstar) with the forward weights; this holds for any
// number of cells, wrap-around included.  The kernel is the forward one with
// that gather along x, y (LDS) and z (a register window of 2P rows sliding by
// one cell).
// ---------------------------------------------------------------------------
template <int P, int V = 1, int YN_ = 8>
struct ZTileT {
    static constexpr int ORDER = P;
    static constexpr int XN = 32, YN = YN_;
    static constexpr int TXC = XN / P > 0 ? XN / P : 1, TYC = YN / P > 0 ? YN / P : 1;
    static constexpr int TX = TXC * P, TY = TYC * P;
    static constexpr int WXC = (TX + P + V - 1 + V - 1) / V;  // loads per window row (V-aligned start)
    static constexpr int WX = WXC * V, WY = TY + P;
    static constexpr int NT = (TX * TY + 63) / 64 * 64;
    static constexpr int LK = (WXC * WY + NT - 1) / NT;
    static constexpr int BS = TX % 2 ? TX : TX + 1;
};

// Tile rows of the transposed march, chosen as in the forward one: 16 on
// grids larger than the Infinity Cache if the LDS stays within 64 KB
template <typename S, class Z>
constexpr size_t zt_lds_bytes()
{
    constexpr int WXO = Z::WX % 2 ? Z::WX : Z::WX + 1;
    return static_cast<size_t>(Z::ORDER) * (static_cast<size_t>(WXO) * Z::WY + Z::WY * Z::BS) * sizeof(S);
}

template <typename S, int P, int V, bool BIG>
constexpr int zt_tile_rows()
{
    return BIG && zt_lds_bytes<S, ZTileT<P, V, 16>>() <= 64 * 1024 ? 16 : 8;
}

template <typename S, int P, int V, bool NTH>
using ZTileTOf = ZTileT<P, V, zt_tile_rows<S, P, V, NTH>()>;

// NTH: non-temporal output stores and the larger tile (states larger than
// the Infinity Cache)
template <typename S, int P, int V, bool NTH>
__global__ void __launch_bounds__((ZTileTOf<S, P, V, NTH>::NT))
    k_stream_zt(Geometry g, CellTables<S> tab, const S *__restrict__ in, S *__restrict__ out, int ntile_x,
                int ntiles, int zcells, int nchunk)
{
    using Z = ZTileTOf<S, P, V, NTH>;
    using VT = typename VecOf<S, V>::T;
    constexpr int TX = Z::TX, TY = Z::TY, WY = Z::WY, NT = Z::NT, LK = Z::LK, BS = Z::BS;
    constexpr int WX = Z::WX % 2 ? Z::WX : Z::WX + 1;      // odd LDS row stride
    constexpr int NLD = Z::WXC * WY;
    __shared__ __align__(16) S pl[P][WX * WY];
    __shared__ S bx[P][WY * BS];

    const int tid = threadIdx.x;
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(blockIdx.x, gridDim.x));
    const int q = L / (ntiles * nchunk);
    const int rem = L - q * ntiles * nchunk;
    const int chunk = rem / ntiles, tile = rem - chunk * ntiles;
    const int i = q >> 1, pop = q & 1;
    const int X0 = (tile % ntile_x) * TX, Y0 = (tile / ntile_x) * TY;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int64_t N = g.nodes, NP = static_cast<int64_t>(Nx) * Ny;
    const int omx = tab.omin[i * 3 + 0], omy = tab.omin[i * 3 + 1], omz = tab.omin[i * 3 + 2];
    const int lsx = tab.lstar[i * 3 + 0], lsy = tab.lstar[i * 3 + 1], lsz = tab.lstar[i * 3 + 2];
    const S *Wx = tab.w + (i * 3 + 0) * P * (P + 1);
    const S *Wy = tab.w + (i * 3 + 1) * P * (P + 1);
    const S *Wz = tab.w + (i * 3 + 2) * P * (P + 1);
    const S *__restrict__ src = in + static_cast<int64_t>(pop * 45 + i) * N;
    S *__restrict__ dst = out + static_cast<int64_t>(pop * 45 + i) * N;

    // input window: x from X0 + (-2 - omx)*P + lsx (rounded down to V: shift sx), y from Y0 + (-2 - omy)*P + lsy
    const int offx = (-2 - omx) * P + lsx;
    const int offxa = offx - ((offx % V) + V) % V, sx = offx - offxa;
    const int offy = (-2 - omy) * P + lsy;
    int loff[LK], soff[LK];                                // HBM and LDS offsets of this thread's loads
#pragma unroll
    for (int k = 0; k < LK; ++k) {
        int e = tid + k * NT;
        e = e < NLD ? e : NLD - 1;
        const int wx = (e % Z::WXC) * V, wy = e / Z::WXC;
        loff[k] = wrapi(Y0 + offy + wy, Ny) * Nx + wrapi(X0 + offxa + wx, Nx);
        soff[k] = wy * WX + wx;
    }
    // x and z weights, the same for every thread: w*[j][k] = W[(ls + j) mod P][k]
    S wxu[P][P + 1], wzu[P][P + 1];
#pragma unroll
    for (int j = 0; j < P; ++j)
#pragma unroll
        for (int k = 0; k <= P; ++k) {
            wxu[j][k] = Wx[((lsx + j) % P) * (P + 1) + k];
            wzu[j][k] = Wz[((lsz + j) % P) * (P + 1) + k];
        }
    // output node (X0 + tx, Y0 + ty): point ky of tile cell cy along y gathers
    // window rows (cy + 1)*P + j with yw[j], and for ky = 0 rows cy*P + j with yp[j]
    const int tx = tid % TX, ty = tid / TX;
    const bool own = tid < TX * TY && X0 + tx < Nx && Y0 + ty < Ny;
    const int cy = ty / P, ky = ty % P;
    const int ybase = cy * P * BS + (tid < TX * TY ? tx : 0);
    S yw[P], yp[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
        yw[j] = Wy[((lsy + j) % P) * (P + 1) + ky];
        yp[j] = ky == 0 ? Wy[((lsy + j) % P) * (P + 1) + P] : S(0);
    }
    const int64_t oxy = static_cast<int64_t>(Y0 + ty) * Nx + (X0 + tx);

    // input rows in march order: z = (ez0 - omz - 2)*P + lsz + k (mod Nz), k = 0 .. P + nel*P - 1
    const int ez0 = chunk * zcells, ez1 = min(g.nel[2], ez0 + zcells);
    // row k < P + (ez1 - ez0) P <= Nz + P and zb < Nz: two conditional
    // subtractions wrap zb + k
    const int zb = wrapi((ez0 - omz - 2) * P + lsz, Nz);
    VT rawA[P][LK], rawB[P][LK];
    auto load_rows = [&](auto &raw, int k0, int nr) {
#pragma unroll
        for (int r = 0; r < P; ++r) {
            if (r < nr) {
                int z = zb + k0 + r;
                z -= z >= Nz ? Nz : 0;
                z -= z >= Nz ? Nz : 0;
                const int64_t zo = static_cast<int64_t>(z) * NP;
#pragma unroll
                for (int j = 0; j < LK; ++j) raw[r][j] = *reinterpret_cast<const VT *>(src + zo + loff[j]);
            }
        }
    };
    // P rows: registers -> LDS, reload with the rows two batches ahead, x-gather, y-gather
    auto batch = [&](auto &raw, int next_k0, int next_nr, S *res) {
#pragma unroll
        for (int r = 0; r < P; ++r)
#pragma unroll
            for (int j = 0; j < LK; ++j)
                if (tid + j * NT < NLD) {
#pragma unroll
                    for (int c = 0; c < V; ++c) pl[r][soff[j] + c] = vcomp(raw[r][j], c);
                }
        if (next_nr > 0) load_rows(raw, next_k0, next_nr);
        __syncthreads();
        // x: task (row, window row, output cell cl) reads groups cl and cl + 1 of the row
        constexpr int XT = P * WY * Z::TXC;
#pragma unroll
        for (int k = 0; k < (XT + NT - 1) / NT; ++k) {
            const int e = tid + k * NT;
            if (e < XT) {
                const int r = e / (WY * Z::TXC), rem2 = e - r * (WY * Z::TXC);
                const int cl = rem2 / WY, wy = rem2 - cl * WY;
                const S *c = &pl[r][wy * WX + sx + cl * P];
                S prev[P], cur[P];
#pragma unroll
                for (int j = 0; j < P; ++j) {
                    prev[j] = c[j];
                    cur[j] = c[P + j];
                }
                S *o = &bx[r][wy * BS + cl * P];
#pragma unroll
                for (int kk = 0; kk < P; ++kk) {
                    S acc = 0;
#pragma unroll
                    for (int j = 0; j < P; ++j) acc = fma(wxu[j][kk], cur[j], acc);
                    if (kk == 0) {
#pragma unroll
                        for (int j = 0; j < P; ++j) acc = fma(wxu[j][P], prev[j], acc);
                    }
                    o[kk] = acc;
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < P; ++r) {
            S acc = 0;
#pragma unroll
            for (int j = 0; j < P; ++j) acc = fma(yw[j], bx[r][ybase + (P + j) * BS], acc);
#pragma unroll
            for (int j = 0; j < P; ++j) acc = fma(yp[j], bx[r][ybase + j * BS], acc);
            res[r] = acc;
        }
    };
    S a[2 * P];
    auto emit = [&](int ez) {
        if (own) {
#pragma unroll
            for (int k = 0; k < P; ++k) {
                S acc = 0;
#pragma unroll
                for (int j = 0; j < P; ++j) acc = fma(wzu[j][k], a[P + j], acc);
                if (k == 0) {
#pragma unroll
                    for (int j = 0; j < P; ++j) acc = fma(wzu[j][P], a[j], acc);
                }
                store_hint<NTH>(&dst[static_cast<int64_t>(ez * P + k) * NP + oxy], acc);
            }
        }
#pragma unroll
        for (int j = 0; j < P; ++j) a[j] = a[P + j];
    };

    const int nel = ez1 - ez0;
    auto rows_of = [&](int e) { return e < nel ? P : 0; };
    load_rows(rawA, 0, P);
    load_rows(rawB, P, rows_of(0));
    batch(rawA, 2 * P, rows_of(1), a);
    for (int e = 0; e < nel; e += 2) {
        batch(rawB, P + (e + 2) * P, rows_of(e + 2), a + P);
        emit(ez0 + e);
        if (e + 1 < nel) {
            batch(rawA, P + (e + 3) * P, rows_of(e + 3), a + P);
            emit(ez0 + e + 1);
        }
    }
}

template <typename S, int P, int V, bool NTH>
static hipError_t launch_ztvn(const Geometry &g, const CellTables<S> &t, const S *in, S *out, hipStream_t st)
{
    using Z = ZTileTOf<S, P, V, NTH>;
    const int ntx = (g.N[0] + Z::TX - 1) / Z::TX, nty = (g.N[1] + Z::TY - 1) / Z::TY;
    const int ntiles = ntx * nty;
    // each chunk re-reads P rows
    const int nchunk = z_chunks(g, ntiles, Z::YN == 16 ? ZCHUNK_MAX_CELLS_LARGE
                                                     : ZCHUNK_MAX_CELL_BYTES / static_cast<int>(sizeof(S)));
    const int zcells = (g.nel[2] + nchunk - 1) / nchunk;
    const int64_t nb = static_cast<int64_t>(ntiles) * 90 * nchunk;
    if (nb > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_stream_zt<S, P, V, NTH>), dim3(static_cast<unsigned>(nb)), dim3(Z::NT), 0, st, g, t, in,
                       out, ntx, ntiles, zcells, nchunk);
    return hipGetLastError();
}

template <typename S, int P, int V>
static hipError_t launch_ztv(const Geometry &g, const CellTables<S> &t, const S *in, S *out, hipStream_t st)
{
    if (use_nontemporal(90 * g.nodes * static_cast<int64_t>(sizeof(S))))
        return launch_ztvn<S, P, V, true>(g, t, in, out, st);
    return launch_ztvn<S, P, V, false>(g, t, in, out, st);
}

// 16-byte window loads need V-aligned window starts: tiles and rows of a
// multiple of V nodes and a 16-byte aligned buffer (the start is rounded down)
template <typename S, int P>
static hipError_t launch_zt(const Geometry &g, const CellTables<S> &t, const S *in, S *out, hipStream_t st)
{
    constexpr int V = 16 / sizeof(S);
    if constexpr (ZTileT<P, V>::TX % V == 0) {
        if ((g.N[0] * sizeof(S)) % 16 == 0 && reinterpret_cast<uintptr_t>(in) % 16 == 0)
            return launch_ztv<S, P, V>(g, t, in, out, st);
    }
    return launch_ztv<S, P, 1>(g, t, in, out, st);
}

template <typename S>
hipError_t launch_stream_zt(const Geometry &g, const CellTables<S> &t, const S *in, S *out, hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_zt<S, 1>(g, t, in, out, st);
    case 2: return launch_zt<S, 2>(g, t, in, out, st);
    case 3: return launch_zt<S, 3>(g, t, in, out, st);
    case 4: return launch_zt<S, 4>(g, t, in, out, st);
    case 5: return launch_zt<S, 5>(g, t, in, out, st);
    case 6: return launch_zt<S, 6>(g, t, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_zt<double>(const Geometry &, const CellTables<double> &, const double *, double *,
                                             hipStream_t);
template hipError_t launch_stream_zt<float>(const Geometry &, const CellTables<float> &, const float *, float *,
                                            hipStream_t);

template <typename S>
hipError_t launch_stream_z(const Geometry &g, const CellTables<S> &t, const S *in, S *out, hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_z<S, 1>(g, t, in, out, st);
    case 2: return launch_z<S, 2>(g, t, in, out, st);
    case 3: return launch_z<S, 3>(g, t, in, out, st);
    case 4: return launch_z<S, 4>(g, t, in, out, st);
    case 5: return launch_z<S, 5>(g, t, in, out, st);
    case 6: return launch_z<S, 6>(g, t, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_z<double>(const Geometry &, const CellTables<double> &, const double *, double *,
                                            hipStream_t);
template hipError_t launch_stream_z<float>(const Geometry &, const CellTables<float> &, const float *, float *,
                                           hipStream_t);

}  // namespace sllbm
