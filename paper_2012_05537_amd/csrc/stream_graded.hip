// Semi-Lagrangian streaming (Sec. II A, Eqs. (8)-(9)) on a graded mesh:
// periodic, axis-aligned cells of unequal width.
//
// The departure point of every node still factorises per axis, but the
// departure cell and the 1-D Lagrange weights now depend on the node, not
// only on its local point: each axis carries per-node tables (first source
// node, p + 1 weights), built once per mesh.  Along an axis the first source
// node is non-decreasing in the output node, so the source window of an x-y
// tile is one contiguous (wrapped) range per axis.
//
// Two kernels, forward and transposed, work by source cell (k_stream_graded_cells);
// what they do not take (graded_by_cell) is marched, in either direction:
// a block owns one (velocity, population) plane over a 32 x 8 x-y tile and a
// range of output z-rows.  It walks the source z-rows in order, two at a
// time: it stores their tile windows (loaded into registers while the
// previous two rows were processed) in LDS, interpolates along x (per-thread
// taps) and then along y, and keeps the results in a per-thread ring of
// source rows, from which each output z-row takes its p + 1 taps.
// Every source row is read once per plane and tile column of the chunk.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "rows.h"
#include "sllbm_internal.h"
#include "xcd.h"

namespace sllbm {

namespace {

constexpr int GTX = 32, GTY = 8, GNT = GTX * GTY;
constexpr int GRB = 2;                         // source z-rows interpolated per batch
constexpr int64_t GRADED_TARGET_BLOCKS = 2048;

}  // namespace

template <typename S, int V>
struct VecG {
    typedef S T __attribute__((ext_vector_type(V)));
};
template <typename S>
struct VecG<S, 1> {
    typedef S T;
};

template <typename S, int K, int LK, int V>
__global__ void __launch_bounds__(GNT) k_stream_graded(Geometry g, NodeTables<S> tab, const S *__restrict__ in,
                                                        S *__restrict__ out, int ntile_x, int ntiles, int zrows,
                                                        int nchunk)
{
    constexpr int RB = GRB;                                // source rows per batch (two barriers each)
    constexpr int RZ = K - 1 + RB;                         // ring of source rows per thread
    constexpr int AS = GTX + 1;                            // odd row stride of the x-pass result
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int wxm = tab.wxm, wym = tab.wym;
    const int WP = wym * wxm, AP = wym * AS;
    S *pl = reinterpret_cast<S *>(smem_raw);               // [RB][wym][wxm] source windows of a batch
    S *A = pl + RB * WP;                                   // [RB][wym][AS] x-interpolated rows
    S *ring = A + RB * AP;                                 // [RZ][GNT]     x-y interpolated source rows

    const int tid = threadIdx.x;
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(blockIdx.x, gridDim.x));
    const int q = L / (ntiles * nchunk);
    const int rem = L - q * ntiles * nchunk;
    const int chunk = rem / ntiles, tile = rem - chunk * ntiles;
    const int i = q >> 1, pop = q & 1;
    const int X0 = (tile % ntile_x) * GTX, Y0 = (tile / ntile_x) * GTY;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int64_t N = g.nodes, NP = static_cast<int64_t>(Nx) * Ny;
    const int32_t *sx = tab.src[0] + static_cast<int64_t>(i) * Nx;
    const int32_t *sy = tab.src[1] + static_cast<int64_t>(i) * Ny;
    const int32_t *sz = tab.src[2] + static_cast<int64_t>(i) * Nz;
    const S *wxt = tab.w[0] + static_cast<int64_t>(i) * Nx * K;
    const S *wyt = tab.w[1] + static_cast<int64_t>(i) * Ny * K;
    const S *wzt = tab.w[2] + static_cast<int64_t>(i) * Nz * K;
    const S *__restrict__ src = in + static_cast<int64_t>(pop * 45 + i) * N;
    S *__restrict__ dst = out + static_cast<int64_t>(pop * 45 + i) * N;

    // source window of the tile (first source nodes are non-decreasing); its
    // x start is rounded down to V nodes (shift sh) for V-wide loads
    using VT = typename VecG<S, V>::T;
    const int xs = sx[X0], wxb = sx[min(X0 + GTX, Nx) - 1] - xs + K;
    const int sh = ((xs % V) + V) % V, xs0 = xs - sh;
    const int wxv = (wxb + sh + V - 1) / V;                // V-wide loads per window row
    const int ys0 = sy[Y0], wyb = sy[min(Y0 + GTY, Ny) - 1] - ys0 + K;
    const int nwin = wxv * wyb;                            // <= LK * GNT (checked by the launcher)
    // this thread's window loads: offset inside a z-plane and in LDS
    int loff[LK], soff[LK];
#pragma unroll
    for (int k = 0; k < LK; ++k) {
        const int e = min(tid + k * GNT, nwin - 1);
        const int wy_ = e / wxv, wx_ = (e - wy_ * wxv) * V;
        loff[k] = wrapi(ys0 + wy_, Ny) * Nx + wrapi(xs0 + wx_, Nx);
        soff[k] = wy_ * wxm + wx_;
    }

    // taps of this thread's output column (clamped on ragged tiles, not stored)
    const int tx = tid % GTX, ty = tid / GTX;
    const bool own = X0 + tx < Nx && Y0 + ty < Ny;
    const int gx = min(X0 + tx, Nx - 1), gy = min(Y0 + ty, Ny - 1);
    const int ox = sx[gx] - xs0, oy = sy[gy] - ys0;        // ox includes the shift sh
    S wx[K], wy[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        wx[k] = wxt[gx * K + k];
        wy[k] = wyt[gy * K + k];
    }
    const int64_t oxy = static_cast<int64_t>(gy) * Nx + gx;

    const int zo0 = chunk * zrows, zo1 = min(Nz, zo0 + zrows);
    const int r0 = sz[zo0];                                // first source row of the chunk (not wrapped)
    // the windows of the next batch of source rows are loaded into registers
    // while the current batch is interpolated
    VT raw[RB][LK];
    auto load_batch = [&](int r) {
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const S *base = src + static_cast<int64_t>(wrapi(r + b, Nz)) * NP;
#pragma unroll
            for (int k = 0; k < LK; ++k) raw[b][k] = *reinterpret_cast<const VT *>(base + loff[k]);
        }
    };
    load_batch(r0);
    int rnext = r0;                                        // first source row not yet in the ring
    for (int zo = zo0; zo < zo1; ++zo) {
        const int s = sz[zo];
        // bring in batches until row s + K - 1 is in the ring; the ring then
        // holds rows s .. s + K - 1 (older rows are no longer needed)
        for (; rnext <= s + K - 1; rnext += RB) {
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int k = 0; k < LK; ++k)
                    if (tid + k * GNT < nwin) *reinterpret_cast<VT *>(&pl[b * WP + soff[k]]) = raw[b][k];
            load_batch(rnext + RB);                        // in bounds (wrapped); unused past the chunk
            __syncthreads();
#pragma unroll
            for (int b = 0; b < RB; ++b)
                for (int wy_ = ty; wy_ < wyb; wy_ += GTY) {
                    S acc = 0;
#pragma unroll
                    for (int k = 0; k < K; ++k) acc = fma(wx[k], pl[b * WP + wy_ * wxm + ox + k], acc);
                    A[b * AP + wy_ * AS + tx] = acc;
                }
            __syncthreads();
#pragma unroll
            for (int b = 0; b < RB; ++b) {
                S acc = 0;
#pragma unroll
                for (int k = 0; k < K; ++k) acc = fma(wy[k], A[b * AP + (oy + k) * AS + tx], acc);
                ring[((rnext + b - r0) % RZ) * GNT + tid] = acc;
            }
        }
        S acc = 0;
#pragma unroll
        for (int k = 0; k < K; ++k)
            acc = fma(wzt[zo * K + k], ring[((s + k - r0) % RZ) * GNT + tid], acc);
        if (own) dst[static_cast<int64_t>(zo) * NP + oxy] = acc;
    }
}

// ---------------------------------------------------------------------------
// The same streaming by source cell.  The departure cell is non-decreasing
// along an axis, so the output nodes that depart into cell c are consecutive,
// first[c] .. first[c + 1] - 1 (not wrapped); there are P of them on average,
// none in some cells.  As on equal cells every source cell maps to outputs of
// its own: a lane takes one column (x) of a source cell, loads its P + 1 nodes
// along y and z once, and a wave, all of whose lanes are in one cell along y,
// walks the cell's outputs along z and y with uniform weights; x follows out of
// LDS, one output column per lane.  N_x <= 256 (a block holds whole rows).
// ---------------------------------------------------------------------------
namespace {

constexpr int GCW = 4;                         // waves per block

template <typename T>
using Uniform = const __attribute__((address_space(4))) T *;

__device__ __forceinline__ int wrap1(int x, int n) { return x >= n ? x - n : x; }

// waves per row of columns, and cells along y per block
__host__ __device__ __forceinline__ int gc_row_waves(int Nx) { return (Nx + 63) / 64; }

}  // namespace

// Forward.  The outputs of one z-row at a time go through LDS ([2][cells along
// y][rows][columns], two buffers in turn, one barrier per z-row).  Bound by HBM at
// 128^3 nodes (P = 4, FP64: 535 us, 5.7 TB/s), on smaller grids and in FP32 by the
// chain of a z-row (uniform weights from the scalar cache, barrier, LDS): 64^3 nodes
// 77 us in FP64 and 44 us in FP32.  The march above interpolates every source row out of
// LDS with per-thread taps: 139 and 84 us.
template <typename S, int P>
__global__ void __launch_bounds__(64 * GCW) k_stream_graded_cells(Geometry g, CellReaders<S> tab, const S *__restrict__ in,
                                                           S *__restrict__ out, int cw, int tyc, int nty, int rows)
{
    constexpr int K = P + 1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    S *lds = reinterpret_cast<S *>(smem_raw);
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                            static_cast<int>(gridDim.x * gridDim.y)));
    const int per = nty * g.nel[2];
    const int q = L / per, rem = L - q * per;
    const int cz = rem / nty, ty = rem - cz * nty;
    const int i = q >> 1, pop = q & 1;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int64_t N = g.nodes, NP = static_cast<int64_t>(Nx) * Ny;
    const Uniform<int32_t> fy = (Uniform<int32_t>)(tab.first[1] + static_cast<int64_t>(i) * (g.nel[1] + 1));
    const Uniform<int32_t> fz = (Uniform<int32_t>)(tab.first[2] + static_cast<int64_t>(i) * (g.nel[2] + 1));
    const int z0 = fz[cz], mz = fz[cz + 1] - z0;
    if (mz == 0) return;                                   // nothing departs into this layer of cells
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cyl = wave / cw, xl = (wave - cyl * cw) * 64 + (threadIdx.x & 63);
    const int cy = min(ty * tyc + cyl, g.nel[1] - 1);
    const bool own = xl < Nx;
    const int xc = own ? xl : Nx - 1;
    const int y0 = fy[cy], my = ty * tyc + cyl < g.nel[1] ? fy[cy + 1] - y0 : 0;
    S *src = const_cast<S *>(in) + static_cast<int64_t>(pop * 45 + i) * N;
    S *dst = out + static_cast<int64_t>(pop * 45 + i) * N;
    const uint32_t xoff = plane_offset<S>(xc);

    S v[K][K];                                             // [z][y]
#pragma unroll
    for (int r = 0; r < K; ++r)
#pragma unroll
        for (int m = 0; m < K; ++m)
            v[r][m] = load_at<S>(plane_row(src, wrap1(cz * P + r, Nz) * NP +
                                                    static_cast<int64_t>(wrap1(cy * P + m, Ny)) * Nx), xoff);
    // taps of output column xc
    S wx[K];
#pragma unroll
    for (int k = 0; k < K; ++k) wx[k] = tab.w[0][(static_cast<int64_t>(i) * Nx + xc) * K + k];
    const int b0 = wrapi(tab.src[0][static_cast<int64_t>(i) * Nx + xc], Nx), bl = wrap1(b0 + P, Nx);
    const Uniform<S> wyt = (Uniform<S>)(tab.w[1] + static_cast<int64_t>(i) * Ny * K);
    const Uniform<S> wzt = (Uniform<S>)(tab.w[2] + static_cast<int64_t>(i) * Nz * K);
    const int cx = cw * 64;
    int yo0 = wrapi(y0, Ny), zo = wrapi(z0, Nz);
    for (int l = 0; l < mz; ++l) {
        S *cell = lds + (static_cast<size_t>(l & 1) * tyc + cyl) * rows * cx;
        S t[K];
        {
            S w[K];
#pragma unroll
            for (int r = 0; r < K; ++r) w[r] = wzt[static_cast<int64_t>(zo) * K + r];
#pragma unroll
            for (int m = 0; m < K; ++m) {
                t[m] = w[0] * v[0][m];
#pragma unroll
                for (int r = 1; r < K; ++r) t[m] = fma(w[r], v[r][m], t[m]);
            }
        }
        int yo = yo0;
        for (int j = 0; j < my; j += 2) {                  // two rows at a time (a surplus one is not used)
            const int yn = wrap1(yo + 1, Ny);
            S a = 0, b = 0;
#pragma unroll
            for (int m = 0; m < K; ++m) {
                a = fma(static_cast<S>(wyt[static_cast<int64_t>(yo) * K + m]), t[m], a);
                b = fma(static_cast<S>(wyt[static_cast<int64_t>(yn) * K + m]), t[m], b);
            }
            cell[j * cx + xl] = a;
            cell[(j + 1) * cx + xl] = b;
            yo = wrap1(yn + 1, Ny);
        }
        __syncthreads();
        yo = yo0;
        for (int j = 0; j < my; j += 2) {
            const S *b = cell + j * cx, *d = b + cx;
            S a = wx[P] * b[bl], e = wx[P] * d[bl];
#pragma unroll
            for (int k = 0; k < P; ++k) {
                a = fma(wx[k], b[b0 + k], a);
                e = fma(wx[k], d[b0 + k], e);
            }
            if (own) store_at<false, S>(plane_row(dst, zo * NP + static_cast<int64_t>(yo) * Nx), xoff, a);
            yo = wrap1(yo + 1, Ny);
            if (own && j + 1 < my) store_at<false, S>(plane_row(dst, zo * NP + static_cast<int64_t>(yo) * Nx), xoff, e);
            yo = wrap1(yo + 1, Ny);
        }
        zo = wrap1(zo + 1, Nz);
    }
}

// Transpose, by output cell: node k of cell c collects from the readers of c
// (group c) with weight w[reader][k], and node 0 also from the readers of cell
// c - 1 with weight w[reader][P].  A lane takes one input column and the output
// cell cy along y; it loads the rows of both groups (at most MO each), forms
// the cell's P sums along y, and adds every z-row into the P nodes along z of
// the cell it departs into; what a group adds to the next cell's node 0 is
// carried in registers (a block marches zcells cells and first reads the group
// before them).  x is gathered out of LDS.
template <typename S, int P, int MO>
__global__ void __launch_bounds__(64 * GCW) k_stream_graded_cells_t(Geometry g, CellReaders<S> tab, const S *__restrict__ in,
                                                             S *__restrict__ out, int cw, int tyc, int nty, int zcells,
                                                             int nchunk)
{
    constexpr int K = P + 1;
    __shared__ S lds[2][P][64 * GCW];                      // P output rows of a z-row, per lane (two buffers in turn)
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                            static_cast<int>(gridDim.x * gridDim.y)));
    const int per = nty * nchunk;
    const int q = L / per, rem = L - q * per;
    const int chunk = rem / nty, ty = rem - chunk * nty;
    const int i = q >> 1, pop = q & 1;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int64_t N = g.nodes, NP = static_cast<int64_t>(Nx) * Ny;
    const Uniform<int32_t> fy = (Uniform<int32_t>)(tab.first[1] + static_cast<int64_t>(i) * (g.nel[1] + 1));
    const Uniform<int32_t> fz = (Uniform<int32_t>)(tab.first[2] + static_cast<int64_t>(i) * (g.nel[2] + 1));
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cyl = wave / cw, xl = (wave - cyl * cw) * 64 + (threadIdx.x & 63);
    const bool valid = ty * tyc + cyl < g.nel[1];
    const int cy = valid ? ty * tyc + cyl : g.nel[1] - 1;
    const bool own = valid && xl < Nx;
    const int xc = xl < Nx ? xl : Nx - 1;
    S *src = const_cast<S *>(in) + static_cast<int64_t>(pop * 45 + i) * N;
    S *dst = out + static_cast<int64_t>(pop * 45 + i) * N;
    const uint32_t xoff = plane_offset<S>(xc);

    // both groups' rows along y (surplus entries repeat the last row, and are not used)
    const int r1 = fy[cy], m1 = fy[cy + 1] - r1;
    const int r0 = cy > 0 ? fy[cy - 1] : fy[g.nel[1] - 1] - Ny, m0 = r1 - r0;
    int rowo[2][MO];
#pragma unroll
    for (int j = 0; j < MO; ++j) {
        rowo[0][j] = wrapi(r1 + min(j, max(m1 - 1, 0)), Ny) * Nx;
        rowo[1][j] = wrapi(r0 + min(j, max(m0 - 1, 0)), Ny) * Nx;
    }
    Uniform<S> wyc = (Uniform<S>)(tab.tw[1] + (static_cast<int64_t>(i) * g.nel[1] + cy) * MO * K);
    // output column xc: node kx of cell xc / P; its taps along x (surplus ones repeat the last, with weight 0)
    const int ex = xc / P, kx = xc - ex * P;
    int to[2][MO];
    S wx[2][MO];
    {
        const int32_t *fx = tab.first[0] + static_cast<int64_t>(i) * (g.nel[0] + 1);
        const S *wxc = tab.tw[0] + (static_cast<int64_t>(i) * g.nel[0] + ex) * MO * K;
        const int s1 = fx[ex], n1 = fx[ex + 1] - s1;
        const int s0 = ex > 0 ? fx[ex - 1] : fx[g.nel[0] - 1] - Nx, n0 = s1 - s0;
        const int a1 = wrapi(s1, Nx), a0 = wrapi(s0, Nx), team = cyl * cw * 64;
#pragma unroll
        for (int j = 0; j < MO; ++j) {
            to[0][j] = team + wrap1(a1 + min(j, max(n1 - 1, 0)), Nx);
            to[1][j] = team + wrap1(a0 + min(j, max(n0 - 1, 0)), Nx);
            wx[0][j] = wxc[j * K + kx];
            wx[1][j] = wxc[j * K + P];
        }
    }
    const Uniform<S> wzt = (Uniform<S>)(tab.w[2] + static_cast<int64_t>(i) * Nz * K);

    const int zc0 = chunk * zcells, zc1 = min(g.nel[2], zc0 + zcells);
    const int zr = zc0 > 0 ? fz[zc0 - 1] : fz[g.nel[2] - 1] - Nz;      // first row: the group before the block's cells
    int z = wrapi(zr, Nz);
    S v[2][MO];
    auto load_row = [&] {
        const int64_t zo = z * NP;
#pragma unroll
        for (int j = 0; j < MO; ++j) {
            v[0][j] = load_at<S>(plane_row(src, zo + rowo[0][j]), xoff);
            v[1][j] = load_at<S>(plane_row(src, zo + rowo[1][j]), xoff);
        }
    };
    load_row();
    S acc[K][P];                                           // [z][y]; acc[P]: for node 0 of the next cell
#pragma unroll
    for (int k = 0; k < P; ++k) acc[P][k] = 0;
    int row = zr, buf = 0;
    for (int c = zc0 - 1; c < zc1; ++c) {
        const int end = fz[c + 1];
#pragma unroll
        for (int k = 0; k < P; ++k) {
            acc[0][k] = acc[P][k];
#pragma unroll
            for (int l = 1; l < K; ++l) acc[l][k] = 0;
        }
        for (; row < end; ++row) {
            asm volatile("" : "+s"(wyc));                  // fetched for each row, not kept (scalar registers)
            S Y[P];
#pragma unroll
            for (int k = 0; k < P; ++k) Y[k] = wyc[k] * v[0][0];
#pragma unroll
            for (int j = 0; j < MO; ++j) {
#pragma unroll
                for (int k = 0; k < P; ++k)
                    if (j > 0) Y[k] = fma(static_cast<S>(wyc[j * K + k]), v[0][j], Y[k]);
                Y[0] = fma(static_cast<S>(wyc[j * K + P]), v[1][j], Y[0]);
            }
            S w[K];
#pragma unroll
            for (int l = 0; l < K; ++l) w[l] = wzt[static_cast<int64_t>(z) * K + l];
            z = wrap1(z + 1, Nz);
            load_row();                                    // past the block's last row: a row of the grid, unused
#pragma unroll
            for (int l = 0; l < K; ++l)
#pragma unroll
                for (int k = 0; k < P; ++k) acc[l][k] = fma(w[l], Y[k], acc[l][k]);
        }
        if (c < zc0) continue;
#pragma unroll
        for (int l = 0; l < P; ++l) {
#pragma unroll
            for (int k = 0; k < P; ++k) lds[buf][k][threadIdx.x] = acc[l][k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const S *b = lds[buf][k];
                S a = 0, e = 0;
#pragma unroll
                for (int j = 0; j < MO; ++j) {
                    a = fma(wx[0][j], b[to[0][j]], a);
                    e = fma(wx[1][j], b[to[1][j]], e);
                }
                a = kx == 0 ? a + e : a;
                if (own)
                    store_at<false, S>(plane_row(dst, static_cast<int64_t>(c * P + l) * NP +
                                                          static_cast<int64_t>(cy * P + k) * Nx), xoff, a);
            }
            buf ^= 1;
        }
    }
}

namespace {

struct GcLayout {
    int cw, tyc, nty;
};

GcLayout gc_layout(const Geometry &g)
{
    GcLayout b;
    b.cw = gc_row_waves(g.N[0]);
    b.tyc = std::min(GCW / b.cw, g.nel[1]);
    b.nty = (g.nel[1] + b.tyc - 1) / b.tyc;
    return b;
}

template <typename S, int P>
hipError_t launch_gc(const Geometry &g, const CellReaders<S> &t, const S *in, S *out, hipStream_t st)
{
    const GcLayout b = gc_layout(g);
    const int rows = (t.my + 1) / 2 * 2;
    const int64_t nb = static_cast<int64_t>(b.nty) * g.nel[2];
    if (90 * nb > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_stream_graded_cells<S, P>), dim3(static_cast<unsigned>(nb), 90), dim3(64 * b.cw * b.tyc),
                       2 * sizeof(S) * b.tyc * rows * b.cw * 64, st, g, t, in, out, b.cw, b.tyc, b.nty, rows);
    return hipGetLastError();
}

template <typename S, int P, int MO>
hipError_t launch_gct(const Geometry &g, const CellReaders<S> &t, const S *in, S *out, hipStream_t st)
{
    const GcLayout b = gc_layout(g);
    // most cells along z per block, fewer while there are fewer than 720 blocks
    // (64^3 nodes, P = 4, FP64: 134, 109, 96, 96 and 122 us with 1, 2, 4, 8 and 16
    // cells; 24^3, P = 3: 17, 14, 16 and 20 us with 1, 2, 4 and 8; 80 x 60 x 60, P = 2,
    // FP32: 73, 60 and 57 us with 4, 8 and 16)
    constexpr int MAXC = P == 2 ? 16 : 4;
    const int want = std::min((719 + 90 * b.nty) / (90 * b.nty), g.nel[2]);
    const int n = std::max(want, (g.nel[2] + MAXC - 1) / MAXC);
    const int zcells = (g.nel[2] + n - 1) / n;
    const int nchunk = (g.nel[2] + zcells - 1) / zcells;
    const int64_t nb = static_cast<int64_t>(b.nty) * nchunk;
    if (90 * nb > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_stream_graded_cells_t<S, P, MO>), dim3(static_cast<unsigned>(nb), 90), dim3(64 * b.cw * b.tyc),
                       0, st, g, t, in, out, b.cw, b.tyc, b.nty, zcells, nchunk);
    return hipGetLastError();
}

template <typename S, int P>
hipError_t launch_gcd(const Geometry &g, const CellReaders<S> &t, bool transpose, const S *in, S *out, hipStream_t st)
{
    if (!transpose) {
        if constexpr (P >= 3) return launch_gc<S, P>(g, t, in, out, st);
        else return hipErrorInvalidValue;
    }
    if (t.most == P + 1) return launch_gct<S, P, P + 1>(g, t, in, out, st);
    return launch_gct<S, P, P + 3>(g, t, in, out, st);
}

}  // namespace

int graded_cell_rows(int p, int most) { return most <= p + 1 ? p + 1 : most <= p + 3 ? p + 3 : 0; }

// Where the kernels by source cell run: whole x rows in a block, at most P + 3
// readers of a cell along x and y, and cells large enough for a block of one
// (forward) or a few (transposed) along z.  Against the march, on the
// cosine-graded mesh in FP64: forward P = 4, 64^3 nodes 77 against 139 us, 128^3 535
// against 1003, P = 3, 24^3 12.5 against 21.6; but P = 2, FP32, 80 x 60 x 60 135 against
// 105 and 128^3 604 against 576 (in FP64 and on small FP32 grids P = 2 by cell is ahead:
// 80 x 60 x 60 137 against 160, 128^3 618 against 768, 16^3 8.4 against 12.5, FP32 8.1
// against 11.6; the march stays there as well) and P = 1 374 against 160.  Transposed P = 4 96 against 267 and 684 against 1865 us, P = 2 57
// against 119; P = 1 176 against 175.
bool graded_by_cell(const Geometry &g, bool transpose, int most, int my, size_t elem)
{
    if (g.N[0] > 64 * GCW || most == 0 || g.p < (transpose ? 2 : 3)) return false;
    const GcLayout b = gc_layout(g);
    // one block per plane: at order 6 its chain is longer than the march's (without launch
    // overhead, 2 x 3 x 1 cells: 11.7 against 11.2 us in FP64, 11.5 and 10.1 in FP32; two
    // blocks, 2 x 2 x 2: 10.5 against 15.4 and 10.1 against 13.8; order 5, 2 x 3 x 1, FP32 8.2 and 8.1)
    if (!transpose && g.p == 6 && b.nty * g.nel[2] == 1) return false;
    return transpose || 2 * elem * b.tyc * ((my + 1) / 2 * 2) * b.cw * 64 <= 64 * 1024;
}

template <typename S>
hipError_t launch_graded_cells(const Geometry &g, const CellReaders<S> &t, bool transpose, const S *in, S *out,
                               hipStream_t st)
{
    switch (g.p) {
    case 2: return launch_gcd<S, 2>(g, t, transpose, in, out, st);
    case 3: return launch_gcd<S, 3>(g, t, transpose, in, out, st);
    case 4: return launch_gcd<S, 4>(g, t, transpose, in, out, st);
    case 5: return launch_gcd<S, 5>(g, t, transpose, in, out, st);
    case 6: return launch_gcd<S, 6>(g, t, transpose, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_graded_cells<double>(const Geometry &, const CellReaders<double> &, bool, const double *,
                                                double *, hipStream_t);
template hipError_t launch_graded_cells<float>(const Geometry &, const CellReaders<float> &, bool, const float *,
                                               float *, hipStream_t);

size_t graded_smem_bytes(int taps, int wxm, int wym, size_t elem)
{
    return (GRB * (static_cast<size_t>(wym) * wxm + static_cast<size_t>(wym) * (GTX + 1)) +
            static_cast<size_t>(taps - 1 + GRB) * GNT) * elem;
}

// largest source window of a 32 x 8 tile along an axis (tile extent T)
int graded_window(const int32_t *src, int N, int taps, int T)
{
    int w = 0;
    for (int t0 = 0; t0 < N; t0 += T) w = std::max(w, src[std::min(t0 + T, N) - 1] - src[t0] + taps);
    return w;
}

int graded_taps_supported(int taps)
{
    static const int ks[] = {2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24};
    for (int k : ks)
        if (k >= taps) return k;
    return 0;
}

int graded_tile_x() { return GTX; }
int graded_window_pad(size_t elem) { return static_cast<int>(16 / elem); }
int graded_max_window() { return 16 * GNT; }
int graded_tile_y() { return GTY; }

template <typename S, int K, int LK, int V>
static hipError_t launch_gk(const Geometry &g, const NodeTables<S> &t, const S *in, S *out, hipStream_t st)
{
    const int ntx = (g.N[0] + GTX - 1) / GTX, nty = (g.N[1] + GTY - 1) / GTY;
    const int ntiles = ntx * nty;
    // split the z-march into chunks (each re-reads p source rows) until the
    // grid has a few blocks per CU slot
    int nchunk = 1;
    while (static_cast<int64_t>(ntiles) * 90 * nchunk < GRADED_TARGET_BLOCKS && g.N[2] / (2 * nchunk) >= 4 * K)
        nchunk *= 2;
    const int zrows = (g.N[2] + nchunk - 1) / nchunk;
    nchunk = (g.N[2] + zrows - 1) / zrows;
    const int64_t nb = static_cast<int64_t>(ntiles) * 90 * nchunk;
    if (nb > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
    const size_t smem = graded_smem_bytes(K, t.wxm, t.wym, sizeof(S));
    if (smem > 160 * 1024) return hipErrorInvalidValue;
    if (smem > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_stream_graded<S, K, LK, V>),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem));
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_stream_graded<S, K, LK, V>), dim3(static_cast<unsigned>(nb)), dim3(GNT), smem, st, g, t, in,
                       out, ntx, ntiles, zrows, nchunk);
    return hipGetLastError();
}

// window loads per thread: the smallest LK with LK * 256 >= the largest window
template <typename S, int K, int V>
static hipError_t launch_gv(const Geometry &g, const NodeTables<S> &t, const S *in, S *out, hipStream_t st)
{
    const int nw = (t.wxm / V) * t.wym;                    // V-wide loads of the largest window
    if (nw <= 1 * GNT) return launch_gk<S, K, 1, V>(g, t, in, out, st);
    if (nw <= 2 * GNT) return launch_gk<S, K, 2, V>(g, t, in, out, st);
    if (nw <= 4 * GNT) return launch_gk<S, K, 4, V>(g, t, in, out, st);
    if (nw <= 8 * GNT) return launch_gk<S, K, 8, V>(g, t, in, out, st);
    if (nw <= 16 * GNT) return launch_gk<S, K, 16, V>(g, t, in, out, st);
    return hipErrorInvalidValue;
}

// 16-byte window loads when x rows hold a multiple of 16 bytes and the
// buffer is 16-byte aligned (the window start is rounded down)
template <typename S, int K>
static hipError_t launch_g(const Geometry &g, const NodeTables<S> &t, const S *in, S *out, hipStream_t st)
{
    constexpr int V = 16 / sizeof(S);
    if ((g.N[0] * sizeof(S)) % 16 == 0 && reinterpret_cast<uintptr_t>(in) % 16 == 0 && t.wxm % V == 0)
        return launch_gv<S, K, V>(g, t, in, out, st);
    return launch_gv<S, K, 1>(g, t, in, out, st);
}

// taps per output: p + 1 for the forward tables, the padded band width of
// the transposed ones (graded_taps_supported)
template <typename S>
hipError_t launch_stream_graded(const Geometry &g, const NodeTables<S> &t, const S *in, S *out, hipStream_t st)
{
    switch (t.k) {
    case 2: return launch_g<S, 2>(g, t, in, out, st);
    case 3: return launch_g<S, 3>(g, t, in, out, st);
    case 4: return launch_g<S, 4>(g, t, in, out, st);
    case 5: return launch_g<S, 5>(g, t, in, out, st);
    case 6: return launch_g<S, 6>(g, t, in, out, st);
    case 7: return launch_g<S, 7>(g, t, in, out, st);
    case 8: return launch_g<S, 8>(g, t, in, out, st);
    case 10: return launch_g<S, 10>(g, t, in, out, st);
    case 12: return launch_g<S, 12>(g, t, in, out, st);
    case 14: return launch_g<S, 14>(g, t, in, out, st);
    case 16: return launch_g<S, 16>(g, t, in, out, st);
    case 20: return launch_g<S, 20>(g, t, in, out, st);
    case 24: return launch_g<S, 24>(g, t, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_graded<double>(const Geometry &, const NodeTables<double> &, const double *,
                                                 double *, hipStream_t);
template hipError_t launch_stream_graded<float>(const Geometry &, const NodeTables<float> &, const float *, float *,
                                                hipStream_t);

}  // namespace sllbm
