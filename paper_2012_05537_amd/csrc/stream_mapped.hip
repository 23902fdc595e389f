// Semi-Lagrangian streaming on a distorted mesh (Sec. II A: departure points
// traced once through the cells; with distorted cells the interpolation does
// not factorise per axis and the paper's subsection "Numerical efficiency"
// expects a memory-bound kernel), and its transpose.
//
// The cells are the isoparametric images of the equal-cell reference grid
// (node displacements, build_mapped_tables); populations are interpolated in
// reference coordinates.  The host stores, per velocity and node, the
// departure cell and the three local coordinates (28 bytes in FP64, 16 in
// FP32); the weights are formed here ("matrix-free": 3 (P+1) Lagrange values
// instead of (P+1)^3 stored coefficients).  Kernels:
//   * k_stream_mapped_cells (P >= 3): the forward streaming by departure cell;
//   * k_stream_mapped_win (P < 3): the forward streaming by node tile, its
//     source window staged in LDS;
//   * k_stream_mapped_t_cells / _nodes: the transpose in a fixed order.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sllbm_internal.h"
#include "xcd.h"

namespace sllbm {

template <typename S, int V>
struct MVec {
    typedef S T __attribute__((ext_vector_type(V)));
};

// w[a][k] = ell_k(t_a), formed in double from the coordinates tl[a]
template <typename S, int P>
__device__ __forceinline__ void lagrange_weights(const GlcBasis &gb, const double (&tl)[3], S (&w)[3][P + 1])
{
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double d[P + 1], pre[P + 1];                       // t - t_k, product of the d before k
#pragma unroll
        for (int k = 0; k <= P; ++k) d[k] = tl[a] - gb.t[k];
        pre[0] = 1.0;
#pragma unroll
        for (int k = 1; k <= P; ++k) pre[k] = pre[k - 1] * d[k - 1];
        double suf = 1.0;
#pragma unroll
        for (int k = P; k >= 0; --k) {
            w[a][k] = static_cast<S>(gb.inv_den[k] * (pre[k] * suf));
            suf *= d[k];
        }
    }
}

// G elements (8 or 9) of a cell and their weights: f into a0, a1 in turn, g into
// b0, b1.  Element k sits in lane (E + k) % 16 of its 16-lane row and enters its
// FMAs as a row broadcast (row_newbcast).  A register that a vector instruction
// wrote may be read by such an FMA no less than two wait states later, and the
// compiler does not see into the block: the s_nop covers whatever is written before
// it (values, weights, cleared sums, copies, reloads), and inside it the FMAs of
// one sum have three others between them.
#define SLLBM_ROW_FMA(OP, ACC, SRC, W, LANE) \
    OP " %" #ACC ", %" #SRC ", %" #W " row_newbcast:%" #LANE " row_mask:0xf bank_mask:0xf\n\t"
#define SLLBM_AT(V, K) V[(E + K) / 16]
#define SLLBM_ROW_FMAS(S, OP)                                                                                  \
    template <int E, int G, int NR, int NW>                                                                    \
    __device__ __forceinline__ void fma_rows(S &a0, S &a1, S &b0, S &b1, const S (&vf)[NR], const S (&vg)[NR], \
                                             const S (&w)[NW], int wi)                                         \
    {                                                                                                          \
        static_assert(G == 8 || G == 9, "elements per block");                                                 \
        if constexpr (G == 8)                                                                                  \
            asm("s_nop 1\n\t"                                                                                  \
                SLLBM_ROW_FMA(OP, 0, 4, 20, 28) SLLBM_ROW_FMA(OP, 2, 12, 20, 28)                               \
                SLLBM_ROW_FMA(OP, 1, 5, 21, 29) SLLBM_ROW_FMA(OP, 3, 13, 21, 29)                               \
                SLLBM_ROW_FMA(OP, 0, 6, 22, 30) SLLBM_ROW_FMA(OP, 2, 14, 22, 30)                               \
                SLLBM_ROW_FMA(OP, 1, 7, 23, 31) SLLBM_ROW_FMA(OP, 3, 15, 23, 31)                               \
                SLLBM_ROW_FMA(OP, 0, 8, 24, 32) SLLBM_ROW_FMA(OP, 2, 16, 24, 32)                               \
                SLLBM_ROW_FMA(OP, 1, 9, 25, 33) SLLBM_ROW_FMA(OP, 3, 17, 25, 33)                               \
                SLLBM_ROW_FMA(OP, 0, 10, 26, 34) SLLBM_ROW_FMA(OP, 2, 18, 26, 34)                              \
                SLLBM_ROW_FMA(OP, 1, 11, 27, 35) SLLBM_ROW_FMA(OP, 3, 19, 27, 35)                              \
                : "+&v"(a0), "+&v"(a1), "+&v"(b0), "+&v"(b1)                                                   \
                : "v"(SLLBM_AT(vf, 0)), "v"(SLLBM_AT(vf, 1)), "v"(SLLBM_AT(vf, 2)), "v"(SLLBM_AT(vf, 3)),      \
                  "v"(SLLBM_AT(vf, 4)), "v"(SLLBM_AT(vf, 5)), "v"(SLLBM_AT(vf, 6)), "v"(SLLBM_AT(vf, 7)),      \
                  "v"(SLLBM_AT(vg, 0)), "v"(SLLBM_AT(vg, 1)), "v"(SLLBM_AT(vg, 2)), "v"(SLLBM_AT(vg, 3)),      \
                  "v"(SLLBM_AT(vg, 4)), "v"(SLLBM_AT(vg, 5)), "v"(SLLBM_AT(vg, 6)), "v"(SLLBM_AT(vg, 7)),      \
                  "v"(w[wi + 0]), "v"(w[wi + 1]), "v"(w[wi + 2]), "v"(w[wi + 3]),                              \
                  "v"(w[wi + 4]), "v"(w[wi + 5]), "v"(w[wi + 6]), "v"(w[wi + 7]),                              \
                  "n"((E + 0) % 16), "n"((E + 1) % 16), "n"((E + 2) % 16), "n"((E + 3) % 16),                  \
                  "n"((E + 4) % 16), "n"((E + 5) % 16), "n"((E + 6) % 16), "n"((E + 7) % 16));                 \
        else                                                                                                   \
            asm("s_nop 1\n\t"                                                                                  \
                SLLBM_ROW_FMA(OP, 0, 4, 22, 31) SLLBM_ROW_FMA(OP, 2, 13, 22, 31)                               \
                SLLBM_ROW_FMA(OP, 1, 5, 23, 32) SLLBM_ROW_FMA(OP, 3, 14, 23, 32)                               \
                SLLBM_ROW_FMA(OP, 0, 6, 24, 33) SLLBM_ROW_FMA(OP, 2, 15, 24, 33)                               \
                SLLBM_ROW_FMA(OP, 1, 7, 25, 34) SLLBM_ROW_FMA(OP, 3, 16, 25, 34)                               \
                SLLBM_ROW_FMA(OP, 0, 8, 26, 35) SLLBM_ROW_FMA(OP, 2, 17, 26, 35)                               \
                SLLBM_ROW_FMA(OP, 1, 9, 27, 36) SLLBM_ROW_FMA(OP, 3, 18, 27, 36)                               \
                SLLBM_ROW_FMA(OP, 0, 10, 28, 37) SLLBM_ROW_FMA(OP, 2, 19, 28, 37)                              \
                SLLBM_ROW_FMA(OP, 1, 11, 29, 38) SLLBM_ROW_FMA(OP, 3, 20, 29, 38)                              \
                SLLBM_ROW_FMA(OP, 0, 12, 30, 39) SLLBM_ROW_FMA(OP, 2, 21, 30, 39)                              \
                : "+&v"(a0), "+&v"(a1), "+&v"(b0), "+&v"(b1)                                                   \
                : "v"(SLLBM_AT(vf, 0)), "v"(SLLBM_AT(vf, 1)), "v"(SLLBM_AT(vf, 2)), "v"(SLLBM_AT(vf, 3)),      \
                  "v"(SLLBM_AT(vf, 4)), "v"(SLLBM_AT(vf, 5)), "v"(SLLBM_AT(vf, 6)), "v"(SLLBM_AT(vf, 7)),      \
                  "v"(SLLBM_AT(vf, 8)),                                                                        \
                  "v"(SLLBM_AT(vg, 0)), "v"(SLLBM_AT(vg, 1)), "v"(SLLBM_AT(vg, 2)), "v"(SLLBM_AT(vg, 3)),      \
                  "v"(SLLBM_AT(vg, 4)), "v"(SLLBM_AT(vg, 5)), "v"(SLLBM_AT(vg, 6)), "v"(SLLBM_AT(vg, 7)),      \
                  "v"(SLLBM_AT(vg, 8)),                                                                        \
                  "v"(w[wi + 0]), "v"(w[wi + 1]), "v"(w[wi + 2]), "v"(w[wi + 3]),                              \
                  "v"(w[wi + 4]), "v"(w[wi + 5]), "v"(w[wi + 6]), "v"(w[wi + 7]),                              \
                  "v"(w[wi + 8]),                                                                              \
                  "n"((E + 0) % 16), "n"((E + 1) % 16), "n"((E + 2) % 16), "n"((E + 3) % 16),                  \
                  "n"((E + 4) % 16), "n"((E + 5) % 16), "n"((E + 6) % 16), "n"((E + 7) % 16),                  \
                  "n"((E + 8) % 16));                                                                          \
    }
SLLBM_ROW_FMAS(double, "v_fmac_f64_dpp")
SLLBM_ROW_FMAS(float, "v_fmac_f32_dpp")
#undef SLLBM_ROW_FMAS
#undef SLLBM_AT
#undef SLLBM_ROW_FMA

// sf, sg += sum over the cell's elements E, E + 1, ... of weight times value.
// z: sums of the current z plane so far, two for f and two for g (element
// pairs alternate).
template <typename S, int P, int E, int NR>
__device__ __forceinline__ void cell_sum(const S (&vf)[NR], const S (&vg)[NR], const S (&wxy)[(P + 1) * (P + 1)],
                                         const S (&wz)[P + 1], S (&z)[4], S &sf, S &sg)
{
    constexpr int K = P + 1, K2 = K * K, e = E % K2, G = (K2 - e) % 8 == 0 ? 8 : 9;
    fma_rows<E, G>(z[e % 2], z[1 - e % 2], z[2 + e % 2], z[3 - e % 2], vf, vg, wxy, e);
    if constexpr (e + G == K2) {
        sf = fma(wz[E / K2], z[0] + z[1], sf);
        sg = fma(wz[E / K2], z[2] + z[3], sg);
        z[0] = z[1] = z[2] = z[3] = 0;
    }
    if constexpr (E + G < K2 * K) cell_sum<S, P, E + G>(vf, vg, wxy, wz, z, sf, sg);
}

// Streaming by departure cell.  A block owns one velocity and a run of cells
// along x (MappedRuns): it stages the run's source rows of f and g in LDS
// (coalesced, each value once) and takes the nodes that depart into the run.
// A 16-lane row takes one chunk, up to 16 nodes that depart into one cell
// (build_mapped_chunks), and holds that cell's (P+1)^3 support values of f and
// of g once, spread over its lanes; they enter the FMAs as row broadcasts, so
// that a support value costs one LDS read per 16 outputs and not one per output.
// Bound by the vector pipes (about 400 instructions per 64 lanes at P = 4, 250
// of them the FMAs of f and g; rows are 80 % full) together with the scattered
// reads and writes; measured at 64^3 nodes, P = 4: 235 us in FP64 and 163 us in
// FP32, against 376 and 249 us for the gather out of LDS by node tile, which
// read 2 KB from LDS per output (P = 3, 48^3 nodes: 77 / 54 against 109 / 77 us;
// P = 6: 184 / 126 against 518 / 219 us on 42 x 42 x 48).
// Also measured: the support values as scalar operands through the scalar cache
// 774 us (its misses serialise); rows loaded straight from global memory
// 310 us (every cache line is fetched by four cells).
// tloc: local coordinates in list order; chunk: [Q][nch] (cell in the run and
// count, first list position); rstart: [Q][runs + 1] first chunk of a run.
template <typename S, int P>
__global__ void __launch_bounds__(256, P <= 4 ? 4 : 2)
    k_stream_mapped_cells(Geometry g, GlcBasis gb, MappedRuns runs, const int32_t *__restrict__ order,
                          const int2 *__restrict__ chunk, int nch, const int32_t *__restrict__ rstart,
                          const S *__restrict__ tloc, const S *__restrict__ in, S *__restrict__ out)
{
    constexpr int K = P + 1, K3 = K * K * K, NR = (K3 + 15) / 16;
    using S2 = typename MVec<S, 2>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    S2 *lw = reinterpret_cast<S2 *>(smem);                 // [K][K][width] f and g of the run's window
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(static_cast<int>(blockIdx.y * gridDim.x + blockIdx.x),
                                                            static_cast<int>(gridDim.x * gridDim.y)));
    const int nruns = runs.nx * g.nel[1] * g.nel[2];
    const int i = L / nruns, run = L - i * nruns;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int row = (threadIdx.x >> 4) & 3, j = threadIdx.x & 15;
    const int64_t N = g.nodes;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const S *__restrict__ fi = in + static_cast<int64_t>(i) * N;
    const S *__restrict__ gi = in + static_cast<int64_t>(Q + i) * N;
    S *__restrict__ fo = out + static_cast<int64_t>(i) * N;
    S *__restrict__ go = out + static_cast<int64_t>(Q + i) * N;
    const int q0 = rstart[static_cast<int64_t>(i) * (nruns + 1) + run];
    const int q1 = rstart[static_cast<int64_t>(i) * (nruns + 1) + run + 1];
    if (q0 == q1) return;                                  // nothing departs into this run
    const int2 *__restrict__ ch = chunk + static_cast<int64_t>(i) * nch;
    int2 d;
    int n_next;
    S tl_next[3];
    auto load_entry = [&](int q) {                         // the row's chunk of group q, and its list entry
        d = ch[min(q + row, q1 - 1)];
        const int count = d.x >> 8;
        const int64_t le = static_cast<int64_t>(i) * N + d.y + min(j, count - 1);
        n_next = order[le];
#pragma unroll
        for (int a = 0; a < 3; ++a) tl_next[a] = tloc[static_cast<int64_t>(a) * Q * N + le];
    };
    {
        const int rx = run % runs.nx, r1 = run / runs.nx;
        const int ey = r1 % g.nel[1], ez = r1 / g.nel[1];
        const int ex = rx * runs.cells;
        const int width = min(runs.cells, g.nel[0] - ex) * P + 1;
        const int x0 = ex * P, y0 = ey * P, z0 = ez * P;
        const float rw = 1.0f / static_cast<float>(width);
        for (int k = threadIdx.x; k < K * K * width; k += 256) {
            // exact quotient: (k + 1/2) / width lies at least 1 / (2 width) from an
            // integer, and k < 2^13
            const int r = static_cast<int>((static_cast<float>(k) + 0.5f) * rw);
            const int x = k - r * width;
            int xx = x0 + x, yy = y0 + r % K, zz = z0 + r / K;
            xx -= xx >= Nx ? Nx : 0;
            yy -= yy >= Ny ? Ny : 0;
            zz -= zz >= Nz ? Nz : 0;
            const int64_t node = (static_cast<int64_t>(zz) * Ny + yy) * Nx + xx;
            S2 v;
            v.x = fi[node];
            v.y = gi[node];
            lw[r * runs.width + x] = v;
        }
    }
    // elements 16 r + j of a cell: LDS offset from its first node
    int off[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int e = min(16 * r + j, K3 - 1);
        off[r] = e / K * runs.width + e % K;
    }
    load_entry(q0 + wave * 4);
    __syncthreads();
    for (int q = q0 + wave * 4; q < q1; q += 16) {
        const int count = q + row < q1 ? d.x >> 8 : 0;
        const int n = n_next;
        const double tl[3] = {static_cast<double>(tl_next[0]), static_cast<double>(tl_next[1]),
                              static_cast<double>(tl_next[2])};
        const S2 *cell = lw + (d.x & 255) * P;
        S vf[NR], vg[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const S2 v = cell[off[r]];
            vf[r] = v.x;
            vg[r] = v.y;
        }
        load_entry(q + 16);                                // past the run: its last chunk again
        S w[3][K], wxy[K * K];
        lagrange_weights<S, P>(gb, tl, w);
#pragma unroll
        for (int y = 0; y < K; ++y)
#pragma unroll
            for (int x = 0; x < K; ++x) wxy[y * K + x] = w[1][y] * w[0][x];
        S sf = 0, sg = 0, z[4] = {0, 0, 0, 0};
        cell_sum<S, P, 0>(vf, vg, wxy, w[2], z, sf, sg);
        if (j < count) {
            fo[n] = sf;
            go[n] = sg;
        }
    }
}

// Streaming by node tile, for orders below MAPPED_LIST_ORDER, whose cells have
// too few nodes (P^3 = 1 or 8) to fill the 16-lane rows of
// k_stream_mapped_cells (64^3 nodes, P = 2, FP64: 186 against 233 us).  A block
// owns one velocity and a tile of MAPPED_TX x MAPPED_TY x MAPPED_TZ nodes; the
// host has found the box of cells that holds the departure cells of all of
// them (build_mapped_windows), the block loads that window once (coalesced
// rows), f and g of a node side by side so that one LDS read returns both, and
// every thread gathers its (P+1)^3 support pairs from LDS.  The blocks run in
// XCD-aware order (consecutive tiles of a velocity on one XCD, where their
// overlapping windows and the table lines they share meet in one L2).  A
// block whose window exceeds the LDS budget gathers from global memory
// instead; both paths sum in the same order, so they give the same bits.
template <typename S, int P>
__global__ void __launch_bounds__(256, MAPPED_MIN_WAVES) k_stream_mapped_win(
    Geometry g, GlcBasis gb, const int32_t *__restrict__ cell, const S *__restrict__ tloc,
    const int32_t *__restrict__ win, int ntiles, int ntx, int nty, const S *__restrict__ in, S *__restrict__ out)
{
    using S2 = typename MVec<S, 2>::T;
    extern __shared__ __align__(16) unsigned char smem[];
    const int L = __builtin_amdgcn_readfirstlane(xcd_linear(blockIdx.x, gridDim.x));
    const int i = L / ntiles;
    const int t = L - i * ntiles;
    const int64_t N = g.nodes;
    const int Nx = g.N[0], Ny = g.N[1], Nz = g.N[2];
    const int32_t *w = win + (static_cast<int64_t>(i) * ntiles + t) * 4;
    const int ocx = w[0], ocy = w[1], ocz = w[2], dims = w[3];
    const int gx = (t % ntx) * MAPPED_TX + (threadIdx.x % MAPPED_TX);
    const int gy = ((t / ntx) % nty) * MAPPED_TY + (threadIdx.x / MAPPED_TX) % MAPPED_TY;
    const int gz = (t / (ntx * nty)) * MAPPED_TZ + threadIdx.x / (MAPPED_TX * MAPPED_TY);
    const bool own = gx < Nx && gy < Ny && gz < Nz;
    const S *fi = in + static_cast<int64_t>(i) * N;
    const S *gi = in + static_cast<int64_t>(Q + i) * N;
    const int wx = dims & 1023, wy = (dims >> 10) & 1023, wz = dims >> 20;
    S2 *lw = reinterpret_cast<S2 *>(smem);
    if (dims != 0) {
        const int wt = wx * wy * wz;
        const int ox = ocx * P, oy = ocy * P, oz = ocz * P;
        const float rx = 1.0f / static_cast<float>(wx), ry = 1.0f / static_cast<float>(wy);
        for (int k = threadIdx.x; k < wt; k += blockDim.x) {
            // k = (z wy + y) wx + x.  The quotients in single precision are
            // exact: (k + 1/2)/wx lies at least 1/(2 wx) from an integer, and
            // the two roundings move it by less than that while k < 2^21
            // (a window holds at most a few thousand nodes).
            const int r = static_cast<int>((static_cast<float>(k) + 0.5f) * rx);
            const int z = static_cast<int>((static_cast<float>(r) + 0.5f) * ry);
            const int x = k - r * wx, y = r - z * wy;
            // origin node < N and window extent <= N + 1 along every axis
            int xx = ox + x, yy = oy + y, zz = oz + z;
            xx -= xx >= Nx ? Nx : 0;
            yy -= yy >= Ny ? Ny : 0;
            zz -= zz >= Nz ? Nz : 0;
            const int64_t node = (static_cast<int64_t>(zz) * Ny + yy) * Nx + xx;
            S2 v;
            v.x = fi[node];
            v.y = gi[node];
            lw[k] = v;
        }
        __syncthreads();
    }
    if (!own) return;
    const int64_t n = (static_cast<int64_t>(gz) * Ny + gy) * Nx + gx;
    const int c = cell[static_cast<int64_t>(i) * N + n];
    const int ex = c % g.nel[0], rest = c / g.nel[0];
    const int ey = rest % g.nel[1], ez = rest / g.nel[1];
    S wt3[3][P + 1];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double tt = static_cast<double>(tloc[(static_cast<int64_t>(a) * Q + i) * N + n]);
#pragma unroll
        for (int k = 0; k <= P; ++k) {
            double v = gb.inv_den[k];
#pragma unroll
            for (int m = 0; m <= P; ++m)
                if (m != k) v *= tt - gb.t[m];
            wt3[a][k] = static_cast<S>(v);
        }
    }
    S sf = 0, sg = 0;
    if (dims != 0) {
        int bx = ex - ocx, by = ey - ocy, bz = ez - ocz;       // the departure cell inside the window
        bx += bx < 0 ? g.nel[0] : 0;
        by += by < 0 ? g.nel[1] : 0;
        bz += bz < 0 ? g.nel[2] : 0;
#pragma unroll
        for (int kz = 0; kz <= P; ++kz)
#pragma unroll
            for (int ky = 0; ky <= P; ++ky) {
                const int base = ((bz * P + kz) * wy + by * P + ky) * wx + bx * P;
                S af = 0, ag = 0;
#pragma unroll
                for (int kx = 0; kx <= P; ++kx) {
                    const S2 v = lw[base + kx];
                    af = fma(wt3[0][kx], v.x, af);
                    ag = fma(wt3[0][kx], v.y, ag);
                }
                const S wyz = wt3[1][ky] * wt3[2][kz];
                sf = fma(wyz, af, sf);
                sg = fma(wyz, ag, sg);
            }
    } else {
#pragma unroll
        for (int kz = 0; kz <= P; ++kz) {
            int zz = ez * P + kz;
            zz = zz >= Nz ? zz - Nz : zz;
#pragma unroll
            for (int ky = 0; ky <= P; ++ky) {
                int yy = ey * P + ky;
                yy = yy >= Ny ? yy - Ny : yy;
                const int64_t row = (static_cast<int64_t>(zz) * Ny + yy) * Nx;
                S af = 0, ag = 0;
#pragma unroll
                for (int kx = 0; kx <= P; ++kx) {
                    int xx = ex * P + kx;
                    xx = xx >= Nx ? xx - Nx : xx;
                    af = fma(wt3[0][kx], fi[row + xx], af);
                    ag = fma(wt3[0][kx], gi[row + xx], ag);
                }
                const S wyz = wt3[1][ky] * wt3[2][kz];
                sf = fma(wyz, af, sf);
                sg = fma(wyz, ag, sg);
            }
        }
    }
    out[static_cast<int64_t>(i) * N + n] = sf;
    out[static_cast<int64_t>(Q + i) * N + n] = sg;
}

// Transposed streaming S^T on a distorted mesh, summed in a fixed order.
// Output n of velocity i read the (P+1)^3 support values of its departure
// cell c with the weights l_a(t_x) l_b(t_y) l_c(t_z); transposed, support
// point (a, b, c) of cell c receives the sum, over the nodes n departing into
// c, of the same weight times the adjoint of n.
//   Pass 1 (k_stream_mapped_t_cells): one block per (cell, velocity) forms
//   these (P+1)^3 partial sums for f and g, walking the cell's inverse list
//   (build_mapped_inverse) in increasing node order.
//   Pass 2 (k_stream_mapped_t_nodes): every node adds the partial sums of the
//   1, 2, 4 or 8 cells that share it, in a fixed order.
// No atomics: the result is the same bit for bit on every run.
template <int P>
constexpr int mt_threads()
{
    return ((P + 1) * (P + 1) * (P + 1) + 63) / 64 * 64;
}

template <typename S, int P>
__global__ void __launch_bounds__(mt_threads<P>()) k_stream_mapped_t_cells(
    Geometry g, GlcBasis gb, const int32_t *__restrict__ order, const int32_t *__restrict__ start,
    const S *__restrict__ tloc, const S *__restrict__ in, S *__restrict__ partial, int i0)
{
    constexpr int K = P + 1, K3 = K * K * K;
    constexpr int CH = 64;                                 // list entries staged per round
    __shared__ S lw[CH][3][K];
    __shared__ S ly[CH][2];
    const int c = blockIdx.x;
    const int C = static_cast<int>(gridDim.x);
    const int i = i0 + static_cast<int>(blockIdx.y);
    const int64_t N = g.nodes;
    const int32_t *st = start + static_cast<int64_t>(i) * (C + 1);
    const int b0 = st[c], b1 = st[c + 1];
    const int tid = threadIdx.x;
    const int a = tid % K, b = (tid / K) % K, e = tid / (K * K);   // this thread's support point
    S accf = 0, accg = 0;
    for (int base = b0; base < b1; base += CH) {
        const int nb = min(CH, b1 - base);
        if (tid < nb) {
            const int64_t n = order[static_cast<int64_t>(i) * N + base + tid];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax) {
                const int64_t at = P >= MAPPED_LIST_ORDER ? base + tid : n;
                const double tt = static_cast<double>(tloc[(static_cast<int64_t>(ax) * Q + i) * N + at]);
#pragma unroll
                for (int k = 0; k <= P; ++k) {
                    double v = gb.inv_den[k];
#pragma unroll
                    for (int m = 0; m <= P; ++m)
                        if (m != k) v *= tt - gb.t[m];
                    lw[tid][ax][k] = static_cast<S>(v);
                }
            }
            ly[tid][0] = in[static_cast<int64_t>(i) * N + n];
            ly[tid][1] = in[static_cast<int64_t>(Q + i) * N + n];
        }
        __syncthreads();
        if (tid < K3) {
            for (int k = 0; k < nb; ++k) {
                const S w = lw[k][0][a] * (lw[k][1][b] * lw[k][2][e]);
                accf = fma(w, ly[k][0], accf);
                accg = fma(w, ly[k][1], accg);
            }
        }
        __syncthreads();
    }
    if (tid < K3) {
        S *pp = partial + (static_cast<int64_t>(blockIdx.y) * C + c) * 2 * K3;
        pp[tid] = accf;
        pp[K3 + tid] = accg;
    }
}

template <typename S, int P>
__global__ void __launch_bounds__(256) k_stream_mapped_t_nodes(Geometry g, const S *__restrict__ partial,
                                                               S *__restrict__ out, int i0)
{
    constexpr int K = P + 1, K3 = K * K * K;
    const int i = i0 + static_cast<int>(blockIdx.y);
    const int64_t N = g.nodes;
    const int64_t m = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (m >= N) return;
    const int Nx = g.N[0], Ny = g.N[1];
    const int64_t NP = static_cast<int64_t>(Nx) * Ny;
    const int gz = static_cast<int>(m / NP), gy = static_cast<int>((m / Nx) % Ny), gx = static_cast<int>(m % Nx);
    const int C = g.nel[0] * g.nel[1] * g.nel[2];
    // along an axis node q lies in cell q / P at local point q % P, and when
    // q % P == 0 also in the previous cell (wrapped) at local point P
    int cs[3][2], ls[3][2], nc[3];
    const int gq[3] = {gx, gy, gz};
#pragma unroll
    for (int ax = 0; ax < 3; ++ax) {
        const int e = gq[ax] / P, l = gq[ax] - e * P;
        nc[ax] = 1;
        cs[ax][0] = e;
        ls[ax][0] = l;
        if (l == 0) {
            cs[ax][1] = e == 0 ? g.nel[ax] - 1 : e - 1;
            ls[ax][1] = P;
            nc[ax] = 2;
        }
    }
    const S *pb = partial + static_cast<int64_t>(blockIdx.y) * C * 2 * K3;
    S sf = 0, sg = 0;
    for (int z = 0; z < nc[2]; ++z)
        for (int y = 0; y < nc[1]; ++y)
            for (int x = 0; x < nc[0]; ++x) {
                const int c = (cs[2][z] * g.nel[1] + cs[1][y]) * g.nel[0] + cs[0][x];
                const int k = (ls[2][z] * K + ls[1][y]) * K + ls[0][x];
                const S *pp = pb + static_cast<int64_t>(c) * 2 * K3;
                sf += pp[k];
                sg += pp[K3 + k];
            }
    out[static_cast<int64_t>(i) * N + m] = sf;
    out[static_cast<int64_t>(Q + i) * N + m] = sg;
}

namespace {

template <typename S, int P>
hipError_t launch_mt(const Geometry &g, const MappedTables &t, const S *in, S *out, hipStream_t st)
{
    const int64_t cells = static_cast<int64_t>(g.nel[0]) * g.nel[1] * g.nel[2];
    const int64_t bx = (g.nodes + 255) / 256;
    if (bx > (int64_t(1) << 31) - 1 || cells > (int64_t(1) << 31) - 1 || !t.inv_order || !t.partial)
        return hipErrorInvalidValue;
    for (int i0 = 0; i0 < Q; i0 += t.qchunk) {
        const int qc = std::min(t.qchunk, Q - i0);
        hipLaunchKernelGGL((k_stream_mapped_t_cells<S, P>), dim3(static_cast<unsigned>(cells), qc),
                           dim3(mt_threads<P>()), 0, st, g, t.basis, t.inv_order, t.inv_start,
                           static_cast<const S *>(t.tloc), in, static_cast<S *>(t.partial), i0);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL((k_stream_mapped_t_nodes<S, P>), dim3(static_cast<unsigned>(bx), qc), dim3(256), 0, st, g,
                           static_cast<const S *>(t.partial), out, i0);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename S, int P>
hipError_t launch_m(const Geometry &g, const MappedTables &t, const S *in, S *out, hipStream_t st)
{
    if constexpr (P >= MAPPED_LIST_ORDER) {
        unsigned runs;
        if (!mapped_run_grid(t.runs, g.nel, runs)) return hipErrorInvalidValue;
        const size_t lds = 2 * static_cast<size_t>(P + 1) * (P + 1) * t.runs.width * sizeof(S);
        hipLaunchKernelGGL((k_stream_mapped_cells<S, P>), dim3(runs, Q), dim3(256), lds, st, g, t.basis,
                           t.runs, t.inv_order, reinterpret_cast<const int2 *>(t.chunk), t.nch, t.rstart,
                           static_cast<const S *>(t.tloc), in, out);
        return hipGetLastError();
    } else {
        const int ntx = (g.N[0] + MAPPED_TX - 1) / MAPPED_TX, nty = (g.N[1] + MAPPED_TY - 1) / MAPPED_TY,
                  ntz = (g.N[2] + MAPPED_TZ - 1) / MAPPED_TZ;
        const int64_t ntiles = static_cast<int64_t>(ntx) * nty * ntz;
        if (ntiles * Q > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
        const size_t lds = 2 * static_cast<size_t>(t.win_nodes) * sizeof(S);
        hipLaunchKernelGGL((k_stream_mapped_win<S, P>), dim3(static_cast<unsigned>(ntiles * Q)), dim3(256), lds, st,
                           g, t.basis, t.cell, static_cast<const S *>(t.tloc), t.win, static_cast<int>(ntiles), ntx,
                           nty, in, out);
        return hipGetLastError();
    }
}

}  // namespace

template <typename S>
hipError_t launch_stream_mapped(const Geometry &g, const MappedTables &t, const S *in, S *out, hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_m<S, 1>(g, t, in, out, st);
    case 2: return launch_m<S, 2>(g, t, in, out, st);
    case 3: return launch_m<S, 3>(g, t, in, out, st);
    case 4: return launch_m<S, 4>(g, t, in, out, st);
    case 5: return launch_m<S, 5>(g, t, in, out, st);
    case 6: return launch_m<S, 6>(g, t, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template <typename S>
hipError_t launch_stream_mapped_t(const Geometry &g, const MappedTables &t, const S *in, S *out, hipStream_t st)
{
    switch (g.p) {
    case 1: return launch_mt<S, 1>(g, t, in, out, st);
    case 2: return launch_mt<S, 2>(g, t, in, out, st);
    case 3: return launch_mt<S, 3>(g, t, in, out, st);
    case 4: return launch_mt<S, 4>(g, t, in, out, st);
    case 5: return launch_mt<S, 5>(g, t, in, out, st);
    case 6: return launch_mt<S, 6>(g, t, in, out, st);
    default: return hipErrorInvalidValue;
    }
}

template hipError_t launch_stream_mapped_t<double>(const Geometry &, const MappedTables &, const double *, double *,
                                                   hipStream_t);
template hipError_t launch_stream_mapped_t<float>(const Geometry &, const MappedTables &, const float *, float *,
                                                  hipStream_t);
template hipError_t launch_stream_mapped<double>(const Geometry &, const MappedTables &, const double *, double *,
                                                 hipStream_t);
template hipError_t launch_stream_mapped<float>(const Geometry &, const MappedTables &, const float *, float *,
                                                hipStream_t);

}  // namespace sllbm
