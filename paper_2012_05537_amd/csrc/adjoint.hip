// Reverse mode of the SLLBM step (kernels and launchers).
//
// One step maps the pre-collision state X_n to X_{n+1} = S(C(X_n)), with C
// the node-local collision (Eq. (5) with App. D) and S the semi-Lagrangian
// streaming (Eq. (9)), which is linear.  Its vector-Jacobian product is
//   lambda_n = J_C(X_n)^T S^T lambda_{n+1}.
// S^T is the transposed streaming (stream.hip, stream_graded.hip,
// stream_mapped.hip); this file
// holds the collision VJP, the VJP of the equilibrium initialisation, and the
// flow functional used for gradients with its derivative.  All reverse arithmetic is
// in double; states are stored in the context's storage type.
//
// Collision VJP (per node, f on the even lane of a pair, g on the odd lane).
// With adjoints alpha_i of the post-collision values of the lane's population
// (alpha = a for f, b for g) and the forward quantities recomputed from X_n:
//   h'_i = h_i + omega (s h^eq_i - h_i) + kappa h*_i,  s = 1 (f), beta T (g),
//   omega = 1/tau, kappa = 1/tau - 1/tau_Pr,
// the reverse sweep accumulates, per lane, the scalars
//   sum alpha (s h^eq - h)            -> d omega
//   sum alpha h*                      -> d kappa
//   sum alpha s h^eq omega / rho      -> d rho
//   equilibrium terms in c = xi.u, |u|^2 and theta = T - 1 -> d u, d T
//   Abar_m = kappa sum_i alpha_i H3c_im  (adjoint of Qbar) -> d h, d u
// adds them over the pair, pushes them through tau(mu(T), P = rho T),
// T = (K/rho - |u|^2)/(2 C_v) and u = J/rho, and forms per velocity
//   lambda_f,k = (1 - omega) a_k + rho_bar + J_bar . xi_k + K_bar |xi_k|^2 + Abar_f : d_k^3
//   lambda_g,k = (1 - omega) b_k + K_bar + Abar_g : d_k^3,   d_k = xi_k - u.
// The node's contribution to dL/dmu_inf is mu_bar * (mu / mu_inf).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "collision.h"
#include "dma.h"
#include "nt.h"
#include "sllbm_internal.h"
#include "velset.h"
#include "xcd.h"

namespace sllbm {

namespace {

template <int XM>
__device__ __forceinline__ double pair_sum(double v) { return v + __shfl_xor(v, XM); }

__device__ __forceinline__ double viscosity_factor(const CollisionParams &cp, double T, double &dfac_dT)
{
    if (cp.law == SLLBM_CONSTANT) {
        dfac_dT = 0.0;
        return 1.0;
    }
    // (1 + S) T^1.5 / (T + S)
    const double sq = sqrt(T);
    const double den = T + SUTHERLAND_S;
    const double fac = (1.0 + SUTHERLAND_S) * T * sq / den;
    dfac_dT = (1.0 + SUTHERLAND_S) * (1.5 * sq / den - T * sq / (den * den));
    return fac;
}

// bracket b(c) = a0 + a1 c + a2 c^2 + c^3/6 + c^4/24 and its derivatives in
// |u|^2 and theta; d a1/d|u|^2 = -1/2, d a2/d|u|^2 = -1/4, d a1/d theta =
// (x2 - 5)/2 and d a2/d theta = (x2 - 7)/4 are constants of the shell
struct Bracket {
    double a0, a1, a2;           // value coefficients
    double d0u;                  // d a0 / d |u|^2
    double d0t;                  // d a0 / d theta
};

__device__ __forceinline__ Bracket bracket(double u2, double th, double x2)
{
    Bracket b;
    const EqShell e = eq_shell<3>(u2, th, x2);
    b.a0 = e.a0;
    b.a1 = e.a1;
    b.a2 = e.a2;
    b.d0u = -0.5 + 0.25 * u2 - 0.25 * th * (x2 - 5.0);
    b.d0t = 0.5 * (x2 - 3.0) - 0.25 * u2 * (x2 - 5.0) + 0.25 * th * (x2 * x2 - 10.0 * x2 + 15.0);
    return b;
}

constexpr double D1U = -0.5, D2U = -0.25;
__host__ __device__ constexpr double d1t_of(double x2) { return 0.5 * (x2 - 5.0); }
__host__ __device__ constexpr double d2t_of(double x2) { return 0.25 * (x2 - 7.0); }

__device__ __forceinline__ double bval(const Bracket &b, double c)
{
    return fma(c, fma(c, fma(c, fma(c, 1.0 / 24.0, 1.0 / 6.0), b.a2), b.a1), b.a0);
}

__device__ __forceinline__ double bder(const Bracket &b, double c)    // d b / d c
{
    return fma(c, fma(c, fma(c, 1.0 / 6.0, 0.5), 2.0 * b.a2), b.a1);
}

}  // namespace

// ---------------------------------------------------------------------------
// Collision VJP: lam = J_C(X)^T mu, two lanes per node.  dmu_part[block]
// receives the block's sum of dL/dmu_inf.
// ---------------------------------------------------------------------------
// alpha of a lane in registers
struct AlphaReg {
    double v[vs::Q];
    __device__ __forceinline__ double operator()(int i) const { return v[i]; }
    __device__ __forceinline__ void refresh(double &) { __builtin_amdgcn_sched_barrier(0); }
};

// alpha of a lane in LDS (velocity i at base[i * NB + off]).  refresh(x) makes
// the compiler read it again afterwards, and not before x is known, instead
// of holding 45 values in registers through the sweep.
template <typename S, int NB>
struct AlphaLds {
    const S *base;
    int off;
    __device__ __forceinline__ double operator()(int i) const { return static_cast<double>(base[i * NB + off]); }
    __device__ __forceinline__ void refresh(double &x)
    {
        asm volatile("" : "+v"(off), "+v"(x));
        __builtin_amdgcn_sched_barrier(0);
    }
};

// One lane of the collision VJP (its node's population is_g): X of the node
// from X + off (stride N), the lane's adjoint inputs alpha_i from AL(i), the
// partner lane l ^ XM; writes lambda of its population at lam + off (stride N)
// and returns the node's dL/dmu_inf (counted on the f lane).  Inactive lanes (a
// node past the end) compute on node 0 for their partner and write nothing.
// X is read in groups of pairs, and the sums over the velocities are pinned
// where they are formed, so that alpha (90 registers, or LDS) and the sums are
// all that lives through the sweep.
template <typename S, bool NTH, int XM, class Alpha>
__device__ __forceinline__ double collide_vjp_lane(int64_t N, const CollisionParams &cp, const S *__restrict__ X,
                                                   int64_t off, bool is_g, bool active, Alpha AL, S *lam)
{
    // X enters only through its raw moments and sum alpha h, so it is dead
    // before the sweep
    RawMoments<D3Q45> rm;
    double dot_ah;
    {
        // two groups of GP pairs in registers: the next group's loads are in
        // flight while a group is summed
        constexpr int GP = 8, NG = (22 + GP - 1) / GP;
        S h[2][2 * GP];
        auto load_group = [&](int g) {
#pragma unroll
            for (int k = 0; k < GP; ++k) {
                const int q = g * GP + k;
                if (q >= 22) continue;
                h[g & 1][2 * k] = load_hint<NTH>(&X[off + static_cast<int64_t>(vs::PAIRS.a[q]) * N]);
                h[g & 1][2 * k + 1] = load_hint<NTH>(&X[off + static_cast<int64_t>(vs::PAIRS.b[q]) * N]);
            }
        };
        const S h0 = load_hint<NTH>(&X[off]);
        load_group(0);
        clear_moments<D3Q45>(rm);
        rm.m0 = static_cast<double>(h0);
        dot_ah = AL(0) * static_cast<double>(h0);
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            asm volatile("" ::: "memory");
            if (g + 1 < NG) load_group(g + 1);
            AL.refresh(dot_ah);
#pragma unroll
            for (int k = 0; k < GP; ++k) {
                const int q = g * GP + k;
                if (q >= 22) continue;
                const double hi = static_cast<double>(h[g & 1][2 * k]), hj = static_cast<double>(h[g & 1][2 * k + 1]);
                add_pair_moments<D3Q45>(rm, q, hi, hj);
                dot_ah = fma(AL(vs::PAIRS.a[q]), hi, dot_ah);
                dot_ah = fma(AL(vs::PAIRS.b[q]), hj, dot_ah);
            }
        }
    }
    pin(dot_ah);
    pin_moments<D3Q45>(rm);
    AL.refresh(rm.m0);

    // ---- forward quantities (as in collide_half) ----
    const double ktr = rm.m2[0] + rm.m2[3] + rm.m2[5];
    const double p_m0 = __shfl_xor(rm.m0, XM);
    const double p_j0 = __shfl_xor(rm.m1[0], XM), p_j1 = __shfl_xor(rm.m1[1], XM), p_j2 = __shfl_xor(rm.m1[2], XM);
    const double p_tr = __shfl_xor(ktr, XM);
    const double rho = is_g ? p_m0 : rm.m0;
    const double J[3] = {is_g ? p_j0 : rm.m1[0], is_g ? p_j1 : rm.m1[1], is_g ? p_j2 : rm.m1[2]};
    const double ir = 1.0 / rho;
    const double u[3] = {J[0] * ir, J[1] * ir, J[2] * ir};
    const double K = is_g ? p_tr + rm.m0 : ktr + p_m0;
    const double u2 = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
    const double Cv = cp.Cv;
    const double T = (K * ir - u2) / (2.0 * Cv);
    double qb[10];
    centred_third<D3Q45>(rm, u, qb);
    const double th = T - 1.0;

    // centred second moment of the own population (for the Qbar -> u term);
    // the raw moments are dead after this
    double C2[6];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a; b < 3; ++b)
            C2[sym2(a, b)] = rm.m2[sym2(a, b)] - u[a] * rm.m1[b] - u[b] * rm.m1[a] + rm.m0 * u[a] * u[b];

    // ---- reverse sweep over the velocities (own population) ----
    // With b(c) = a0 + a1 c + a2 c^2 + c^3/6 + c^4/24 and, over the pairs of a
    // shell, S0 = sum s, S1 = sum d c, S2 = sum s c^2, S3 = sum d c^3,
    // S4 = sum s c^4 (s, d: sum and difference of the pair's alpha), the
    // shell adds w times
    //   a0 S0 + a1 S1 + a2 S2 + S3/6 + S4/24    to sum alpha b,
    //   its derivatives in |u|^2 and theta      to s_u2, s_th,
    //   xi (d o' + s e'), o' = a1 + c^2/2, e' = c (2 a2 + c^2/6), to ubar;
    // rho and the population's factor of f^eq come in at the end, and
    // sum alpha h* = sum_m abar_m Qbar_m needs no h* per velocity.
    double s_b, s_u2, s_th;
    double ubar[3] = {0, 0, 0};
    double abar[10];
#pragma unroll
    for (int m = 0; m < 10; ++m) abar[m] = 0.0;
    {   // rest velocity: c = 0, h* = 0
        const Bracket b = bracket(u2, th, vs::SHELL_X2[0]);
        const double wa = vs::T.w[0] * AL(0);
        s_b = wa * b.a0;
        s_u2 = wa * b.d0u;
        s_th = wa * b.d0t;
    }
#pragma unroll
    for (int s = 1; s < 4; ++s) {
        const Bracket b = bracket(u2, th, vs::SHELL_X2[s]);
        const double x2 = vs::SHELL_X2[s];
        double S0 = 0, S1 = 0, S2 = 0, S3 = 0, S4 = 0, g[3] = {0, 0, 0}, w = 0;
        const double two_a2 = 2.0 * b.a2;
#pragma unroll
        for (int q = 0; q < 22; ++q) {
            const int i = vs::PAIRS.a[q], j = vs::PAIRS.b[q];
            if (vs::T.shell[i] != s) continue;
            w = vs::T.w[i];
            const double c = fma_nz(vs::T.xi[i][2], u[2],
                                    fma_nz(vs::T.xi[i][1], u[1], vs::T.xi[i][0] == 0.0 ? 0.0 : vs::T.xi[i][0] * u[0]));
            const double ai = AL(i), aj = AL(j);
            const double sp = ai + aj, sm = ai - aj;
            const double c2 = c * c, d1 = sm * c, e2 = sp * c2;
            S0 += sp;
            S1 += d1;
            S2 += e2;
            S3 = fma(d1, c2, S3);
            S4 = fma(e2, c2, S4);
            const double gu = fma(sm, fma(c2, 0.5, b.a1), sp * (c * fma(c2, 1.0 / 6.0, two_a2)));
#pragma unroll
            for (int a = 0; a < 3; ++a) g[a] = fma_nz(vs::T.xi[i][a], gu, g[a]);
#pragma unroll
            for (int m = 0; m < 10; ++m) abar[m] = fma_nz(vs::H3.c[i][m], sm, abar[m]);
            if (q % 2 == 2 - 1) AL.refresh(S4);
        }
        s_b = fma(w, fma(b.a0, S0, fma(b.a1, S1, fma(b.a2, S2, fma(S3, 1.0 / 6.0, S4 * (1.0 / 24.0))))), s_b);
        s_u2 = fma(w, fma(b.d0u, S0, fma(D1U, S1, D2U * S2)), s_u2);
        s_th = fma(w, fma(b.d0t, S0, fma(d1t_of(x2), S1, d2t_of(x2) * S2)), s_th);
#pragma unroll
        for (int a = 0; a < 3; ++a) ubar[a] = fma(w, g[a], ubar[a]);
    }
    pin(s_b);
    pin(s_u2);
    pin(s_th);
#pragma unroll
    for (int a = 0; a < 3; ++a) pin(ubar[a]);
#pragma unroll
    for (int m = 0; m < 10; ++m) pin(abar[m]);
    const double P = rho * T;
    double dfac;
    const double fac = viscosity_factor(cp, T, dfac);
    const double mu_v = cp.mu_inf * fac;
    const double tau = mu_v / (P * cp.dt) + 0.5;
    const double tau_pr = (tau - 0.5) * cp.inv_pr + 0.5;
    const double om = 1.0 / tau;
    const double kap = 1.0 / tau - 1.0 / tau_pr;
    const double eqs = is_g ? cp.beta * T : 1.0;
    double s_ka = 0.0;
#pragma unroll
    for (int m = 0; m < 10; ++m) {
        s_ka = fma(abar[m], qb[m], s_ka);
        abar[m] *= kap;
    }
    const double s_eqT = rho * s_b, s_heq = eqs * s_eqT, re = rho * eqs;
    s_u2 *= re;
    s_th *= re;
#pragma unroll
    for (int a = 0; a < 3; ++a) ubar[a] *= re;

    // Qbar -> u: -sum_m abar_m (delta_ad C2_bc + delta_bd C2_ac + delta_cd C2_ab)
    double uq[3] = {0, 0, 0};
#pragma unroll
    for (int m = 0; m < 10; ++m) {
        const int a = vs::IDX3[m][0], b = vs::IDX3[m][1], c = vs::IDX3[m][2];
        uq[a] -= abar[m] * C2[sym2(b, c)];
        uq[b] -= abar[m] * C2[sym2(a, c)];
        uq[c] -= abar[m] * C2[sym2(a, b)];
    }

    // ---- pair totals (sum alpha (s h^eq - h) = s_heq - dot_ah) ----
    const double S_om = pair_sum<XM>(s_heq - dot_ah), S_ka = pair_sum<XM>(s_ka);
    const double S_heq = pair_sum<XM>(om * s_heq);
    const double S_eqT = pair_sum<XM>(is_g ? om * cp.beta * s_eqT : 0.0);
    const double S_u2 = pair_sum<XM>(om * s_u2), S_th = pair_sum<XM>(om * s_th);
    double U[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) U[a] = pair_sum<XM>(om * ubar[a] + uq[a]);

    // omega = 1/tau, kappa = 1/tau - 1/tau_pr
    const double om_bar = S_om + S_ka;
    const double ompr_bar = -S_ka;
    const double tau_bar = -om_bar / (tau * tau) - ompr_bar / (tau_pr * tau_pr) * cp.inv_pr;
    const double mu_bar = tau_bar / (P * cp.dt);
    const double P_bar = -tau_bar * mu_v / (P * P * cp.dt);
    double T_bar = mu_bar * cp.mu_inf * dfac + P_bar * rho + S_th + S_eqT;
    double rho_bar = P_bar * T + S_heq * ir;
    double ub[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) ub[a] = U[a] + 2.0 * u[a] * S_u2;
    // T = (K/rho - |u|^2) / (2 C_v)
    const double K_bar = T_bar / (2.0 * Cv * rho);
    rho_bar -= T_bar * K * ir * ir / (2.0 * Cv);
#pragma unroll
    for (int a = 0; a < 3; ++a) ub[a] -= T_bar * u[a] / Cv;
    // u = J / rho
    double J_bar[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) J_bar[a] = ub[a] * ir;
    rho_bar -= (ub[0] * u[0] + ub[1] * u[1] + ub[2] * u[2]) * ir;

    // ---- per-velocity outputs ----
    // Abar : (xi - u)^3 = T3 - T2 + T1 - T0 and Abar : (-xi - u)^3 = -(T3 + T2 + T1 + T0)
    // with T3 = Abar : xi xi xi, T2 = B : xi xi, T1 = C . xi, T0 = Abar : u u u,
    // where B and C collect Abar with one and two of its indices contracted
    // with u.  The pair's outputs are (1 - omega) alpha + E +- O with the even
    // part E = E0 + Ev : xi xi and the odd part O = Ov . xi + T3.
    if (active) {
        double Ev[6] = {0, 0, 0, 0, 0, 0}, Ov[3], T0 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            Ov[a] = is_g ? 0.0 : J_bar[a];
            Ev[sym2(a, a)] = is_g ? 0.0 : K_bar;
        }
#pragma unroll
        for (int m = 0; m < 10; ++m) {
            const int a = vs::IDX3[m][0], b = vs::IDX3[m][1], c = vs::IDX3[m][2];
            Ev[sym2(b, c)] = fma(-abar[m], u[a], Ev[sym2(b, c)]);
            Ev[sym2(a, c)] = fma(-abar[m], u[b], Ev[sym2(a, c)]);
            Ev[sym2(a, b)] = fma(-abar[m], u[c], Ev[sym2(a, b)]);
            const double bc = u[b] * u[c];
            Ov[a] = fma(abar[m], bc, Ov[a]);
            Ov[b] = fma(abar[m], u[a] * u[c], Ov[b]);
            Ov[c] = fma(abar[m], u[a] * u[b], Ov[c]);
            T0 = fma(abar[m], u[a] * bc, T0);
        }
        int64_t so = off;
        asm volatile("" : "+v"(so));      // fresh store addresses (the load addresses are not kept live)
        AL.refresh(T0);
        S *lp = lam + so;
        const double one_m = 1.0 - om;
        double E0 = (is_g ? K_bar : rho_bar) - T0;
        store_hint<NTH>(&lp[0], static_cast<S>(fma(one_m, AL(0), E0)));      // rest velocity: xi = 0
#pragma unroll
        for (int q = 0; q < 22; ++q) {
            const int i = vs::PAIRS.a[q], j = vs::PAIRS.b[q];
            const double *x = vs::T.xi[i];
            double E = E0, O = 0.0;
#pragma unroll
            for (int k = 0; k < 6; ++k) E = fma_nz(x[IDX2[k][0]] * x[IDX2[k][1]], Ev[k], E);
#pragma unroll
            for (int a = 0; a < 3; ++a) O = fma_nz(x[a], Ov[a], O);
#pragma unroll
            for (int m = 0; m < 10; ++m) O = fma_nz(vs::H3.mono[i][m], abar[m], O);
            store_hint<NTH>(&lp[static_cast<int64_t>(i) * N], static_cast<S>(fma(one_m, AL(i), E + O)));
            const double rj = fma(one_m, AL(j), E - O);
            store_hint<NTH>(&lp[static_cast<int64_t>(j) * N], static_cast<S>(rj));
            if (q % 2 == 2 - 1) AL.refresh(E0);
        }
    }

    // ---- dL/dmu_inf: mu = mu_inf * fac, counted once per node (f lane) ----
    return active && !is_g ? mu_bar * fac : 0.0;
}

// sum of the block's 256 values in thread 0's red[0], in a fixed order
__device__ __forceinline__ double block_sum256(double v, double *red)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    return red[0];
}

// One lane pair per node, alpha in registers; no grid-stride loop, out of
// which the compiler would hoist the sweep's FP64 constants (230 SGPR
// spills).  mu and lam may be the same buffer: each lane reads its 45 values
// before writing them.  255 VGPRs and 4 more spilled, 2 waves per SIMD; in FP64 6.78 ms at 256^3
// nodes (36.2 GB, 5.3 TB/s: HBM-bound), 114 us at 64^3 (175 us with 332
// registers and one wave per SIMD).
// NTH: non-temporal loads and stores (states larger than the Infinity Cache)
template <typename S, bool NTH>
__global__ void __launch_bounds__(256, 2) k_collide_vjp(int64_t N, CollisionParams cp, const S *__restrict__ X,
                                                     const S *mu, S *lam, double *__restrict__ dmu_part)
{
    __shared__ double red[256];
    const int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    const int64_t n = t >> 1;
    const int pop = static_cast<int>(t & 1);
    const bool active = n < N;
    const int64_t off = static_cast<int64_t>(pop) * vs::Q * N + (active ? n : 0);
    AlphaReg al;
#pragma unroll
    for (int i = 0; i < vs::Q; ++i) al.v[i] = static_cast<double>(load_hint<NTH>(&mu[off + static_cast<int64_t>(i) * N]));
    const double dmu = collide_vjp_lane<S, NTH, 1>(N, cp, X, off, pop != 0, active, al, lam);
    if (dmu_part) {
        const double s = block_sum256(dmu, red);
        if (threadIdx.x == 0) dmu_part[blockIdx.x] = s;
    }
}

// The collision VJP with the adjoint inputs alpha staged in LDS: a block takes
// NB = 512 / sizeof(S) consecutive nodes (blocks in XCD order), copies their
// 90 rows of mu (row r = pop * 45 + i, 512 contiguous bytes) into LDS by
// DMA (stage_rows; WIDE: 16-byte copies, for aligned rows), and each lane reads
// its alpha_i from there (lane l of
// wave w: node w * 32 + (l & 31), population l >> 5, partner l ^ 32).
// mu and lam may be the same buffer (every copy has landed before the block's
// first write).
// Bound by HBM: it reads X and alpha and writes lambda once, 3.53 ms at 256^3
// nodes in FP32 (18.1 GB, 5.1 TB/s; 166 VGPRs and 6 more spilled, 3 waves per SIMD), 451 us at
// 128^3 and 63 us at 64^3.  While the sweep's sums sank past the branch on the
// viscosity law it needed 256 VGPRs (2 waves) and took 5.73 ms.
template <typename S, bool NTH, bool WIDE>
__global__ void __launch_bounds__(1024 / sizeof(S), sizeof(S) == 4 ? 3 : 2) k_collide_vjp_lds(int64_t N, CollisionParams cp,
                                                            const S *__restrict__ X, const S *mu, S *lam,
                                                            double *__restrict__ dmu_part)
{
    constexpr int NB = 512 / sizeof(S), ROWS = 2 * vs::Q, NW = NB / 32;
    __shared__ S tile[ROWS][NB];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int pop = lane >> 5;
    const int c = w * 32 + (lane & 31);
    const int64_t nb = static_cast<int64_t>(xcd_linear(blockIdx.x, gridDim.x)) * NB;
    stage_rows<S, ROWS, NB, NW, WIDE, NTH>(N, nb, mu, tile, w, lane);
    __syncthreads();                             // the other waves' copies too
    const int64_t n = nb + c;
    const bool active = n < N;
    const int64_t off = static_cast<int64_t>(pop) * vs::Q * N + (active ? n : 0);
    const double dmu = collide_vjp_lane<S, NTH, 32>(N, cp, X, off, pop != 0, active,
                                                    AlphaLds<S, NB>{&tile[0][0], pop * vs::Q * NB + c}, lam);
    if (dmu_part) {
        __syncthreads();                         // the tile's reads are done: its memory takes the sums
        double *red = reinterpret_cast<double *>(&tile[0][0]);
        red[threadIdx.x] = dmu;
        __syncthreads();
        for (int s = 2 * NB / 2; s > 0; s >>= 1) {
            if (static_cast<int>(threadIdx.x) < s) red[threadIdx.x] += red[threadIdx.x + s];
            __syncthreads();
        }
        if (threadIdx.x == 0) dmu_part[blockIdx.x] = red[0];
    }
}

// Fixed-order sum of n block partials by one block of 256 threads; the
// result is added to *acc (add != 0) or stored there.  Deterministic.
__global__ void __launch_bounds__(256) k_accumulate(const double *__restrict__ part, int n, double *__restrict__ acc,
                                                    int add)
{
    __shared__ double red[256];
    // eight interleaved running sums per thread (eight loads in flight), combined in a fixed order
    double a[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int b = threadIdx.x;
    for (; b + 7 * 256 < n; b += 8 * 256) {
#pragma unroll
        for (int k = 0; k < 8; ++k) a[k] += part[b + k * 256];
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
        if (b + k * 256 < n) a[k] += part[b + k * 256];
    const double s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    red[threadIdx.x] = s;
    __syncthreads();
    for (int k = 128; k > 0; k >>= 1) {
        if (threadIdx.x < k) red[threadIdx.x] += red[threadIdx.x + k];
        __syncthreads();
    }
    if (threadIdx.x == 0) *acc = add ? *acc + red[0] : red[0];
}

// ---------------------------------------------------------------------------
// VJP of the equilibrium initialisation: fields -> (f^eq, g^eq)
// ---------------------------------------------------------------------------
template <typename S>
__global__ void __launch_bounds__(256) k_init_vjp(int64_t N, CollisionParams cp, const double *__restrict__ rho,
                                                  const double *__restrict__ u, const double *__restrict__ T,
                                                  const S *__restrict__ lam, double *__restrict__ drho,
                                                  double *__restrict__ du, double *__restrict__ dT)
{
    const int64_t n = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (n >= N) return;
    const double r = rho[n], uu[3] = {u[n], u[N + n], u[2 * N + n]}, Tn = T[n];
    const double u2 = uu[0] * uu[0] + uu[1] * uu[1] + uu[2] * uu[2];
    const double th = Tn - 1.0;
    const double bT = cp.beta * Tn;
    double gr = 0, gu[3] = {0, 0, 0}, gu2 = 0, gt = 0;
#pragma unroll
    for (int i = 0; i < vs::Q; ++i) {
        const double a = static_cast<double>(lam[static_cast<int64_t>(i) * N + n]);
        const double b = static_cast<double>(lam[static_cast<int64_t>(vs::Q + i) * N + n]);
        const Bracket br = bracket(u2, th, vs::T.x2[i]);
        const double c = vs::T.xi[i][0] * uu[0] + vs::T.xi[i][1] * uu[1] + vs::T.xi[i][2] * uu[2];
        const double w = vs::T.w[i];
        const double e = a + bT * b;                       // adjoint of f^eq_i (through f and g)
        const double bv = bval(br, c);
        gr += e * w * bv;
        const double gc = e * w * r * bder(br, c);
        gu[0] = fma(gc, vs::T.xi[i][0], gu[0]);
        gu[1] = fma(gc, vs::T.xi[i][1], gu[1]);
        gu[2] = fma(gc, vs::T.xi[i][2], gu[2]);
        const double x2 = vs::T.x2[i];
        gu2 += e * w * r * (br.d0u + c * D1U + c * c * D2U);
        gt += e * w * r * (br.d0t + c * d1t_of(x2) + c * c * d2t_of(x2)) + b * cp.beta * w * r * bv;
    }
    if (drho) drho[n] = gr;
    if (du) {
        du[n] = gu[0] + 2.0 * uu[0] * gu2;
        du[N + n] = gu[1] + 2.0 * uu[1] * gu2;
        du[2 * N + n] = gu[2] + 2.0 * uu[2] * gu2;
    }
    if (dT) dT[n] = gt;
}

// ---------------------------------------------------------------------------
// VJP of the moments (Eq. (7) with 2 rho E = rho |u|^2 + 2 C_v rho T): given
// adjoints of rho, u, T at every node, lam = d(rho, u, T)/d(state)^T (...).
// ---------------------------------------------------------------------------
template <typename S>
__global__ void __launch_bounds__(256) k_moments_vjp(int64_t N, CollisionParams cp, const S *__restrict__ st,
                                                     const double *__restrict__ drho, const double *__restrict__ du,
                                                     const double *__restrict__ dT, S *__restrict__ lam)
{
    const int64_t n = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (n >= N) return;
    double r = 0, j[3] = {0, 0, 0}, K = 0;
#pragma unroll
    for (int i = 0; i < vs::Q; ++i) {
        const double f = static_cast<double>(st[static_cast<int64_t>(i) * N + n]);
        const double g = static_cast<double>(st[static_cast<int64_t>(vs::Q + i) * N + n]);
        r += f;
        j[0] = fma(f, vs::T.xi[i][0], j[0]);
        j[1] = fma(f, vs::T.xi[i][1], j[1]);
        j[2] = fma(f, vs::T.xi[i][2], j[2]);
        K += fma(f, vs::T.x2[i], g);
    }
    const double ir = 1.0 / r;
    const double u[3] = {j[0] * ir, j[1] * ir, j[2] * ir};
    const double Tb = dT ? dT[n] : 0.0;
    double rb = drho ? drho[n] : 0.0;
    double ub[3] = {du ? du[n] : 0.0, du ? du[N + n] : 0.0, du ? du[2 * N + n] : 0.0};
    // T = (K/rho - |u|^2) / (2 C_v)
    const double Kb = Tb / (2.0 * cp.Cv * r);
    rb -= Tb * K * ir * ir / (2.0 * cp.Cv);
#pragma unroll
    for (int a = 0; a < 3; ++a) ub[a] -= Tb * u[a] / cp.Cv;
    // u = J / rho
    rb -= (ub[0] * u[0] + ub[1] * u[1] + ub[2] * u[2]) * ir;
    const double Jb[3] = {ub[0] * ir, ub[1] * ir, ub[2] * ir};
#pragma unroll
    for (int i = 0; i < vs::Q; ++i) {
        lam[static_cast<int64_t>(i) * N + n] = static_cast<S>(rb + Jb[0] * vs::T.xi[i][0] + Jb[1] * vs::T.xi[i][1] +
                                                              Jb[2] * vs::T.xi[i][2] + Kb * vs::T.x2[i]);
        lam[static_cast<int64_t>(vs::Q + i) * N + n] = static_cast<S>(Kb);
    }
}

// ---------------------------------------------------------------------------
// Flow functional L = sum over cells of the tensor Clenshaw-Curtis quadrature
// of (1/2) rho |u|^2 + (div u)^2, div u from each cell's own polynomial.
// ---------------------------------------------------------------------------
template <typename S>
__global__ void __launch_bounds__(256) k_rho_u(int64_t N, const S *__restrict__ st, double *__restrict__ rho,
                                               double *__restrict__ u)
{
    const int64_t n = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (n >= N) return;
    double r = 0, j[3] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < vs::Q; ++i) {
        const double f = static_cast<double>(st[static_cast<int64_t>(i) * N + n]);
        r += f;
        j[0] = fma(f, vs::T.xi[i][0], j[0]);
        j[1] = fma(f, vs::T.xi[i][1], j[1]);
        j[2] = fma(f, vs::T.xi[i][2], j[2]);
    }
    rho[n] = r;
    u[n] = j[0] / r;
    u[N + n] = j[1] / r;
    u[2 * N + n] = j[2] / r;
}

struct CellGeo {
    int N[3], nel[3], p;
    int64_t nodes;
    double h[3];                 // cell width per axis (equal cells)
    const double *hw;            // graded mesh: widths of the x, then y, then z cells (NULL: equal cells)
    const double *jac;           // distorted mesh: per cell point J^-1 (row-major) and |det J| (NULL: J = I)
    const double *full_w;        // distorted mesh: per-node quadrature weights (NULL: separable weights)
};

// width of cell e along axis a
__device__ __forceinline__ double cell_h(const CellGeo &g, int a, int e)
{
    if (!g.hw) return g.h[a];
    const int off = a == 0 ? 0 : (a == 1 ? g.nel[0] : g.nel[0] + g.nel[1]);
    return g.hw[off + e];
}

__device__ __forceinline__ int64_t node_of(const CellGeo &g, int gx, int gy, int gz)
{
    gx %= g.N[0];
    gy %= g.N[1];
    gz %= g.N[2];
    return (static_cast<int64_t>(gz) * g.N[1] + gy) * g.N[0] + gx;
}

// per cell point: partial loss; sdiv[c] = 2 W_c div_c (for the gradient)
__global__ void __launch_bounds__(256) k_loss_cells(CellGeo g, const double *__restrict__ dmat,
                                                    const double *__restrict__ ccw, const double *__restrict__ rho,
                                                    const double *__restrict__ u, double *__restrict__ sdiv,
                                                    double *__restrict__ part)
{
    __shared__ double red[256];
    const int p = g.p, p1 = p + 1;
    const int64_t ncp = static_cast<int64_t>(g.nel[0]) * g.nel[1] * g.nel[2] * p1 * p1 * p1;
    double acc = 0.0;
    for (int64_t c = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; c < ncp;
         c += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int64_t r = c;
        const int kx = static_cast<int>(r % p1); r /= p1;
        const int ky = static_cast<int>(r % p1); r /= p1;
        const int kz = static_cast<int>(r % p1); r /= p1;
        const int ex = static_cast<int>(r % g.nel[0]); r /= g.nel[0];
        const int ey = static_cast<int>(r % g.nel[1]);
        const int ez = static_cast<int>(r / g.nel[1]);
        const int gx = ex * p + kx, gy = ey * p + ky, gz = ez * p + kz;
        const double hx = cell_h(g, 0, ex), hy = cell_h(g, 1, ey), hz = cell_h(g, 2, ez);
        double div = 0.0;
        double W = (0.5 * hx * ccw[kx]) * (0.5 * hy * ccw[ky]) * (0.5 * hz * ccw[kz]);
        if (!g.jac) {
            for (int m = 0; m <= p; ++m) {
                div += dmat[kx * p1 + m] * u[node_of(g, ex * p + m, gy, gz)] / hx;
                div += dmat[ky * p1 + m] * u[g.nodes + node_of(g, gx, ey * p + m, gz)] / hy;
                div += dmat[kz * p1 + m] * u[2 * g.nodes + node_of(g, gx, gy, ez * p + m)] / hz;
            }
        } else {
            // distorted cell: div u = sum_ab (d u_a / d r_b) (J^-1)_ba
            double gr[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
            for (int m = 0; m <= p; ++m) {
                const int64_t nx = node_of(g, ex * p + m, gy, gz), ny = node_of(g, gx, ey * p + m, gz),
                              nz = node_of(g, gx, gy, ez * p + m);
                const double dx = dmat[kx * p1 + m] / hx, dy = dmat[ky * p1 + m] / hy, dz = dmat[kz * p1 + m] / hz;
                for (int a = 0; a < 3; ++a) {
                    gr[a][0] = fma(dx, u[a * g.nodes + nx], gr[a][0]);
                    gr[a][1] = fma(dy, u[a * g.nodes + ny], gr[a][1]);
                    gr[a][2] = fma(dz, u[a * g.nodes + nz], gr[a][2]);
                }
            }
            const double *Ji = g.jac + c * 10;
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) div = fma(gr[a][b], Ji[b * 3 + a], div);
            W *= Ji[9];
        }
        const int64_t n = node_of(g, gx, gy, gz);
        const double ux = u[n], uy = u[g.nodes + n], uz = u[2 * g.nodes + n];
        acc += W * (0.5 * rho[n] * (ux * ux + uy * uy + uz * uz) + div * div);
        if (sdiv) sdiv[c] = 2.0 * W * div;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

// TGV diagnostics (Sec. III C) per cell point: (1/2) rho |u|^2, mu(T) |curl u|^2
// and (4/3) mu(T) (div u)^2, derivatives from the cell's own polynomial,
// weighted by the tensor Clenshaw-Curtis rule; per-block partial sums.
__global__ void __launch_bounds__(256) k_diag_cells(CellGeo g, CollisionParams cp, const double *__restrict__ dmat,
                                                    const double *__restrict__ ccw, const double *__restrict__ rho,
                                                    const double *__restrict__ u, const double *__restrict__ T,
                                                    double *__restrict__ part)
{
    __shared__ double red[3][256];
    const int p = g.p, p1 = p + 1;
    const int64_t ncp = static_cast<int64_t>(g.nel[0]) * g.nel[1] * g.nel[2] * p1 * p1 * p1;
    double acc[3] = {0.0, 0.0, 0.0};
    for (int64_t c = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; c < ncp;
         c += static_cast<int64_t>(gridDim.x) * blockDim.x) {
        int64_t r = c;
        int k[3], e[3];
        k[0] = static_cast<int>(r % p1); r /= p1;
        k[1] = static_cast<int>(r % p1); r /= p1;
        k[2] = static_cast<int>(r % p1); r /= p1;
        e[0] = static_cast<int>(r % g.nel[0]); r /= g.nel[0];
        e[1] = static_cast<int>(r % g.nel[1]);
        e[2] = static_cast<int>(r / g.nel[1]);
        const int gx = e[0] * p + k[0], gy = e[1] * p + k[1], gz = e[2] * p + k[2];
        const double hx = cell_h(g, 0, e[0]), hy = cell_h(g, 1, e[1]), hz = cell_h(g, 2, e[2]);
        double grad[3][3];                       // grad[a][b] = d u_a / d x_b
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) grad[a][b] = 0.0;
        for (int m = 0; m <= p; ++m) {
            const int64_t nx = node_of(g, e[0] * p + m, gy, gz);
            const int64_t ny = node_of(g, gx, e[1] * p + m, gz);
            const int64_t nz = node_of(g, gx, gy, e[2] * p + m);
            const double dx = dmat[k[0] * p1 + m] / hx, dy = dmat[k[1] * p1 + m] / hy,
                         dz = dmat[k[2] * p1 + m] / hz;
            for (int a = 0; a < 3; ++a) {
                grad[a][0] = fma(dx, u[a * g.nodes + nx], grad[a][0]);
                grad[a][1] = fma(dy, u[a * g.nodes + ny], grad[a][1]);
                grad[a][2] = fma(dz, u[a * g.nodes + nz], grad[a][2]);
            }
        }
        double W = (0.5 * hx * ccw[k[0]]) * (0.5 * hy * ccw[k[1]]) * (0.5 * hz * ccw[k[2]]);
        if (g.jac) {
            // distorted cell: physical gradient (d u / d r) J^-1, weight times |det J|
            const double *Ji = g.jac + c * 10;
            double gp[3][3];
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b)
                    gp[a][b] = grad[a][0] * Ji[b] + grad[a][1] * Ji[3 + b] + grad[a][2] * Ji[6 + b];
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) grad[a][b] = gp[a][b];
            W *= Ji[9];
        }
        const int64_t n = node_of(g, gx, gy, gz);
        const double w0 = grad[2][1] - grad[1][2], w1 = grad[0][2] - grad[2][0], w2 = grad[1][0] - grad[0][1];
        const double div = grad[0][0] + grad[1][1] + grad[2][2];
        const double ux = u[n], uy = u[g.nodes + n], uz = u[2 * g.nodes + n];
        const double mu = viscosity_of(cp, T[n]);
        acc[0] = fma(W, 0.5 * rho[n] * (ux * ux + uy * uy + uz * uz), acc[0]);
        acc[1] = fma(W, mu * (w0 * w0 + w1 * w1 + w2 * w2), acc[1]);
        acc[2] = fma(W, (4.0 / 3.0) * mu * div * div, acc[2]);
    }
    for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s)
            for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) part[blockIdx.x * 3 + q] = red[q][0];
}

// Fixed-order sum of n partial triples by one block (deterministic).
__global__ void __launch_bounds__(256) k_sum3(const double *__restrict__ part, int n, double *__restrict__ out)
{
    __shared__ double red[3][256];
    double acc[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < n; b += 256)
        for (int q = 0; q < 3; ++q) acc[q] += part[b * 3 + q];
    for (int q = 0; q < 3; ++q) red[q][threadIdx.x] = acc[q];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s)
            for (int q = 0; q < 3; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 3; ++q) out[q] = red[q][0];
}

// dL/d(state) at every node: dL/drho and dL/du gathered from the cell points
// whose value or derivative stencil contains the node, then chained through
// rho = sum f and u = sum f xi / rho (g does not enter L).
template <typename S>
__global__ void __launch_bounds__(256) k_loss_grad(CellGeo g, const double *__restrict__ dmat,
                                                   const double *__restrict__ nodew, const double *__restrict__ rho,
                                                   const double *__restrict__ u, const double *__restrict__ sdiv,
                                                   S *__restrict__ lam)
{
    const int64_t n = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (n >= g.nodes) return;
    const int p = g.p, p1 = p + 1;
    const int gi[3] = {static_cast<int>(n % g.N[0]), static_cast<int>((n / g.N[0]) % g.N[1]),
                       static_cast<int>(n / (static_cast<int64_t>(g.N[0]) * g.N[1]))};
    const double W = g.full_w ? g.full_w[n] : nodew[gi[0]] * nodew[g.N[0] + gi[1]] * nodew[g.N[0] + g.N[1] + gi[2]];
    const double r = rho[n];
    const double uu[3] = {u[n], u[g.nodes + n], u[2 * g.nodes + n]};
    double du[3];
    // the cell (and local index) containing node index gi along an axis: own cell, and
    // for a cell end point also the previous cell with local index p
    int ce[3][2], ck[3][2], nopt[3];
    for (int a = 0; a < 3; ++a) {
        const int e = gi[a] / p, l = gi[a] % p;
        ce[a][0] = e;
        ck[a][0] = l;
        nopt[a] = 1;
        if (l == 0) {
            ce[a][1] = (e - 1 + g.nel[a]) % g.nel[a];
            ck[a][1] = p;
            nopt[a] = 2;
        }
    }
    // component a of u enters div u at the cell points whose derivative
    // stencil along axis d holds the node: on undistorted cells only d = a,
    // on distorted cells every d, with the factor (J^-1)_da of the point
    for (int a = 0; a < 3; ++a) {
        double s = 0.0;
        for (int d = 0; d < 3; ++d) {
            if (!g.jac && d != a) continue;
            const int b = (d + 1) % 3, c = (d + 2) % 3;
            for (int od = 0; od < nopt[d]; ++od)           // cell along d and the node's index in it
                for (int ob = 0; ob < nopt[b]; ++ob)
                    for (int oc = 0; oc < nopt[c]; ++oc)
                        for (int kd = 0; kd <= p; ++kd) {    // cell point along d
                            int E[3], kk[3];
                            E[d] = ce[d][od];
                            kk[d] = kd;
                            E[b] = ce[b][ob];
                            kk[b] = ck[b][ob];
                            E[c] = ce[c][oc];
                            kk[c] = ck[c][oc];
                            const int64_t cp =
                                ((static_cast<int64_t>(E[2]) * g.nel[1] + E[1]) * g.nel[0] + E[0]) * (p1 * p1 * p1) +
                                (kk[2] * p1 + kk[1]) * p1 + kk[0];
                            double f = dmat[kd * p1 + ck[d][od]] / cell_h(g, d, E[d]);
                            if (g.jac) f *= g.jac[cp * 10 + d * 3 + a];
                            s += sdiv[cp] * f;
                        }
        }
        du[a] = r * uu[a] * W + s;
    }
    const double drho = 0.5 * (uu[0] * uu[0] + uu[1] * uu[1] + uu[2] * uu[2]) * W -
                        (du[0] * uu[0] + du[1] * uu[1] + du[2] * uu[2]) / r;
    const double dj[3] = {du[0] / r, du[1] / r, du[2] / r};
#pragma unroll
    for (int i = 0; i < vs::Q; ++i) {
        lam[static_cast<int64_t>(i) * g.nodes + n] =
            static_cast<S>(drho + dj[0] * vs::T.xi[i][0] + dj[1] * vs::T.xi[i][1] + dj[2] * vs::T.xi[i][2]);
        lam[static_cast<int64_t>(vs::Q + i) * g.nodes + n] = static_cast<S>(0);
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

static CellGeo cell_geo(const Geometry &g, const double *hh, const double *hw, const double *jac = nullptr,
                        const double *full_w = nullptr)
{
    CellGeo c;
    for (int a = 0; a < 3; ++a) {
        c.N[a] = g.N[a];
        c.nel[a] = g.nel[a];
        c.h[a] = hh[a];
    }
    c.hw = hw;
    c.jac = jac;
    c.full_w = full_w;
    c.p = g.p;
    c.nodes = g.nodes;
    return c;
}

template <typename S>
hipError_t Launch<S>::loss(const Geometry &g, const S *state, const double *dmat, const double *ccw, const double *h,
                           const double *hw, const double *cjac, double *scratch_rho, double *scratch_u,
                           double *partials, int nblocks, double *out1, hipStream_t st)
{
    const unsigned nb = static_cast<unsigned>((g.nodes + 255) / 256);
    hipLaunchKernelGGL((k_rho_u<S>), dim3(nb), dim3(256), 0, st, g.nodes, state, scratch_rho, scratch_u);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_loss_cells, dim3(nblocks), dim3(256), 0, st, cell_geo(g, h, hw, cjac), dmat, ccw,
                       scratch_rho, scratch_u, static_cast<double *>(nullptr), partials);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_accumulate, dim3(1), dim3(256), 0, st, partials, nblocks, out1, 0);
    return hipGetLastError();
}

template <typename S>
hipError_t Launch<S>::loss_grad(const Geometry &g, const S *state, const double *dmat, const double *ccw,
                                const double *nodew, const double *h, const double *hw, const double *cjac,
                                const double *full_w, double *scratch_rho, double *scratch_u, double *scratch_div,
                                double *partials, int nblocks, S *lam, hipStream_t st)
{
    const unsigned nb = static_cast<unsigned>((g.nodes + 255) / 256);
    hipLaunchKernelGGL((k_rho_u<S>), dim3(nb), dim3(256), 0, st, g.nodes, state, scratch_rho, scratch_u);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const CellGeo cg = cell_geo(g, h, hw, cjac, full_w);
    hipLaunchKernelGGL(k_loss_cells, dim3(nblocks), dim3(256), 0, st, cg, dmat, ccw, scratch_rho, scratch_u,
                       scratch_div, partials);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_loss_grad<S>), dim3(nb), dim3(256), 0, st, cg, dmat, nodew, scratch_rho, scratch_u,
                       scratch_div, lam);
    return hipGetLastError();
}

template <typename S>
hipError_t Launch<S>::diagnostics(const Geometry &g, const CollisionParams &cp, const S *state, const double *dmat,
                                  const double *ccw, const double *h, const double *hw, const double *cjac,
                                  double *scratch_rho, double *scratch_u, double *scratch_T, double *partials,
                                  int nblocks, double *out3, hipStream_t st)
{
    hipError_t e = moments(g, cp, state, scratch_rho, scratch_u, scratch_T, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_diag_cells, dim3(nblocks), dim3(256), 0, st, cell_geo(g, h, hw, cjac), cp, dmat, ccw,
                       scratch_rho, scratch_u, scratch_T, partials);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_sum3, dim3(1), dim3(256), 0, st, partials, nblocks, out3);
    return hipGetLastError();
}

template <typename S>
hipError_t Launch<S>::collide_vjp(const Geometry &g, const CollisionParams &cp, const S *state_n, S *lam,
                                  double *dmu_partials, double *dmu, hipStream_t st)
{
    // lam <- J_C(X_n)^T lam in place
    const int64_t plane = g.nodes * static_cast<int64_t>(sizeof(S));
    const bool nt = use_nontemporal(90 * plane, plane);
    int blocks = 0;
    // alpha staged in LDS (see k_collide_vjp_lds): in FP32 always; in FP64 it
    // leaves 1.5 waves per SIMD, which is faster while the grid has at most one
    // block per CU (10.3 against 12.4 us at 512 nodes, 11.4 against 14.2 at
    // 13,824; the adjoint step at 16,250 nodes 24.9 us either way, at 17,576 29.9 and
    // 25.4, at 32,768 31.8 and 29.5).  Rows that are not 16-byte
    // aligned are staged by words on large FP32 grids (adjoint step at 63^3 nodes
    // 112 -> 102 us, 129^3 1032 -> 948, 45^3 equal, 39 x 33 x 27 27.4 -> 29.4), otherwise not.
    const bool wide = g.nodes % (16 / sizeof(S)) == 0 && reinterpret_cast<uintptr_t>(lam) % 16 == 0;
    if (wide ? sizeof(S) == 4 || g.nodes <= 16384 : sizeof(S) == 4 && g.nodes > 65536) {
        constexpr int NB = 512 / sizeof(S);
        blocks = static_cast<int>((g.nodes + NB - 1) / NB);
        auto launch = [&](auto nth, auto wd) {
            hipLaunchKernelGGL((k_collide_vjp_lds<S, decltype(nth)::value, decltype(wd)::value>),
                               dim3(static_cast<unsigned>(blocks)), dim3(2 * NB), 0, st, g.nodes, cp, state_n, lam, lam,
                               dmu ? dmu_partials : nullptr);
        };
        if constexpr (sizeof(S) == 4) {
            if (!wide) launch(std::false_type(), std::false_type());
            else if (nt) launch(std::true_type(), std::true_type());
            else launch(std::false_type(), std::true_type());
        } else {
            launch(std::false_type(), std::true_type());
        }
    } else {
        blocks = static_cast<int>((2 * g.nodes + 255) / 256);
        auto launch = [&](auto nth) {
            hipLaunchKernelGGL((k_collide_vjp<S, decltype(nth)::value>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                               st, g.nodes, cp, state_n, lam, lam, dmu ? dmu_partials : nullptr);
        };
        // (FP32: only small grids come here)
        if constexpr (sizeof(S) == 4) {
            launch(std::false_type());
        } else {
            if (nt) launch(std::true_type());
            else launch(std::false_type());
        }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (dmu) {
        hipLaunchKernelGGL(k_accumulate, dim3(1), dim3(256), 0, st, dmu_partials, blocks, dmu, 1);
        e = hipGetLastError();
    }
    return e;
}

template <typename S>
hipError_t Launch<S>::init_equilibrium_vjp(const Geometry &g, const CollisionParams &cp, const double *rho,
                                           const double *u, const double *T, const S *lam0, double *drho, double *du,
                                           double *dT, hipStream_t st)
{
    const unsigned nb = static_cast<unsigned>((g.nodes + 255) / 256);
    hipLaunchKernelGGL((k_init_vjp<S>), dim3(nb), dim3(256), 0, st, g.nodes, cp, rho, u, T, lam0, drho, du, dT);
    return hipGetLastError();
}

template <typename S>
hipError_t Launch<S>::moments_vjp(const Geometry &g, const CollisionParams &cp, const S *state, const double *drho,
                                  const double *du, const double *dT, S *lam, hipStream_t st)
{
    const unsigned nb = static_cast<unsigned>((g.nodes + 255) / 256);
    hipLaunchKernelGGL((k_moments_vjp<S>), dim3(nb), dim3(256), 0, st, g.nodes, cp, state, drho, du, dT, lam);
    return hipGetLastError();
}

template struct Launch<double>;
template struct Launch<float>;

}  // namespace sllbm
