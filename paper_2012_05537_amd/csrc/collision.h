// Node-local collision of the SLLBM (Eq. (5) with the quasi-equilibrium
// extension of App. D) for populations held in registers.
//
// Arithmetic layout (equal to the definitions term by term):
//  * Moments in double for both storage types (Eq. (7)); the set is centrally
//    symmetric, so each pair (xi, -xi) contributes s = h_i + h_-i to the even
//    moments and d = h_i - h_-i to the odd ones.
//  * T from 2 rho E = rho |u|^2 + 2 C_v rho T; P = rho T; Sutherland mu(T);
//    tau = mu/(P dt) + 1/2, tau_Pr = (tau - 1/2)/Pr + 1/2.
//  * Centred third moments Qbar[h] = sum h (xi-u)^3 from the raw moments
//    M0..M3 of h; Qbar[h^eq] = 0 identically, so Qbar^neq = Qbar[h].
//  * Equilibrium (Eq. (6), App. A/B) in scalar form: with c = xi.u,
//      f^eq = w rho (A0 + A1 c + A2 c^2 + c^3/6 + c^4/24),
//    A0..A2 depending on |u|^2, T - 1, the shell radius |xi|^2 and the
//    dimension D only (the traces of the Hermite tensors), and
//    g^eq = (2 C_v - D) T f^eq.
// Every function is generic over the lattice L (D3Q45 or D2Q19 traits of
// velset.h); in two dimensions the z components are absent.
//  * h* = (w/3!) Qbar : H^(3)(xi); odd in xi, so h*_-i = -h*_i.
//  * Relaxation h' = h + (h^eq - h)/tau + (1/tau - 1/tau_Pr) h*.
// In FP32-mixed storage (S = float) the populations are read and written in
// float once per collision and every operation in between is double: on
// gfx950 an unpacked float FMA issues at the rate of a double one, and the
// per-velocity polynomial in float loses up to c^4/24 (about 50 at the
// outer shell and Mach 1.25) times its ulp to cancellation.
#pragma once

#include <hip/hip_runtime.h>

#include "sllbm_internal.h"
#include "velset.h"

namespace sllbm {

constexpr double SUTHERLAND_S = 0.40417;

// acc + c x for a coefficient c from the velocity-set tables.  After the loops
// over velocities are unrolled c is a compile-time constant, and the term is
// dropped where it is zero: an FMA with a literal zero is otherwise issued
// (x * 0 may be NaN or -0, so the compiler keeps it), 172 of them in the
// D3Q45 collision.  The result is the same except for the sign of a zero sum.
__device__ __forceinline__ double fma_nz(double c, double x, double acc)
{
    return c == 0.0 ? acc : fma(x, c, acc);
}

__device__ __forceinline__ double viscosity_of(const CollisionParams &cp, double T)
{
    if (cp.law == SLLBM_CONSTANT) return cp.mu_inf;
    return cp.mu_inf * (1.0 + SUTHERLAND_S) * T * sqrt(T) / (T + SUTHERLAND_S);
}

// Raw moments of one population array over the pairs (d = odd part, s =
// even part).  m2 in the 3-D component order xx xy xz yy yz zz (the z
// entries stay zero in two dimensions); m3 over the lattice's unique
// rank-3 components.
template <class L>
struct RawMoments {
    double m0, m1[3], m2[6], m3[L::NM3];
};

constexpr int IDX2[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};

template <class L>
__device__ __forceinline__ void clear_moments(RawMoments<L> &r)
{
    r.m0 = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) r.m1[k] = 0.0;
#pragma unroll
    for (int k = 0; k < 6; ++k) r.m2[k] = 0.0;
#pragma unroll
    for (int k = 0; k < L::NM3; ++k) r.m3[k] = 0.0;
}

// adds pair q, whose values are hi (velocity xi) and hj (velocity -xi)
template <class L>
__device__ __forceinline__ void add_pair_moments(RawMoments<L> &r, int q, double hi, double hj)
{
    const int i = L::PAIRS.a[q];
    const double s = hi + hj, d = hi - hj;
    const double *x = L::T.xi[i];
    r.m0 += s;
#pragma unroll
    for (int a = 0; a < L::D; ++a) r.m1[a] = fma_nz(x[a], d, r.m1[a]);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        if (IDX2[k][1] < L::D) r.m2[k] = fma_nz(x[IDX2[k][0]] * x[IDX2[k][1]], s, r.m2[k]);
#pragma unroll
    for (int m = 0; m < L::NM3; ++m) r.m3[m] = fma_nz(L::H3.mono[i][m], d, r.m3[m]);
}

// x is computed here.  Without it the compiler moves sums that are used only
// after the branch on the viscosity law past that branch, with all their
// inputs live until then.
__device__ __forceinline__ void pin(double &x) { asm volatile("" : "+v"(x)); }

template <class L>
__device__ __forceinline__ void pin_moments(RawMoments<L> &r)
{
    pin(r.m0);
#pragma unroll
    for (int k = 0; k < L::D; ++k) pin(r.m1[k]);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        if (IDX2[k][1] < L::D) pin(r.m2[k]);
#pragma unroll
    for (int k = 0; k < L::NM3; ++k) pin(r.m3[k]);
}

template <class L, class Get>
__device__ __forceinline__ RawMoments<L> raw_moments_of(Get &&h)
{
    RawMoments<L> r;
    clear_moments<L>(r);
    r.m0 = static_cast<double>(h(0));
#pragma unroll
    for (int q = 0; q < L::NPAIR; ++q)
        add_pair_moments<L>(r, q, static_cast<double>(h(L::PAIRS.a[q])), static_cast<double>(h(L::PAIRS.b[q])));
    return r;
}

template <class L, typename S>
__device__ __forceinline__ RawMoments<L> raw_moments(const S (&h)[L::Q])
{
    return raw_moments_of<L>([&](int i) { return h[i]; });
}

// index of (a, b) in the 6 unique components xx xy xz yy yz zz
__host__ __device__ constexpr int sym2(int a, int b)
{
    return (a > b) ? sym2(b, a) : (a == 0 ? b : (a == 1 ? 2 + b : 5));
}

// Qbar_abc = M3 - sym3(u M2) + sym3(u u M1) - M0 u u u
template <class L>
__device__ __forceinline__ void centred_third(const RawMoments<L> &r, const double (&u)[3], double (&qb)[L::NM3])
{
#pragma unroll
    for (int m = 0; m < L::NM3; ++m) {
        const int a = L::IDX3[m][0], b = L::IDX3[m][1], c = L::IDX3[m][2];
        qb[m] = r.m3[m] - (u[a] * r.m2[sym2(b, c)] + u[b] * r.m2[sym2(a, c)] + u[c] * r.m2[sym2(a, b)]) +
                (u[a] * u[b] * r.m1[c] + u[a] * u[c] * r.m1[b] + u[b] * u[c] * r.m1[a]) - r.m0 * u[a] * u[b] * u[c];
    }
}

struct EqShell {
    double a0, a1, a2;
};

// Hermite series to fourth order contracted in the scalar invariants
// c = xi.u, |u|^2, |xi|^2 and theta = T - 1; the traces of H^(n) bring in
// D, D + 2 and D + 4 (for D = 3: x2 - 3, x2 - 5, x2 - 7, x2^2 - 10 x2 + 15).
template <int D>
__host__ __device__ __forceinline__ EqShell eq_shell(double u2, double th, double x2)
{
    constexpr double d0 = D, d2 = D + 2, d4 = D + 4;
    EqShell e;
    e.a0 = 1.0 - 0.5 * u2 + 0.5 * th * (x2 - d0) + 0.125 * u2 * u2 - 0.25 * th * u2 * (x2 - d2) +
           0.125 * th * th * (x2 * x2 - 2.0 * d2 * x2 + d0 * d2);
    e.a1 = 1.0 - 0.5 * u2 + 0.5 * th * (x2 - d2);
    e.a2 = 0.5 - 0.25 * u2 + 0.25 * th * (x2 - d4);
    return e;
}

// What the relaxation of one population at one node needs besides its values.
template <class L>
struct RelaxCoef {
    double om, kap;          // 1/tau, 1/tau - 1/tau_Pr
    double eqs;              // h^eq = eqs f^eq: 1 (f), (2 C_v - D) T (g)
    double rho, u2, th;      // density, |u|^2, T - 1
    double u[3];
    double qb[L::NM3];       // Qbar of the population
};

// From the raw moments rm of the population, and rho, momentum J and K = 2 rho E
// of the node.
template <class L>
__device__ __forceinline__ RelaxCoef<L> relax_coef(const RawMoments<L> &rm, double rho, const double (&J)[3], double K,
                                                   bool is_g, const CollisionParams &cp)
{
    constexpr bool D3 = L::D == 3;
    RelaxCoef<L> c;
    const double ir = 1.0 / rho;
    c.rho = rho;
    c.u[0] = J[0] * ir;
    c.u[1] = J[1] * ir;
    c.u[2] = D3 ? J[2] * ir : 0.0;
    c.u2 = D3 ? c.u[0] * c.u[0] + c.u[1] * c.u[1] + c.u[2] * c.u[2] : c.u[0] * c.u[0] + c.u[1] * c.u[1];
    const double T = (K * ir - c.u2) / (2.0 * cp.Cv);
    centred_third<L>(rm, c.u, c.qb);
    const double P = rho * T;
    const double tau = viscosity_of(cp, T) / (P * cp.dt) + 0.5;
    const double tau_pr = (tau - 0.5) * cp.inv_pr + 0.5;
    c.om = 1.0 / tau;
    c.kap = 1.0 / tau - 1.0 / tau_pr;
    c.th = T - 1.0;
    c.eqs = is_g ? cp.beta * T : 1.0;
    return c;
}

// relaxed value of the rest velocity
template <class L>
__device__ __forceinline__ double relax_rest(const RelaxCoef<L> &c, double v)
{
    const EqShell e = eq_shell<L::D>(c.u2, c.th, L::SHELL_X2[0]);
    const double heq = c.eqs * L::T.w[0] * (e.a0 * c.rho);
    return fma(c.om, heq - v, v);
}

// relaxed values of pair q (vi, vj in, replaced); A: rho times the shell's
// coefficients, rho6 = rho / 6, rho24 = rho / 24
template <class L>
__device__ __forceinline__ void relax_pair(const RelaxCoef<L> &k, const EqShell &A, double rho6, double rho24, int q,
                                           double &vi, double &vj)
{
    const int i = L::PAIRS.a[q];
    double c = fma_nz(L::T.xi[i][1], k.u[1], L::T.xi[i][0] == 0.0 ? 0.0 : L::T.xi[i][0] * k.u[0]);
    if constexpr (L::D == 3) c = fma_nz(L::T.xi[i][2], k.u[2], c);
    const double c2 = c * c;
    const double even = fma(c2, fma(c2, rho24, A.a2), A.a0);
    const double odd = c * fma(c2, rho6, A.a1);
    const double we = k.eqs * L::T.w[i];
    double hs = 0.0;
#pragma unroll
    for (int m = 0; m < L::NM3; ++m) hs = fma_nz(L::H3.c[i][m], k.qb[m], hs);
    vi = fma(k.kap, hs, fma(k.om, fma(we, even, we * odd) - vi, vi));
    vj = fma(-k.kap, hs, fma(k.om, fma(we, even, -we * odd) - vj, vj));
}

template <class L>
__device__ __forceinline__ EqShell rho_shell(const RelaxCoef<L> &k, int s)
{
    EqShell e = eq_shell<L::D>(k.u2, k.th, L::SHELL_X2[s]);
    e.a0 *= k.rho;
    e.a1 *= k.rho;
    e.a2 *= k.rho;
    return e;
}

// Collision of one node whose two populations are held by a lane pair,
// lanes l and l ^ XM: the lane with is_g = false holds f, its partner g.
// Each lane forms the raw moments of its own population; the pair exchanges
// rho, j, and the energy parts (tr M2[f] and M0[g]); each lane then builds
// Qbar of its own population and relaxes it (g^eq = (2 C_v - D) T f^eq).
// Both lanes of a pair must be active.
// get(i) returns the pre-collision value of velocity i (storage type S).  It
// is called twice per velocity, for the moments and for the relaxation, with
// fence() in between: a source in memory is then read again rather than held
// in registers through the collision.
// sink(i, value) receives every post-collision value as soon as it is formed.
// PIN: the moments are finished before the branch on the viscosity law.
template <class L, typename S, int XM = 1, bool PIN = false, class Get, class Fence, class Sink>
__device__ __forceinline__ void collide_core(Get &&get, Fence &&fence, bool is_g, const CollisionParams &cp,
                                             Sink &&sink)
{
    constexpr bool D3 = L::D == 3;
    RawMoments<L> rm = raw_moments_of<L>(get);
    if constexpr (PIN) pin_moments<L>(rm);
    fence();
    const double ktr = D3 ? rm.m2[0] + rm.m2[3] + rm.m2[5] : rm.m2[0] + rm.m2[3];
    const double p_m0 = __shfl_xor(rm.m0, XM);
    const double p_j0 = __shfl_xor(rm.m1[0], XM);
    const double p_j1 = __shfl_xor(rm.m1[1], XM);
    const double p_j2 = D3 ? __shfl_xor(rm.m1[2], XM) : 0.0;
    const double p_tr = __shfl_xor(ktr, XM);
    const double rho = is_g ? p_m0 : rm.m0;
    const double J[3] = {is_g ? p_j0 : rm.m1[0], is_g ? p_j1 : rm.m1[1], is_g ? p_j2 : rm.m1[2]};
    const double K = is_g ? p_tr + rm.m0 : ktr + p_m0;          // 2 rho E
    const RelaxCoef<L> k = relax_coef<L>(rm, rho, J, K, is_g, cp);
    EqShell A[L::NSHELL];
#pragma unroll
    for (int s = 1; s < L::NSHELL; ++s) A[s] = rho_shell<L>(k, s);
    const double rho6 = rho / 6.0, rho24 = rho / 24.0;
    sink(0, static_cast<S>(relax_rest<L>(k, static_cast<double>(get(0)))));
#pragma unroll
    for (int q = 0; q < L::NPAIR; ++q) {
        const int i = L::PAIRS.a[q], j = L::PAIRS.b[q];
        double vi = get(i), vj = get(j);
        relax_pair<L>(k, A[L::T.shell[i]], rho6, rho24, q, vi, vj);
        sink(i, static_cast<S>(vi));
        sink(j, static_cast<S>(vj));
    }
}

// The same on values held in registers: sink(i, value) receives every
// post-collision value as soon as it is formed, and v holds them all on
// return as well.
template <class L, typename S, bool PIN = false, class Sink>
__device__ __forceinline__ void collide_half_s(S (&v)[L::Q], bool is_g, const CollisionParams &cp, Sink &&sink)
{
    collide_core<L, S, 1, PIN>([&](int i) { return v[i]; }, [] {}, is_g, cp, [&](int i, S x) {
        v[i] = x;
        sink(i, x);
    });
}

template <class L, typename S, bool PIN = false>
__device__ __forceinline__ void collide_half(S (&v)[L::Q], bool is_g, const CollisionParams &cp)
{
    collide_half_s<L, S, PIN>(v, is_g, cp, [](int, S) {});
}

}  // namespace sllbm
