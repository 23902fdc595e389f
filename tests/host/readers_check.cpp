// Host-logic check of the departures by source cell (graded meshes): for 60
// random graded or equal axes (p = 1..6, shifts up to several cells) the outputs
// first[c] .. first[c + 1] - 1 must be those that depart into cell c, each output
// once, and the transposed weights by cell, gathered as the transposed kernel
// gathers them (both groups, surplus readers clamped to the last one), must be
// the exact transpose of the forward rows.  Exits non-zero on failure.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>
#include "sllbm_internal.h"
using namespace sllbm;
int main()
{
    VelocitySet vs;
    build_velocity_set(vs);
    std::mt19937_64 rng(5);
    std::uniform_real_distribution<double> U(-1, 1);
    double worst = 0;
    int most_seen = 0, empty = 0;
    for (int trial = 0; trial < 60; ++trial) {
        const int p = 1 + trial % 6, ne = 1 + (trial * 7) % 11, N = ne * p;
        const double L = 2.0 + trial % 3, dt = 0.05 + 0.3 * (trial % 5);
        std::vector<double> faces;
        if (trial % 4 != 0) {
            faces.push_back(0);
            double sum = 0;
            std::vector<double> w(ne);
            for (auto &x : w) { x = 1 + 0.85 * U(rng); sum += x; }
            for (auto x : w) faces.push_back(faces.back() + x * L / sum);
            faces.back() = L;
        }
        std::vector<int32_t> src, first;
        std::vector<double> w, tw;
        build_node_tables(vs, p, ne, L, faces, trial % 3, dt, src, w);
        const int most = build_cell_readers(N, p, src, first);
        build_cell_weights(N, p, most, first, w, tw);
        most_seen = std::max(most_seen, most);
        auto wrap = [&](int x) { return ((x % N) + N) % N; };
        for (int i = 0; i < Q; ++i) {
            const int32_t *s = &src[i * N], *f = &first[i * (ne + 1)];
            std::vector<double> S(N * N, 0.0), T(N * N, 0.0);
            std::vector<int> seen(N, 0);
            for (int g = 0; g < N; ++g)
                for (int k = 0; k <= p; ++k) S[g * N + wrap(s[g] + k)] += w[(i * N + g) * (p + 1) + k];
            if (f[ne] != f[0] + N) return std::printf("period %d\n", trial), 1;
            for (int c = 0; c < ne; ++c) {
                if (f[c + 1] < f[c] || f[c + 1] - f[c] > most) return std::printf("order %d\n", trial), 1;
                empty += f[c + 1] == f[c];
                for (int g = f[c]; g < f[c + 1]; ++g) {
                    ++seen[wrap(g)];
                    if (wrap(s[wrap(g)]) != c * p) return std::printf("cell %d\n", trial), 1;
                }
                // as in the kernel
                const int r1 = f[c], m1 = f[c + 1] - r1;
                const int r0 = c > 0 ? f[c - 1] : f[ne - 1] - N, m0 = r1 - r0;
                const double *o = &tw[(static_cast<size_t>(i) * ne + c) * most * (p + 1)];
                for (int j = 0; j < most; ++j) {
                    const int a = wrap(r1 + std::min(j, std::max(m1 - 1, 0)));
                    const int b = wrap(r0 + std::min(j, std::max(m0 - 1, 0)));
                    for (int k = 0; k < p; ++k) T[(c * p + k) * N + a] += o[j * (p + 1) + k];
                    T[c * p * N + b] += o[j * (p + 1) + p];
                }
            }
            for (int g = 0; g < N; ++g)
                if (seen[g] != 1) return std::printf("coverage %d\n", trial), 1;
            for (int g = 0; g < N; ++g)
                for (int m = 0; m < N; ++m) worst = std::max(worst, std::fabs(S[g * N + m] - T[m * N + g]));
        }
    }
    std::printf("max |S^T - T| = %.3e, most readers %d, empty cells %d\n", worst, most_seen, empty);
    return worst < 1e-14 && empty > 0 ? 0 : 1;
}
