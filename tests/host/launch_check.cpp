// Host-logic checks of how the streaming kernels are dealt to blocks; argv[1]
// names the check.  Prints what is wrong and exits non-zero on failure.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include "sllbm_internal.h"
using namespace sllbm;

static int fail(const char *what, const int n[3], int p)
{
    std::printf("%s: %d x %d x %d cells, p = %d\n", what, n[0], n[1], n[2], p);
    return 1;
}

// every grid of up to 60 million nodes has a launch of the streaming by departure
// cell, with less than 2^32 threads along each grid dimension
static int run_grids()
{
    const int sides[] = {1, 2, 3, 7, 16, 61, 200, 611, 900, 3000};
    for (int p = 3; p <= 6; ++p)
        for (int a : sides)
            for (int b : sides)
                for (int c : sides) {
                    const int n[3] = {a, b, c};
                    if (static_cast<int64_t>(a) * b * c * p * p * p > 60000000) continue;
                    for (size_t elem : {sizeof(float), sizeof(double)}) {
                        unsigned runs = 0;
                        const MappedRuns r = mapped_runs(p, a, elem);
                        if (!mapped_run_grid(r, n, runs)) return fail("no launch", n, p);
                        if (runs != static_cast<int64_t>(r.nx) * b * c || static_cast<int64_t>(runs) * 256 >> 32)
                            return fail("grid", n, p);
                    }
                }
    return 0;
}

int main(int argc, char **argv)
{
    if (argc == 2 && !std::strcmp(argv[1], "run_grids")) return run_grids();
    std::printf("unknown check\n");
    return 1;
}
