// Check of the autotuner's trial lengths and of the fewest steps of a pass
// (host code only; built and run by test_plan_tune.py): trials are whole
// passes of the candidate, the fewest that hold the steps asked for; only
// grids of at most 32 rows with more than two tiles per CU wait for longer
// passes, the longer the fewer their rows and the more their tiles.
#include <cstdio>

#include "common.hpp"
using namespace gem;

int main() {
    int bad = 0, runs = 0;
    auto check = [&](int ndim, int variant, int tb, int per) {
        for (int trial = 2; trial < 70; ++trial) {
            fdtd_kernel_config k{};
            k.variant = variant;
            k.tile[0] = 64;
            k.tile[2] = tb;
            const int n = trial_steps_of(k, ndim, trial);
            bad += n % per != 0 || n < trial || n >= trial + per;
            ++runs;
        }
    };
    for (int tb : {2, 4, 8, 10, 12, 14}) check(2, 3, tb, tb);
    for (int v : {1, 2, 4}) check(2, v, 0, 1);
    check(3, 3, 16, 2);
    check(3, 2, 16, 1);
    for (int nx : {3, 4, 8, 12, 20, 32, 33, 100})
        for (int t : {1, 256, 512, 513, 1000, 2000, 4000, 8000, 100000}) {
            const int k = wg2d_least(nx, t, 256);
            bad += k < 2 || k > 16 || ((nx > 32 || t <= 512) && k != 2) || wg2d_least(nx + 1, t, 256) > k ||
                   (t > 512 && nx <= 3 && wg2d_least(nx, 2 * t, 256) < k);
            ++runs;
        }
    bad += wg2d_least(3, 2000, 256) < 4 || wg2d_least(8, 2000, 256) != 3 || wg2d_least(16, 2000, 256) != 2;
    printf("%d bad of %d\n", bad, runs);
    return bad != 0;
}
