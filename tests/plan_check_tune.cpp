// Check of the autotuner's trial lengths (host code only; built and run by
// test_plan_tune.py): whole passes of the candidate, the fewest that hold
// the steps asked for.
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
    printf("%d bad of %d\n", bad, runs);
    return bad != 0;
}
