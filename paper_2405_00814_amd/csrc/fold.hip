// Material maps to update coefficients, in FP64 and rounded once:
//   e = eps0 eps_r, h = sigma dt / (2 e): Ca = (1 - h)/(1 + h),
//   Cb = (dt/e)/(1 + h); Db = dt/(mu0 mu_r).
// Creating a batch of 16 grids of 256 to 900 squared takes 14.6 ms with the
// fold here and one block per axis for its tables, 25 with the fold on the
// host and 18 blocks a problem.  Bound by the upload of the maps.
#include "sim.hpp"

namespace gem {

__global__ __launch_bounds__(256) void k_fold(float *cb, float *ca, float *db, int eps, int64_t n, double dt) {
#pragma clang fp contract(off)
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= n) return;
    const double er = eps ? (double)cb[c] : 1.0, sg = ca ? (double)ca[c] : 0.0;
    const double e = kEps0 * er;
    const double h = sg * dt / (2.0 * e);
    cb[c] = (float)((dt / e) / (1.0 + h));
    if (ca) ca[c] = (float)((1.0 - h) / (1.0 + h));
    if (db) db[c] = (float)(dt / (kMu0 * (double)db[c]));
}

hipError_t launch_fold(float *cb, float *ca, float *db, bool eps, int64_t n, double dt, hipStream_t st) {
    const int64_t nb = (n + 255) / 256;
    if (n <= 0 || nb > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_fold, dim3((unsigned)nb), dim3(256), 0, st, cb, ca, db, eps ? 1 : 0, n, dt);
    return hipGetLastError();
}

}  // namespace gem
