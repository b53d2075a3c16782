// What a simulation does once before it steps: coefficients, cleared state.
//
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

// Clears arrays in one launch: a reset, 64 steps and the read-out of a 32^2
// grid took 127 us with a memset of each array, 100 with this; 250^2, 1024
// steps 1.37 ms, 1.30.  Bound by the launch.
__global__ __launch_bounds__(256) void k_zero_parts(ZeroParts z) {
    int64_t b = blockIdx.x;
    int q = 0;
    while (q < z.count && b >= (z.n[q] + 4095) / 4096) b -= (z.n[q++] + 4095) / 4096;
    if (q >= z.count) return;
    float *const d = z.p[q];
    const int64_t n = z.n[q], a = b * 4096, e = a + 4096 < n ? a + 4096 : n;
    if (((uintptr_t)d & 15) == 0 && e == a + 4096) {
#pragma unroll
        for (int u = 0; u < 4; ++u) *(float4 *)(d + a + 1024 * u + 4 * (int)threadIdx.x) = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (int64_t k = a + threadIdx.x; k < e; k += 256) d[k] = 0.f;
    }
}

hipError_t launch_zero_parts(const ZeroParts &z, hipStream_t st) {
    int64_t nb = 0;
    for (int q = 0; q < z.count; ++q) nb += (z.n[q] + 4095) / 4096;
    if (nb == 0) return hipSuccess;
    if (nb > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_zero_parts, dim3((unsigned)nb), dim3(256), 0, st, z);
    return hipGetLastError();
}

}  // namespace gem
