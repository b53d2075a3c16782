// Dispatch of the 2D workgroup-tile kernel (k2dw.hpp) over its size classes,
// each compiled in a file of its own.
#include "common.hpp"

namespace gem {

hipError_t launch_2d_wg0(const WgArgs &a, int mat, int xt, hipStream_t st);
hipError_t launch_2d_wg1(const WgArgs &a, int mat, int xt, hipStream_t st);
hipError_t launch_2d_wg2(const WgArgs &a, int mat, int xt, hipStream_t st);

hipError_t launch_2d_wg(const WgArgs &a, int cls, int mat, int xt, hipStream_t st) {
    if (a.ntiles <= 0 || a.nsteps <= 0) return hipSuccess;
    if (mat < 0 || mat > 3 || xt < 0 || xt > 2) return hipErrorInvalidValue;
    if (cls == 0) return launch_2d_wg0(a, mat, xt, st);
    if (cls == 1) return launch_2d_wg1(a, mat, xt, st);
    if (cls == 2) return launch_2d_wg2(a, mat, xt, st);
    return hipErrorInvalidValue;
}

}  // namespace gem
