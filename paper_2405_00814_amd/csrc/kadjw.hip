// Dispatch of the adjoint workgroup tiles (kadjw.hpp); size class 1 is
// compiled in kadjw1.hip.
#include "kadjw.hpp"

namespace gem {

hipError_t launch_adj2d_wg1(const AdjWArgs &a, int mat, hipStream_t st);

hipError_t launch_adj2d_wg(const AdjWArgs &a, int cls, int mat, hipStream_t st) {
    if (a.ntiles <= 0 || a.nsteps <= 0) return hipSuccess;
    if (mat < 0 || mat > 2) return hipErrorInvalidValue;
    if (cls == 0) return adj_go<4, 8, 4, 2>(a, mat, st);
    if (cls == 1) return launch_adj2d_wg1(a, mat, st);
    return hipErrorInvalidValue;
}

}  // namespace gem
