// 64-row tiles: 8 rows per wavefront.
#include "k2dw.hpp"

namespace gem {

hipError_t launch_2d_wg1(const WgArgs &a, int mat, int xt, hipStream_t st) {
    if (mat == 0) return wg_go<8, 8, 8, 8, 4, 0>(a, xt, st);
    if (mat == 1) return wg_go<8, 8, 8, 8, 4, 1>(a, xt, st);
    if (mat == 2) return wg_go<8, 8, 8, 8, 4, 2>(a, xt, st);
    return wg_go<8, 8, 8, 8, 4, 3>(a, xt, st);
}

}  // namespace gem
