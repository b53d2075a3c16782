// Tiles of 96 / 80 / 64 rows (by the number of coefficient maps) for grids
// with many tiles per CU: as many rows as 128 registers hold, so that four
// workgroups share a CU and one's loads overlap the others' arithmetic.
#include "k2dw.hpp"

namespace gem {

hipError_t launch_2d_wg2(const WgArgs &a, int mat, int xt, hipStream_t st) {
    if (mat == 0) return wg_go<24, 14, 10, 4, 4, 0>(a, xt, st);
    if (mat == 1) return wg_go<20, 12, 9, 4, 4, 1>(a, xt, st);
    if (mat == 2) return wg_go<16, 10, 8, 4, 4, 2>(a, xt, st);
    return wg_go<20, 12, 9, 4, 4, 3>(a, xt, st);
}

}  // namespace gem
