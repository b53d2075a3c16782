// Adjoint tiles of 64 rows: 8 rows per wavefront.
#include "kadjw.hpp"

namespace gem {

hipError_t launch_adj2d_wg1(const AdjWArgs &a, int mat, hipStream_t st) { return adj_go<8, 8, 2, 2>(a, mat, st); }

}  // namespace gem
