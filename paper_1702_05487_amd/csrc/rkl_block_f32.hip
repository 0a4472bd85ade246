// rkl_block_f32.hip -- the one-stage kernel of small 3-D grids, flux precision FP32 (mixed).
#include "rkl_block.h"

namespace rkl {
template hipError_t launch_block<float>(RKL_SHAPE_ARGS);
}  // namespace rkl
