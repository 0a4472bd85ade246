// rkl_block_f64.hip -- the one-stage kernel of small 3-D grids, flux precision FP64.
#include "rkl_block.h"

namespace rkl {
template hipError_t launch_block<double>(RKL_SHAPE_ARGS);
}  // namespace rkl
