// rkl_flat_f32.hip -- the 1-D and 2-D kernels, flux precision FP32 (mixed).
#include "rkl_flat_kernel.h"

namespace rkl {
template hipError_t launch_flat_r<float>(const FlatLaunch&, hipStream_t, bool);
}  // namespace rkl
