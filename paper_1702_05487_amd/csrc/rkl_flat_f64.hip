// rkl_flat_f64.hip -- the 1-D and 2-D kernels, flux precision FP64.
#include "rkl_flat_kernel.h"

namespace rkl {
template hipError_t launch_flat_r<double>(const FlatLaunch&, hipStream_t, bool);
}  // namespace rkl
