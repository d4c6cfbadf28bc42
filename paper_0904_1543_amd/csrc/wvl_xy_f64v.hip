// Workgroup-wide in-plane kernels, vector FMA engine: F64.
#include "wvl_xy_impl.h"

namespace wvl {
template void xy_launch_v<F64, true>(const XyArgs&, int, int, size_t, hipStream_t);
template void xy_launch_v<F64, false>(const XyArgs&, int, int, size_t, hipStream_t);
template void helm_launch_v<F64>(const HelmArgs&, int, int, size_t, hipStream_t);
}  // namespace wvl
