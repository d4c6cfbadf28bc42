// Workgroup-wide in-plane kernels, vector FMA engine: F32C.
#include "wvl_xy_impl.h"

namespace wvl {
template void xy_launch_v<F32C, true>(const XyArgs&, int, int, size_t, hipStream_t);
template void xy_launch_v<F32C, false>(const XyArgs&, int, int, size_t, hipStream_t);
template void helm_launch_v<F32C>(const HelmArgs&, int, int, size_t, hipStream_t);
}  // namespace wvl
