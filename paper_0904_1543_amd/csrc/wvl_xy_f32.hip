// Workgroup-wide in-plane kernels, vector FMA engine: F32.
#include "wvl_xy_impl.h"

namespace wvl {
template void xy_launch_v<F32, true>(const XyArgs&, int, int, size_t, hipStream_t);
template void xy_launch_v<F32, false>(const XyArgs&, int, int, size_t, hipStream_t);
template void helm_launch_v<F32>(const HelmArgs&, int, int, size_t, hipStream_t);
}  // namespace wvl
