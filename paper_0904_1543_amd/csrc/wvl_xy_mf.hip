// Workgroup-wide in-plane kernels, float64 matrix-core engine.
#include "wvl_xy_impl.h"

namespace wvl {
template void xy_launch_m<true>(const XyArgs&, int, int, size_t, hipStream_t);
template void xy_launch_m<false>(const XyArgs&, int, int, size_t, hipStream_t);
void helm_launch_mf(const HelmArgs& a, int mt, int nblocks, size_t lds, hipStream_t st) {
  helm_launch_m(a, mt, nblocks, lds, st);
}
}  // namespace wvl
