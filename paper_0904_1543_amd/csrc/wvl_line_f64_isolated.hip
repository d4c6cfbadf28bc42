// Plane kernel instantiations: F64, isolated along both in-plane axes.
#include "wvl_line.h"

namespace wvl {
template hipError_t line_launch<F64, LINE_HPSI, true, 3>(int, const XyArgs&, int, int, size_t, hipStream_t);
template hipError_t line_launch<F64, LINE_RHO, true, 3>(int, const XyArgs&, int, int, size_t, hipStream_t);
template hipError_t line_launch<F64, LINE_HELM, true, 3>(int, const XyArgs&, int, int, size_t, hipStream_t);
}  // namespace wvl
