// Plane kernel instantiations: F64, isolated along axis 2.
#include "wvl_line.h"

namespace wvl {
template hipError_t line_launch<F64, LINE_HPSI, true, 2>(int, const XyArgs&, int, int, size_t, hipStream_t);
template hipError_t line_launch<F64, LINE_RHO, true, 2>(int, const XyArgs&, int, int, size_t, hipStream_t);
template hipError_t line_launch<F64, LINE_HELM, true, 2>(int, const XyArgs&, int, int, size_t, hipStream_t);
}  // namespace wvl
