// Plane kernel instantiations: F64, LINE_HELM, groups of orbitals or one plane per tile.
#include "wvl_line.h"

namespace wvl {
template hipError_t line_launch<F64, LINE_HELM, true, 0>(int, const XyArgs&, int, int, size_t, hipStream_t);
template hipError_t line_launch<F64, LINE_HELM, false, 0>(int, const XyArgs&, int, int, size_t, hipStream_t);
}  // namespace wvl
