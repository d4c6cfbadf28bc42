// z passes with whole lines in LDS, F64: the last z step and the preconditioner's z pass.
#include "wvl_line_z.h"

namespace wvl {
template hipError_t line_z_launch<F64, ZL_FINAL>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
template hipError_t line_z_launch<F64, ZL_CG>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
}  // namespace wvl
