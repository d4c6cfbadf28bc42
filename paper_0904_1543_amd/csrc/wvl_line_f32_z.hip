// z passes with whole lines in LDS, F32: W, W^T and K along z.
#include "wvl_line_z.h"

namespace wvl {
template hipError_t line_z_launch<F32, ZL_CW>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
template hipError_t line_z_launch<F32, ZL_CWT>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
template hipError_t line_z_launch<F32, ZL_CK>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
}  // namespace wvl
