// z passes with whole lines in LDS, F32C: W, W^T and K along z.
#include "wvl_line_z.h"

namespace wvl {
template hipError_t line_z_launch<F32C, ZL_CW>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
template hipError_t line_z_launch<F32C, ZL_CWT>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
template hipError_t line_z_launch<F32C, ZL_CK>(int, const PassGeom&, const ZLineArgs&, int, hipStream_t);
}  // namespace wvl
