// Dispatch of the 1D pass kernels by precision (the device code is in
// wvl_passes_impl.h, instantiated per precision by wvl_passes_<prec>.hip).

#include "wvl_kernels.h"
#include "wvl_plane.h"

namespace wvl {

template <int P>
hipError_t launch_op(int op, int axis, const PassGeom& g, int ntiles, const void* in, void* out,
                     const void* k0, int64_t plane, double kmul, double* epart, hipStream_t st);
template <int P>
hipError_t zfinal_p(const PassGeom& g, int ntiles, const void* t, const void* c, const void* kxy,
                    void* out, int64_t plane, double kmul, double* epart, hipStream_t st);

template <int P>
hipError_t cg_z_p(const PassGeom& g, int ntiles, const void* r, const void* pold, void* pnew, void* q,
                  const double* eps, const void* sc, int64_t plane, double* epart, double* ppart,
                  hipStream_t st);

hipError_t launch_cg_z(int prec, const PassGeom& g, int ntiles, const void* r, const void* pold,
                       void* pnew, void* q, const double* eps, const void* sc, int64_t plane,
                       double* epart, double* ppart, hipStream_t st) {
  switch (prec) {
    case F64: return cg_z_p<F64>(g, ntiles, r, pold, pnew, q, eps, sc, plane, epart, ppart, st);
    case F32: return cg_z_p<F32>(g, ntiles, r, pold, pnew, q, eps, sc, plane, epart, ppart, st);
    default:  return cg_z_p<F32C>(g, ntiles, r, pold, pnew, q, eps, sc, plane, epart, ppart, st);
  }
}

hipError_t launch_zfinal(int prec, const PassGeom& g, int ntiles, const void* t, const void* c,
                         const void* kxy, void* out, int64_t plane, double kmul, double* epart,
                         hipStream_t st) {
  switch (prec) {
    case F64: return zfinal_p<F64>(g, ntiles, t, c, kxy, out, plane, kmul, epart, st);
    case F32: return zfinal_p<F32>(g, ntiles, t, c, kxy, out, plane, kmul, epart, st);
    default:  return zfinal_p<F32C>(g, ntiles, t, c, kxy, out, plane, kmul, epart, st);
  }
}

template <int P, int MODE>
hipError_t line_z_launch(int shape, const PassGeom& g, const ZLineArgs& a, int nblocks, hipStream_t st);

template <int P>
static hipError_t line_z_mode(int mode, int shape, const PassGeom& g, const ZLineArgs& a, int nblocks,
                              hipStream_t st) {
  switch (mode) {
    case ZL_CW:    return line_z_launch<P, ZL_CW>(shape, g, a, nblocks, st);
    case ZL_CWT:   return line_z_launch<P, ZL_CWT>(shape, g, a, nblocks, st);
    case ZL_CK:    return line_z_launch<P, ZL_CK>(shape, g, a, nblocks, st);
    case ZL_FINAL: return line_z_launch<P, ZL_FINAL>(shape, g, a, nblocks, st);
    default:       return line_z_launch<P, ZL_CG>(shape, g, a, nblocks, st);
  }
}

hipError_t launch_line_z(int prec, int mode, int shape, const PassGeom& g, const ZLineArgs& a,
                         int nblocks, hipStream_t st) {
  if (nblocks == 0) return hipSuccess;
  switch (prec) {
    case F64: return line_z_mode<F64>(mode, shape, g, a, nblocks, st);
    case F32: return line_z_mode<F32>(mode, shape, g, a, nblocks, st);
    default:  return line_z_mode<F32C>(mode, shape, g, a, nblocks, st);
  }
}

hipError_t launch_pass(int prec, int op, int axis, const PassGeom& g, int ntiles, const void* in,
                       void* out, const void* k0, int64_t plane, double kmul, double* epart,
                       hipStream_t st) {
  switch (prec) {
    case F64: return launch_op<F64>(op, axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case F32: return launch_op<F32>(op, axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    default:  return launch_op<F32C>(op, axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
  }
}

}  // namespace wvl
