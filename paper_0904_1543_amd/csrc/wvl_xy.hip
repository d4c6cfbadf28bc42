// Host dispatch of the in-plane kernel (the device code is in wvl_xy_impl.h,
// instantiated per precision and engine by the wvl_xy_<form>.hip files).

#include <stdlib.h>

#include <algorithm>

#include "wvl_plane.h"

namespace wvl {

template <int P, bool SH>
void xy_launch_v(const XyArgs& a, int mi, int nblocks, size_t lds, hipStream_t st);
template <bool SH>
void xy_launch_m(const XyArgs& a, int mt, int nblocks, size_t lds, hipStream_t st);
template <int P>
void helm_launch_v(const HelmArgs& a, int mi, int nblocks, size_t lds, hipStream_t st);
void helm_launch_mf(const HelmArgs& a, int mt, int nblocks, size_t lds, hipStream_t st);

template <int P, int MODE, bool SH, int FREE>
hipError_t line_launch(int shape, const XyArgs& a, int nblocks, int nt, size_t lds, hipStream_t st);

// rho[r] = sum_g rho_part[g][r] (group order), and per-block sums of V rho
__global__ __launch_bounds__(kThreads) void k_rho_reduce(const double* __restrict__ part, int ngroups,
                                                         int64_t M, const double* __restrict__ V,
                                                         double* rho, int acc,
                                                         double* __restrict__ rvpart) {
  const int64_t r = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  double s = 0.0;
  if (r < M)
    for (int g = 0; g < ngroups; ++g) s += part[(int64_t)g * M + r];
  if (rho && r < M) rho[r] = acc ? rho[r] + s : s;
  if (rvpart) block_sum_store(r < M ? V[r] * s : 0.0, rvpart + blockIdx.x);
}

static int xy_items(int m1, int m2) {
  const int ix = ((m1 + kU - 1) / kU) * m2, iy = ((m2 + kU - 1) / kU) * m1;
  const int it = ix > iy ? ix : iy;
  return (it + kXyThreads - 1) / kXyThreads;
}
static int xy_tiles(int m1, int m2) {
  const int nt = ((m1 + 15) / 16) * ((m2 + 15) / 16);
  return (nt + kXyWaves - 1) / kXyWaves;
}
static int mf_pitch(int m1) { return m1 + ((36 - (m1 & 31)) & 31); }

bool xy_matrix_engine(int prec, int m1, int m2) {
  return prec == F64 && xy_tiles(m1, m2) <= 8 && (size_t)m2 * mf_pitch(m1) * 8 <= 160 * 1024;
}

// The preconditioner's operator over a batch of several grids, planes of up to
// m1 x m2 values: whether one launch of the workgroup-wide kernel is faster than
// the plane kernel, which takes a launch for each of its shapes, sized for the
// class's largest plane, with one plane a workgroup (no second one to load
// ahead).  Three CG steps on 32 / 100 orbitals of 8..48 cells an axis, plane
// kernel against this: float64 618 / 2063 us against 545 / 1984, float32 515 /
// 1454 against 427 / 1266.  Planes of up to 64 x 64 have few shapes (8..24 cells,
// 100 orbitals, 464 and 463 us; 378 and 387); larger ones than 96 x 96 spill the
// instances here (16..64 cells, 100 orbitals: 5.1 and 6.0 ms; 3.4 and 8.6), which
// in float64, up to 112 x 112, a batch of few planes does not notice (8..52 cells,
// 32 orbitals 896 and 812 us, 100 orbitals 2498 and 2800).
bool helm_whole(int prec, int m1, int m2, int nplanes) {
  if (prec == F32C || std::max(m1, m2) <= 64) return false;
  if (prec == F32) return xy_supported(prec, m1, m2, false) && xy_items(m1, m2) <= 5;
  return xy_matrix_engine(prec, m1, m2) && xy_tiles(m1, m2) <= (nplanes <= 2048 ? 7 : 5);
}

size_t xy_lds_bytes(int prec, int m1, int m2, bool engine) {
  if (engine) return (size_t)m2 * mf_pitch(m1) * 8;
  return (size_t)m2 * (m1 + 1) * (prec == F32 ? 4 : 8);
}

bool xy_supported(int prec, int m1, int m2, bool engine) {
  if (engine) return xy_matrix_engine(prec, m1, m2);
  return xy_items(m1, m2) <= kMaxItems && xy_lds_bytes(prec, m1, m2, false) <= 160 * 1024;
}

hipError_t launch_xy(int prec, const XyArgs& a, int m1, int m2, int nblocks, hipStream_t st) {
  if (nblocks == 0) return hipSuccess;
  const bool sh = a.shared != 0;
  const bool mx = a.engine != 0;
  if (mx && !xy_matrix_engine(prec, m1, m2)) return hipErrorInvalidValue;
  const size_t lds = xy_lds_bytes(prec, m1, m2, mx);
  if (mx) {
    const int mt = xy_tiles(m1, m2);
    // one workgroup per CU anyway at 2 waves per SIMD: keep the group's
    // density plane in LDS beside the plane (same pitch) when both fit
    XyArgs b = a;
    b.rho_lds = sh && a.occupancy == 2 && 2 * lds <= 160 * 1024 && !getenv("WVL_NO_RHO_LDS");
    const size_t l = b.rho_lds ? 2 * lds : lds;
    sh ? xy_launch_m<true>(b, mt, nblocks, l, st) : xy_launch_m<false>(b, mt, nblocks, l, st);
    return hipGetLastError();
  }
  const int mi = xy_items(m1, m2);
  switch (prec) {
    case F64: sh ? xy_launch_v<F64, true>(a, mi, nblocks, lds, st) : xy_launch_v<F64, false>(a, mi, nblocks, lds, st); break;
    case F32: sh ? xy_launch_v<F32, true>(a, mi, nblocks, lds, st) : xy_launch_v<F32, false>(a, mi, nblocks, lds, st); break;
    default:  sh ? xy_launch_v<F32C, true>(a, mi, nblocks, lds, st) : xy_launch_v<F32C, false>(a, mi, nblocks, lds, st); break;
  }
  return hipGetLastError();
}

hipError_t launch_helm_xy(int prec, const HelmArgs& a, int m1, int m2, int nblocks, bool engine,
                          hipStream_t st) {
  if (nblocks == 0) return hipSuccess;
  if (engine && !xy_matrix_engine(prec, m1, m2)) return hipErrorInvalidValue;
  const size_t lds = xy_lds_bytes(prec, m1, m2, engine);
  if (engine) {
    helm_launch_mf(a, xy_tiles(m1, m2), nblocks, lds, st);
    return hipGetLastError();
  }
  const int mi = xy_items(m1, m2);
  switch (prec) {
    case F64: helm_launch_v<F64>(a, mi, nblocks, lds, st); break;
    case F32: helm_launch_v<F32>(a, mi, nblocks, lds, st); break;
    default:  helm_launch_v<F32C>(a, mi, nblocks, lds, st); break;
  }
  return hipGetLastError();
}

// shape of the plane kernel for planes of up to m1 x m2 values (-1: none),
// its threads and its LDS
static int line_shape(int prec, int mode, int m1, int m2, int free, int* nt, size_t* lds) {
  const size_t es = prec == F32 ? 4 : 8;
  const int M1 = m1 + line_extra(mode, free & 1), M2 = m2 + line_extra(mode, free & 2);
  for (int s = 0; s < kNumLineShapes; ++s) {
    const LineShape& k = kLineShapes[s];
    const int sx = (M1 + k.U - 1) / k.U, sy = (M2 + k.U - 1) / k.U;   // segments of a line
    const int lx = sx <= 64 ? line_lines(k.U, sx) : 0, ly = sy <= 64 ? line_lines(k.U, sy) : 0;
    if (lx == 0 || ly == 0) continue;
    const int gx = (m2 + lx - 1) / lx, gy = (M1 + ly - 1) / ly;   // groups of lines
    *nt = 64 * ((std::max(gx, gy) + k.mi - 1) / k.mi);
    // (isolated axes: two rows of zeros after the plane)
    *lds = (size_t)(M2 + (free ? 2 : 0) + (k.two && !free ? m2 : 0)) * k.pitch * es;
    if (M1 < k.pitch && *nt <= k.nt && *lds <= 159 * 1024) return s;
  }
  return -1;
}

int line_shape_of(int prec, int m1, int m2, int free) {
  int nt;
  size_t lds;
  return line_shape(prec, LINE_HPSI, m1, m2, free, &nt, &lds);
}

// workgroups of the shape that share a compute unit: by LDS and by waves
int line_per_cu(int prec, int m1, int m2) {
  int nt;
  size_t lds;
  const int s = line_shape(prec, LINE_HPSI, m1, m2, 0, &nt, &lds);
  if (s < 0) return 1;
  const int waves = 4 * kLineShapes[s].wpe;
  return std::max(1, std::min((int)(160 * 1024 / (lds + 1024)), waves / (nt / 64)));
}

hipError_t launch_line(int prec, int mode, const XyArgs& a, int m1, int m2, int nblocks,
                       hipStream_t st) {
  if (nblocks == 0) return hipSuccess;
  int nt;
  size_t lds;
  const int s = line_shape(prec, mode, m1, m2, a.free, &nt, &lds);
  if (s < 0) return hipErrorInvalidValue;
#define WVL_F(P, FR)                                                                             \
  (mode == LINE_HELM  ? line_launch<P, LINE_HELM, true, FR>(s, a, nblocks, nt, lds, st)          \
   : mode == LINE_RHO ? line_launch<P, LINE_RHO, true, FR>(s, a, nblocks, nt, lds, st)           \
                      : line_launch<P, LINE_HPSI, true, FR>(s, a, nblocks, nt, lds, st))
#define WVL_P(P)                                                                                 \
  return a.free == 3 ? WVL_F(P, 3)                                                               \
         : a.free == 2 ? WVL_F(P, 2)                                                             \
         : a.shared ? WVL_F(P, 0)                                                                \
         : mode == LINE_HPSI ? line_launch<P, LINE_HPSI, false, 0>(s, a, nblocks, nt, lds, st)   \
                             : line_launch<P, LINE_HELM, false, 0>(s, a, nblocks, nt, lds, st)
  switch (prec) {
    case F64: WVL_P(F64);
    case F32: WVL_P(F32);
    default: WVL_P(F32C);
  }
#undef WVL_F
#undef WVL_P
}

hipError_t launch_rho_reduce(const double* part, int ngroups, int64_t M, const double* V,
                             double* rho, int accumulate, double* rvpart, hipStream_t st) {
  const int nblk = (int)((M + kThreads - 1) / kThreads);
  hipLaunchKernelGGL(k_rho_reduce, dim3(nblk), dim3(kThreads), 0, st, part, ngroups, M, V, rho,
                     accumulate, rvpart);
  return hipGetLastError();
}

}  // namespace wvl
