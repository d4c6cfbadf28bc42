// 1D periodic convolution passes over a batch of orbitals, gfx950.
//
// The 3D operators of the method are separable: each is three 1D periodic
// convolutions, one along each axis (Sec. 3.1, Eqs. "3dconv", "1dconvtrans";
// the kinetic operator is a sum of three 1D filters, Sec. 3.4, Eq.
// "kinetic1d").  The paper's GPU kernel writes every pass transposed so that
// the next pass again convolves along the slowest axis; here the data stays in
// its natural (m3, m2, m1) layout instead:
//  * passes along axes 2 and 3 (strided axes) give one line to each lane;
//    consecutive lanes own consecutive lines, which are adjacent in memory, so
//    every row of loads and stores is a coalesced 64-lane access, and each lane
//    runs a register sliding window down its line (no LDS needed);
//  * passes along axis 1 (the contiguous axis) stage a block of whole rows in
//    LDS with a periodic halo of 32 values on each side, then every lane
//    computes two neighbouring outputs from a register window read from LDS.
// The periodic boundary (Sec. 3.1) is applied by modular indexing on the
// loads, so lines shorter than the filter are handled as well.

//
// Device code and per-precision launchers (templates); wvl_passes.hip holds
// the dispatch and each wvl_passes_<prec>.hip instantiates one precision.
#pragma once

#include <algorithm>

#include "wvl_internal.h"
#include "wvl_kernels.h"

namespace wvl {

constexpr int kPf = 4;   // output pairs whose loads are in flight (strided passes)

template <int P, int OP>
__device__ __forceinline__ void pair_conv(const typename Prec<P>::V* win, typename Prec<P>::V& y0,
                                          typename Prec<P>::V& y1) {
  using T = Prec<P>;
  constexpr int OLO = OpWin<OP>::OLO, OHI = OpWin<OP>::OHI;
  typename T::Acc a0 = T::zero(), a1 = T::zero();
  #pragma unroll
  for (int o = OLO; o <= OHI; ++o) {
    // window: win[i] = x[k - OHI + i]; so x[k - o] = win[OHI - o]
    if (coef<OP>(0, o, 0) != 0.0) T::template add<OP>(a0, 0, o, win[OHI - o]);
    if (coef<OP>(1, o, 0) != 0.0) T::template add<OP>(a1, 1, o, win[OHI - o + 1]);
  }
  y0 = T::fin(a0);
  y1 = T::fin(a1);
}

// Line of this lane in tile t of an axis-3 pass and the outputs [k0, k1) it
// computes: lines in blocks of kThreads, every block once per segment.
__device__ __forceinline__ int64_t z_segment(int t, int64_t L, int m, int zlen, int& k0, int& k1) {
  const int blocks = (int)((L + kThreads - 1) / kThreads);
  const int seg = t / blocks;
  k0 = seg * zlen;
  k1 = min(m, k0 + zlen);
  return (int64_t)(t - seg * blocks) * kThreads + threadIdx.x;
}

// N values of a periodic line of m from position i0 on, into f(i, position):
// one division for the first position, the others stepped.  With a division for
// each of the up to 88 loads of a first window the last z step of 64 float32
// orbitals of 144 x 20 x 8 points took 28.3 us, now 18.1.
template <int N, typename F>
__device__ __forceinline__ void wrap_run(int i0, int m, F&& f) {
  int s = wrapi(i0, m);
  #pragma unroll
  for (int i = 0; i < N; ++i) {
    f(i, s);
    s = s + 1 == m ? 0 : s + 1;
  }
}

// ---------------------------------------------------------------------------
// Strided-axis pass (AXIS = 2 or 3)
// ---------------------------------------------------------------------------
template <int OP, int P, int AXIS, bool K0, bool EN, bool STREAM = false>
__global__ __launch_bounds__(kThreads) void k_strided(PassGeom g, const void* __restrict__ in,
                                                      void* __restrict__ out, const void* k0,
                                                      int64_t plane, double kmul,
                                                      double* __restrict__ epart) {
  using T = Prec<P>;
  using V = typename T::V;
  constexpr int OLO = OpWin<OP>::OLO, OHI = OpWin<OP>::OHI, W = OHI - OLO + 1;
  for_each_tile(g, [&](int b, int t, int slot) {
  const OrbDev od = g.orbs[b];
  const int m1 = od.m[0], m2 = od.m[1], m3 = od.m[2];
  const int m = AXIS == 3 ? m3 : m2;
  const int64_t L = AXIS == 3 ? (int64_t)m1 * m2 : (int64_t)m1 * m3;
  int k0l = 0, k1l = m;   // outputs of this lane
  int64_t line;
  if (AXIS == 3) {
    line = z_segment(t, L, m, g.zlen, k0l, k1l);
  } else {
    line = (int64_t)t * kThreads + threadIdx.x;
  }
  const double km = g.occ_weight ? kmul * od.occ : kmul;
  double e = 0.0;
  if (line < L) {
    const int64_t stride = AXIS == 3 ? (int64_t)m1 * m2 : (int64_t)m1;
    const int64_t base =
        od.off + (AXIS == 3 ? line : (line / m1) * ((int64_t)m1 * m2) + (line % m1));
    const double ks = AXIS == 3 ? od.kscale[2] : od.kscale[1];
    V win[W + 1];
    wrap_run<W - 1>(k0l - OHI, m, [&](int i, int s) { win[i] = T::ldc(in, base + (int64_t)s * stride, plane); });
    // The loads of the next kPf output pairs are in flight while a pair is
    // computed (ring of registers, refilled as it is consumed): a wave keeps
    // 2 kPf input loads (and as many accumulator loads) outstanding.
    V q0[kPf], q1[kPf], a0[kPf], a1[kPf];
    #pragma unroll
    for (int d = 0; d < kPf; ++d) {
      const int kk = k0l + 2 * d;
      if (kk < k1l) {
        q0[d] = T::ldc(in, base + (int64_t)wrapi(kk - OLO, m) * stride, plane);
        q1[d] = T::ldc(in, base + (int64_t)wrapi(kk + 1 - OLO, m) * stride, plane);
        if (K0) {
          a0[d] = T::ldc(k0, base + (int64_t)kk * stride, plane);
          a1[d] = T::ldc(k0, base + (int64_t)(kk + 1) * stride, plane);
        }
      }
    }
    for (int k = k0l; k < k1l; k += 2 * kPf) {
      #pragma unroll
      for (int d = 0; d < kPf; ++d) {
        const int kk = k + 2 * d;    // ends are even: a pair never straddles one
        if (kk < k1l) {
          win[W - 1] = q0[d];
          win[W] = q1[d];
          V c0, c1;
          if (K0) { c0 = a0[d]; c1 = a1[d]; }
          const int kn = kk + 2 * kPf;
          if (kn < k1l) {
            q0[d] = T::ldc(in, base + (int64_t)wrapi(kn - OLO, m) * stride, plane);
            q1[d] = T::ldc(in, base + (int64_t)wrapi(kn + 1 - OLO, m) * stride, plane);
            if (K0) {
              a0[d] = T::ldc(k0, base + (int64_t)kn * stride, plane);
              a1[d] = T::ldc(k0, base + (int64_t)(kn + 1) * stride, plane);
            }
          }
          V y0, y1;
          pair_conv<P, OP>(win, y0, y1);
          if (OP == OP_KIN || OP == OP_CK) {
            // energies use the unweighted operator; kmul weights the output only
            y0 = T::scale(y0, ks);
            y1 = T::scale(y1, ks);
            if (EN) e += T::d(win[OHI]) * T::d(y0) + T::d(win[OHI + 1]) * T::d(y1);
            if (km != 1.0) { y0 = T::scale(y0, km); y1 = T::scale(y1, km); }
          }
          const int64_t i0 = base + (int64_t)kk * stride, i1 = i0 + stride;
          if (K0) {
            y0 = T::plus(y0, c0);
            y1 = T::plus(y1, c1);
          }
          if (STREAM) {
            T::st_stream(out, i0, plane, y0);
            T::st_stream(out, i1, plane, y1);
          } else {
            T::st(out, i0, plane, y0);
            T::st(out, i1, plane, y1);
          }
          #pragma unroll
          for (int i = 0; i < W - 1; ++i) win[i] = win[i + 2];
        }
      }
    }
  }
  if (EN) block_sum_store(e, epart + slot);
  });
}

// ---------------------------------------------------------------------------
// Last step of the plane-resident H*psi, along z, fused:
//     out = W_z^T t + (kmul K_z c + kxy)
// (the two z passes that would otherwise write and re-read kxy), with the
// kinetic energy <c, K_z c> of each tile.  Same association as the two
// separate passes, so the results are the same bit for bit.
// ---------------------------------------------------------------------------
constexpr int kPfZ = 2;   // output pairs in flight (two register windows here)

template <int P, bool EN>
__global__ __launch_bounds__(kThreads) void k_zfinal(PassGeom g, const void* __restrict__ t,
                                                     const void* __restrict__ c, const void* kxy,
                                                     void* __restrict__ out, int64_t plane,
                                                     double kmul, double* __restrict__ epart) {
  using T = Prec<P>;
  using V = typename T::V;
  constexpr int LT = OpWin<OP_CWT>::OLO, HT = OpWin<OP_CWT>::OHI, WT = HT - LT + 1;
  constexpr int LK = OpWin<OP_CK>::OLO, HK = OpWin<OP_CK>::OHI, WK = HK - LK + 1;
  for_each_tile(g, [&](int b, int tl, int slot) {
  const OrbDev od = g.orbs[b];
  const int m1 = od.m[0], m2 = od.m[1], m = od.m[2];
  const int64_t L = (int64_t)m1 * m2;
  int k0l, k1l;   // outputs of this lane
  const int64_t line = z_segment(tl, L, m, g.zlen, k0l, k1l);
  const double km = g.occ_weight ? kmul * od.occ : kmul;
  double e = 0.0;
  if (line < L) {
    const int64_t stride = L;
    const int64_t base = od.off + line;
    const double ks = od.kscale[2];
    auto at = [&](int i) { return base + (int64_t)wrapi(i, m) * stride; };
    V wt[WT + 1], wk[WK + 1];
    wrap_run<WT - 1>(k0l - HT, m, [&](int i, int s) { wt[i] = T::ldc(t, base + (int64_t)s * stride, plane); });
    wrap_run<WK - 1>(k0l - HK, m, [&](int i, int s) { wk[i] = T::ldc(c, base + (int64_t)s * stride, plane); });
    V qt0[kPfZ], qt1[kPfZ], qk0[kPfZ], qk1[kPfZ], a0[kPfZ], a1[kPfZ];
    auto fetch = [&](int d, int kk) {
      qt0[d] = T::ldc(t, at(kk - LT), plane);
      qt1[d] = T::ldc(t, at(kk + 1 - LT), plane);
      qk0[d] = T::ldc(c, at(kk - LK), plane);
      qk1[d] = T::ldc(c, at(kk + 1 - LK), plane);
      a0[d] = T::ldc(kxy, base + (int64_t)kk * stride, plane);
      a1[d] = T::ldc(kxy, base + (int64_t)(kk + 1) * stride, plane);
    };
    #pragma unroll
    for (int d = 0; d < kPfZ; ++d)
      if (k0l + 2 * d < k1l) fetch(d, k0l + 2 * d);
    for (int k = k0l; k < k1l; k += 2 * kPfZ) {
      #pragma unroll
      for (int d = 0; d < kPfZ; ++d) {
        const int kk = k + 2 * d;    // ends are even: a pair never straddles one
        if (kk < k1l) {
          wt[WT - 1] = qt0[d];
          wt[WT] = qt1[d];
          wk[WK - 1] = qk0[d];
          wk[WK] = qk1[d];
          const V x0 = a0[d], x1 = a1[d];
          if (kk + 2 * kPfZ < k1l) fetch(d, kk + 2 * kPfZ);
          V z0, z1, y0, y1;
          pair_conv<P, OP_CK>(wk, z0, z1);
          z0 = T::scale(z0, ks);
          z1 = T::scale(z1, ks);
          if (EN) e += T::d(wk[HK]) * T::d(z0) + T::d(wk[HK + 1]) * T::d(z1);
          if (km != 1.0) { z0 = T::scale(z0, km); z1 = T::scale(z1, km); }
          z0 = T::plus(z0, x0);
          z1 = T::plus(z1, x1);
          pair_conv<P, OP_CWT>(wt, y0, y1);
          const int64_t i0 = base + (int64_t)kk * stride;
          T::st_stream(out, i0, plane, T::plus(y0, z0));
          T::st_stream(out, i0 + stride, plane, T::plus(y1, z1));
          #pragma unroll
          for (int i = 0; i < WT - 1; ++i) wt[i] = wt[i + 2];
          #pragma unroll
          for (int i = 0; i < WK - 1; ++i) wk[i] = wk[i + 2];
        }
      }
    }
  }
  if (EN) block_sum_store(e, epart + slot);
  });
}

// ---------------------------------------------------------------------------
// Direction update of the preconditioner fused with its z pass:
//     p = r / diag + beta p_old,   q = K_z p
// with the partials of p.q and p.p of each tile.  The update is a pass over
// r and p_old that the z pass reads anyway, so the fused launch moves four
// arrays where the two moved five: 256 float64 orbitals of 48^3 cells 1.53 ms
// (4.7 TB/s) where the two took 0.93 + 1.02.  p goes to another
// array than p_old: lanes re-read the ends of a line for the periodic wrap.
// Loads, not the FMAs, bound it: kPfP pairs of each operand are in flight.
// (Lines held in LDS: wvl_line_z.h.)
// ---------------------------------------------------------------------------
constexpr int kPfP = 2;

template <int P, bool STREAM>
__global__ __launch_bounds__(kThreads, 2) void k_cg_z(PassGeom g, const void* __restrict__ r,
                                                      const void* __restrict__ pold,
                                                      void* __restrict__ pnew, void* __restrict__ q,
                                                      const double* __restrict__ eps,
                                                      const CgScal* __restrict__ sc, int64_t plane,
                                                      double* __restrict__ epart,
                                                      double* __restrict__ ppart) {
  using T = Prec<P>;
  using V = typename T::V;
  constexpr int OLO = OpWin<OP_CK>::OLO, OHI = OpWin<OP_CK>::OHI, W = OHI - OLO + 1;
  int b, t;
  find_tile(g.prefix, g.norb, blockIdx.x, b, t);
  const OrbDev od = g.orbs[b];
  const int m1 = od.m[0], m2 = od.m[1], m = od.m[2];
  const int64_t L = (int64_t)m1 * m2;
  int k0l, k1l;
  const int64_t line = z_segment(t, L, m, g.zlen, k0l, k1l);
  double e = 0.0, pp = 0.0;
  if (line < L) {
    const int64_t base = od.off + line;
    const double ks = od.kscale[2], beta = sc[b].beta, ep = eps[b];
    const int x = (int)(line % m1) & 1, y = (int)(line / m1) & 1;
    const double dxy = (x ? od.kdiag[0][1] : od.kdiag[0][0]) + (y ? od.kdiag[1][1] : od.kdiag[1][0]);
    double w[2];   // 1 / diag at even and odd z
    w[0] = 1.0 / (dxy + od.kdiag[2][0] - ep);
    w[1] = 1.0 / (dxy + od.kdiag[2][1] - ep);
    auto at = [&](int i) { return base + (int64_t)wrapi(i, m) * L; };
    // (the wrap keeps the parity of z: m is even)
    auto dir = [&](V rv, V pv, int par) {
      return T::from_d(__builtin_fma(beta, T::d(pv), T::d(rv) * w[par]));
    };
    V win[W + 1];
    constexpr int FB = 4;   // loads of the first window in batches
    #pragma unroll
    for (int i0 = 0; i0 < W - 1; i0 += FB) {
      V rv[FB], pv[FB];
      wrap_run<FB>(k0l + i0 - OHI, m, [&](int j, int z) {
        if (i0 + j < W - 1) {
          rv[j] = T::ldc(r, base + (int64_t)z * L, plane);
          pv[j] = T::ldc(pold, base + (int64_t)z * L, plane);
        }
      });
      #pragma unroll
      for (int j = 0; j < FB; ++j)
        if (i0 + j < W - 1) win[i0 + j] = dir(rv[j], pv[j], (i0 + j - OHI) & 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    V r0[kPfP], r1[kPfP], p0[kPfP], p1[kPfP];
    auto fetch = [&](int d, int kk) {
      r0[d] = T::ldc(r, at(kk - OLO), plane);
      r1[d] = T::ldc(r, at(kk + 1 - OLO), plane);
      p0[d] = T::ldc(pold, at(kk - OLO), plane);
      p1[d] = T::ldc(pold, at(kk + 1 - OLO), plane);
    };
    #pragma unroll
    for (int d = 0; d < kPfP; ++d)
      if (k0l + 2 * d < k1l) fetch(d, k0l + 2 * d);
    for (int k = k0l; k < k1l; k += 2 * kPfP) {
      #pragma unroll
      for (int d = 0; d < kPfP; ++d) {
        const int kk = k + 2 * d;
        if (kk < k1l) {
          win[W - 1] = dir(r0[d], p0[d], OLO & 1);
          win[W] = dir(r1[d], p1[d], (OLO & 1) ^ 1);
          if (kk + 2 * kPfP < k1l) fetch(d, kk + 2 * kPfP);
          V y0, y1;
          pair_conv<P, OP_CK>(win, y0, y1);
          y0 = T::scale(y0, ks);
          y1 = T::scale(y1, ks);
          const double c0 = T::d(win[OHI]), c1 = T::d(win[OHI + 1]);
          e += c0 * T::d(y0) + c1 * T::d(y1);
          pp += c0 * c0 + c1 * c1;
          const int64_t i0 = base + (int64_t)kk * L, i1 = i0 + L;
          if (STREAM) {
            T::st_stream(q, i0, plane, y0);
            T::st_stream(q, i1, plane, y1);
            T::st_stream(pnew, i0, plane, win[OHI]);
            T::st_stream(pnew, i1, plane, win[OHI + 1]);
          } else {
            T::st(q, i0, plane, y0);
            T::st(q, i1, plane, y1);
            T::st(pnew, i0, plane, win[OHI]);
            T::st(pnew, i1, plane, win[OHI + 1]);
          }
          #pragma unroll
          for (int i = 0; i < W - 1; ++i) win[i] = win[i + 2];
        }
      }
    }
  }
  block_sum_store(e, epart + blockIdx.x);
  block_sum_store(pp, ppart + blockIdx.x);
}

// ---------------------------------------------------------------------------
// Contiguous-axis pass (axis 1), LDS row tiles with periodic halo
// ---------------------------------------------------------------------------
template <int OP, int P, bool K0, bool EN>
__global__ __launch_bounds__(kThreads) void k_contig(PassGeom g, const void* in, void* out,
                                                     const void* k0, int64_t plane, double kmul,
                                                     double* __restrict__ epart) {
  using T = Prec<P>;
  using V = typename T::V;
  constexpr int OLO = OpWin<OP>::OLO, OHI = OpWin<OP>::OHI, W = OHI - OLO + 1;
  static_assert(OHI <= kHalo && -OLO <= kHalo, "halo too small");
  __shared__ V lds[kContigLds];
  for_each_tile(g, [&](int b, int t, int slot) {
  const OrbDev od = g.orbs[b];
  const int m1 = od.m[0];
  const int rows = od.m[1] * od.m[2];
  const int pitch = m1 + 2 * kHalo;
  const int R = contig_rows(m1, g.xdiv);
  const int row0 = t * R;
  const int nrows = min(R, rows - row0);
  const int64_t gbase = od.off + (int64_t)row0 * m1;
  // load rows [row0, row0 + nrows) with halo: lds[r*pitch + p] = x[r][(p - kHalo) mod m1]
  const int nload = nrows * pitch;
  for (int e = threadIdx.x; e < nload; e += kThreads) {
    const int r = e / pitch;
    const int p = e - r * pitch;
    lds[e] = T::ldc(in, gbase + (int64_t)r * m1 + wrapi(p - kHalo, m1), plane);
  }
  __syncthreads();
  const double ks = od.kscale[0];
  const int half = m1 >> 1;
  const int npairs = nrows * half;
  double en = 0.0;
  for (int q = threadIdx.x; q < npairs; q += kThreads) {
    const int r = q / half;
    const int k = 2 * (q - r * half);
    const V* src = lds + r * pitch + kHalo + k - OHI;
    V win[W + 1];
    #pragma unroll
    for (int i = 0; i <= W; ++i) win[i] = src[i];
    V y0, y1;
    pair_conv<P, OP>(win, y0, y1);
    if (OP == OP_KIN || OP == OP_CK) {
      y0 = T::scale(y0, ks);
      y1 = T::scale(y1, ks);
      if (EN) en += T::d(win[OHI]) * T::d(y0) + T::d(win[OHI + 1]) * T::d(y1);
      if (kmul != 1.0) { y0 = T::scale(y0, kmul); y1 = T::scale(y1, kmul); }
    }
    const int64_t i0 = gbase + (int64_t)r * m1 + k;
    if (K0) {
      y0 = T::plus(y0, T::ldc(k0, i0, plane));
      y1 = T::plus(y1, T::ldc(k0, i0 + 1, plane));
    }
    T::st(out, i0, plane, y0);
    T::st(out, i0 + 1, plane, y1);
  }
  if (EN) block_sum_store(en, epart + slot);
  });
}

// ---------------------------------------------------------------------------
// Host launchers
// ---------------------------------------------------------------------------
template <int OP, int P>
static hipError_t launch_axis(int axis, const PassGeom& g, int ntiles, const void* in, void* out,
                              const void* k0, int64_t plane, double kmul, double* epart,
                              hipStream_t st) {
  const bool en = epart != nullptr;
  dim3 grid(g.queue ? std::min(ntiles, g.grid) : ntiles), block(kThreads);
  if (ntiles == 0) return hipSuccess;
#define WVL_L(KERN) hipLaunchKernelGGL((KERN), grid, block, 0, st, g, in, out, k0, plane, kmul, epart)
  if (axis == 1) {
    if (k0) { if (en) WVL_L((k_contig<OP, P, true, true>)); else WVL_L((k_contig<OP, P, true, false>)); }
    else    { if (en) WVL_L((k_contig<OP, P, false, true>)); else WVL_L((k_contig<OP, P, false, false>)); }
  } else if (axis == 2) {
    if (k0) { if (en) WVL_L((k_strided<OP, P, 2, true, true>)); else WVL_L((k_strided<OP, P, 2, true, false>)); }
    else    { if (en) WVL_L((k_strided<OP, P, 2, false, true>)); else WVL_L((k_strided<OP, P, 2, false, false>)); }
  } else {
    constexpr bool S = P == F64;   // (stream_st)
    if (k0) { if (en) WVL_L((k_strided<OP, P, 3, true, true>)); else WVL_L((k_strided<OP, P, 3, true, false>)); }
    else if (S && g.stream) {
      if (en) WVL_L((k_strided<OP, P, 3, false, true, S>)); else WVL_L((k_strided<OP, P, 3, false, false, S>));
    } else  { if (en) WVL_L((k_strided<OP, P, 3, false, true>)); else WVL_L((k_strided<OP, P, 3, false, false>)); }
  }
#undef WVL_L
  return hipGetLastError();
}

template <int P>
hipError_t launch_op(int op, int axis, const PassGeom& g, int ntiles, const void* in,
                            void* out, const void* k0, int64_t plane, double kmul, double* epart,
                            hipStream_t st) {
  switch (op) {
    case OP_MF:  return launch_axis<OP_MF, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case OP_MFT: return launch_axis<OP_MFT, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case OP_SYN: return launch_axis<OP_SYN, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case OP_ANA: return launch_axis<OP_ANA, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case OP_KIN: return launch_axis<OP_KIN, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case OP_CW:  return launch_axis<OP_CW, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    case OP_CWT: return launch_axis<OP_CWT, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
    default:     return launch_axis<OP_CK, P>(axis, g, ntiles, in, out, k0, plane, kmul, epart, st);
  }
}

template <int P>
hipError_t zfinal_p(const PassGeom& g, int ntiles, const void* t, const void* c,
                           const void* kxy, void* out, int64_t plane, double kmul, double* epart,
                           hipStream_t st) {
  if (ntiles == 0) return hipSuccess;
  dim3 grid(g.queue ? std::min(ntiles, g.grid) : ntiles), block(kThreads);
  if (epart)
    hipLaunchKernelGGL((k_zfinal<P, true>), grid, block, 0, st, g, t, c, kxy, out, plane, kmul, epart);
  else
    hipLaunchKernelGGL((k_zfinal<P, false>), grid, block, 0, st, g, t, c, kxy, out, plane, kmul, epart);
  return hipGetLastError();
}

template <int P>
hipError_t cg_z_p(const PassGeom& g, int ntiles, const void* r, const void* pold, void* pnew, void* q,
                  const double* eps, const void* sc, int64_t plane, double* epart, double* ppart,
                  hipStream_t st) {
  if (ntiles == 0) return hipSuccess;
  if (P == F64 && g.stream)
    hipLaunchKernelGGL((k_cg_z<P, P == F64>), dim3(ntiles), dim3(kThreads), 0, st, g, r, pold, pnew, q,
                       eps, (const CgScal*)sc, plane, epart, ppart);
  else
    hipLaunchKernelGGL((k_cg_z<P, false>), dim3(ntiles), dim3(kThreads), 0, st, g, r, pold, pnew, q,
                       eps, (const CgScal*)sc, plane, epart, ppart);
  return hipGetLastError();
}

}  // namespace wvl
