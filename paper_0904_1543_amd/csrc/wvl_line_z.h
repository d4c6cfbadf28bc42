// z passes with whole lines in LDS, gfx950.
//
// A workgroup of four waves takes 64 adjacent lines along axis 3: it loads them
// once into the LDS, each wave every fourth row of 64 values (rows of 16, loaded
// by the wave that needs them, save the barriers but cost 16% with float pairs,
// where they are 64 bytes, and 3% on lines that do not start on a cache line).
// A wave then computes 16 of the lines with line_conv, 16 lines x 4 segments of
// U outputs at a time.  Every value is read from memory once.  The 16 lanes that
// the LDS serves together in float64 read 16 adjacent values; in float32 the row
// pitch puts the segments of a wave on distinct banks.
//
// Bound by memory traffic: 256 orbitals of 48^3 cells take, in float64, 0.65 ms
// for W (5.6 TB/s), 1.41 for the last step (5.1) and 1.31 for the direction
// update with K (5.5; with the update of x 2.07, 5.2); in float pairs 0.75 and 1.49.  The strided passes (0.71,
// 1.77, 1.53; 0.83 and 2.39), whose lanes hold a window of the line, read its
// first 58 values twice, spend a third of their vector instructions on moving
// the window and fill the registers with it; they stay for longer lines than
// the LDS holds a workgroup's worth of, and for the lengths at which they are
// faster (line_z_pays).  Work queues are not used: a queue's
// barriers and its counter cost 12% of the last step.
#pragma once

#include "wvl_line.h"

namespace wvl {

// row pitch of the lines in LDS
template <int U, typename C> constexpr int zline_pitch() {
  return sizeof(C) == 8 ? kZLines : U == 8 ? 66 : U == 10 ? 72 : 68;
}

template <int P, int U, int MI, int MODE>
struct ZLine {
  using IO = LineIO<P>;
  using C = typename IO::C;
  static constexpr int ST = zline_pitch<U, C>();
  static constexpr int NR = U * MI;      // values of a lane when a line has 4 U MI
  static constexpr int OP = MODE == ZL_CW ? OP_CW : MODE == ZL_CWT ? OP_CWT : OP_CK;

  const PassGeom& g;
  const ZLineArgs& a;
  Lds<C> buf;
  int x, s4;           // lane's line in the tile and first segment
  int lr, w;           // line that it loads, first row (the wave)
  uint32_t xl, xr, L;  // line of the orbital that it computes, and that it loads; lines
  int m;
  int64_t off;
  bool on, onr;        // those lines exist

  __device__ __forceinline__ ZLine(const PassGeom& g_, const ZLineArgs& a_, Lds<C> b_, OrbConst od, int t, int w_)
      : g(g_), a(a_), buf(b_) {
    const int lane = threadIdx.x & 63;
    x = w_ * 16 + (lane & 15);
    lr = lane;
    w = w_;
    s4 = lane >> 4;
    L = (uint32_t)od->m[0] * (uint32_t)od->m[1];
    m = od->m[2];
    off = od->off;
    const uint32_t l = (uint32_t)t * 16u + x, r = (uint32_t)t * 16u + lr;
    on = l < L;
    xl = min(l, L - 1);
    onr = r < L;
    xr = min(r, L - 1);
  }
  // rows 4 n + w of the tile, rows and lines past the end clamped
  __device__ __forceinline__ void load(const void* src, C (&r)[NR]) const {
    const char* p = IO::at(src, off);
    #pragma unroll
    for (int n = 0; n < NR; ++n) r[n] = IO::ld(p, (uint32_t)min(4 * n + w, m - 1) * L + xr, a.plane);
  }
  __device__ __forceinline__ void put(const C (&r)[NR]) const {
    #pragma unroll
    for (int n = 0; n < NR; ++n)
      if (4 * n + w < m) buf[(4 * n + w) * ST + lr] = r[n];
    __syncthreads();
  }
  // first output of this lane in group i (idle lanes repeat the first one)
  __device__ __forceinline__ int first(int i) const {
    int k0 = (s4 + 4 * i) * U;
    k0 = k0 < m ? k0 : 0;
    asm volatile("" : "+v"(k0));
    return k0;
  }
  __device__ __forceinline__ bool active(int i) const { return on && (s4 + 4 * i) * U < m; }
  // the values of an array at the outputs of group i
  __device__ __forceinline__ void fetch(const void* src, int i, C (&v)[U]) const {
    const int k0 = first(i);
    const char* p = IO::at(src, off);
    #pragma unroll
    for (int u = 0; u < U; ++u) v[u] = IO::ld(p, (uint32_t)min(k0 + u, m - 1) * L + xl, a.plane);
  }
  template <bool STREAM>
  __device__ __forceinline__ void store_(void* dst, int i, const C (&v)[U]) const {
    const int k0 = first(i);
    if (!active(i)) return;
    uint32_t o = (uint32_t)k0 * L + xl;
    char* d = IO::at(dst, off);
    #pragma unroll
    for (int u = 0; u < U; ++u, o += L)
      if (k0 + u < m) {
        if (STREAM) IO::st(d, o, a.plane, v[u]);
        else IO::st_keep(d, o, a.plane, v[u]);
      }
  }
  __device__ __forceinline__ void store(void* dst, int i, const C (&v)[U], bool stream) const {
    if (P == F64 && stream) store_<true>(dst, i, v);
    else store_<false>(dst, i, v);
  }
  template <int O> __device__ __forceinline__ void conv(int i, C (&r)[U]) const {
    line_conv<O, U, ST, O == OP_CK ? 1 : 2, false>(buf + x, m, 0, first(i), buf, r);
  }
  // v = s v, e += <line, v>
  __device__ __forceinline__ void energy(int i, C s, C (&v)[U], double& e) const {
    const int k0 = first(i);
    const bool act = active(i);
    #pragma unroll
    for (int u = 0; u < U; ++u) {
      v[u] *= s;
      const double c = (double)buf[min(k0 + u, m - 1) * ST + x];
      if (act && k0 + u < m) e = __builtin_fma(c, (double)v[u], e);
    }
  }
  __device__ __forceinline__ static void wave_total(double v, double* dst) {
    #pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s, 64);
    if ((threadIdx.x & 63) == 0) *dst = v;
  }

  __device__ __forceinline__ void run(OrbConst od, int b, int slot) const {
    const C ks = (C)od->kscale[2];
    const C km = (C)(g.occ_weight ? a.kmul * od->occ : a.kmul);
    double e = 0.0, pp = 0.0;
    C r[NR];
    if (MODE == ZL_CG) {
      C po[NR];
      load(a.in, po);
      if (P != F32 && a.x) {
        load(a.x, r);
        const double al = a.sc[b].alpha;
        uint32_t o = w * L + xr;
        char* d = IO::at(a.x, off);
        #pragma unroll
        for (int n = 0; n < NR; ++n, o += 4 * L)
          if (onr && 4 * n + w < m) {
            const C v = (C)((double)r[n] + al * (double)po[n]);
            if (P == F64 && g.stream) IO::st(d, o, a.plane, v);
            else IO::st_keep(d, o, a.plane, v);
          }
      }
      load(a.r, r);
      // 1 / diag at this lane's parities (rows 4 n + w: w's parity)
      const uint32_t m1 = (uint32_t)od->m[0], y = xr / m1;
      const double k0 = (xr - y * m1) & 1 ? od->kdiag[0][1] : od->kdiag[0][0];
      const double k1 = y & 1 ? od->kdiag[1][1] : od->kdiag[1][0];
      const double k2 = w & 1 ? od->kdiag[2][1] : od->kdiag[2][0];
      const double inv = 1.0 / (k0 + k1 + k2 - a.eps[b]), beta = a.sc[b].beta;
      #pragma unroll
      for (int n = 0; n < NR; ++n) r[n] = (C)__builtin_fma(beta, (double)po[n], (double)r[n] * inv);
      uint32_t o = w * L + xr;
      char* d = IO::at(a.pnew, off);
      #pragma unroll
      for (int n = 0; n < NR; ++n, o += 4 * L)
        if (onr && 4 * n + w < m) {
          pp = __builtin_fma((double)r[n], (double)r[n], pp);
          if (P == F64 && g.stream) IO::st(d, o, a.plane, r[n]);
          else IO::st_keep(d, o, a.plane, r[n]);
        }
      wave_total(pp, a.ppart + slot);
      put(r);
    } else {
      load(MODE == ZL_FINAL ? a.t : a.in, r);
      put(r);
    }
    if (MODE == ZL_FINAL) {
      // W^T t first: c and then kxy arrive behind the two convolutions.  (K c
      // first holds three arrays of values at once and spills; a reload waits for
      // every load in flight: 1.74 ms instead of 1.58 with float64, 2.19 instead
      // of 1.70 with float pairs.)
      C y[MI][U], z[MI][U];
      load(a.in, r);
      #pragma unroll
      for (int i = 0; i < MI; ++i)
        if (4 * i * U < m) conv<OP_CWT>(i, y[i]);
      __syncthreads();
      put(r);
      #pragma unroll
      for (int i = 0; i < MI; ++i) fetch(a.k0, i, z[i]);
      #pragma unroll
      for (int i = 0; i < MI; ++i)
        if (4 * i * U < m) {
          C v[U];
          conv<OP_CK>(i, v);
          energy(i, ks, v, e);
          #pragma unroll
          for (int u = 0; u < U; ++u) v[u] = y[i][u] + ((km != C(1) ? v[u] * km : v[u]) + z[i][u]);
          store(a.out, i, v, true);
        }
    } else {
      #pragma unroll
      for (int i = 0; i < MI; ++i)
        if (4 * i * U < m) {
          C v[U], k[U];
          if (MODE != ZL_CG && a.k0) fetch(a.k0, i, k);
          conv<OP>(i, v);
          if (OP == OP_CK) {
            energy(i, ks, v, e);
            if (km != C(1))
              #pragma unroll
              for (int u = 0; u < U; ++u) v[u] *= km;
          }
          if (MODE != ZL_CG && a.k0)
            #pragma unroll
            for (int u = 0; u < U; ++u) v[u] += k[u];
          store(a.out, i, v, g.stream != 0);
        }
    }
    if (OP == OP_CK && a.epart) wave_total(e, a.epart + slot);
  }
};

// Tile of a workgroup.  Workgroups go to the chip's 8 dies in turn, and a die's
// L2 spreads addresses over its channels: with a row of 512 bytes to every eighth
// workgroup a die would use a few of its channels.  Runs of kZRun adjacent tiles
// therefore go to one die (12 orbitals of odd sizes 540 -> 528 us, gradient of
// 128 orbitals of 32^3 cells 1.60 -> 1.58 ms).
constexpr int kZRun = 16;
__device__ __forceinline__ int die_tile(int i, int n) {
  const int full = n / (8 * kZRun) * (8 * kZRun);
  if (i >= full) return i;
  const int j = i % (8 * kZRun);
  return i - j + (j & 7) * kZRun + (j >> 3);
}

template <int P, int U, int MI, int MODE, int WPE>
__global__ __launch_bounds__(64 * kZWaves, WPE) void k_line_z(PassGeom g, ZLineArgs a) {
#ifdef __HIP_DEVICE_COMPILE__
  using K = ZLine<P, U, MI, MODE>;
  using C = typename K::C;
  extern __shared__ __attribute__((aligned(16))) char z_lds[];
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const Lds<C> buf = (Lds<C>)reinterpret_cast<C*>(z_lds);
  int b, t, slot = die_tile(blockIdx.x, gridDim.x) * kZWaves;
  if (g.perm != nullptr) {
    find_tile(g.order, g.norb, slot + g.order[0], b, t);
    b = __ldg(g.perm + b);
    slot = __ldg(g.prefix + b) + t;
  } else {
    find_tile(g.prefix, g.norb, slot, b, t);
  }
  b = __builtin_amdgcn_readfirstlane(b);
  t = __builtin_amdgcn_readfirstlane(t);
  slot = __builtin_amdgcn_readfirstlane(slot) + w;
  const OrbConst od = (OrbConst)g.orbs + b;
  K(g, a, buf, od, t, w).run(od, b, slot);
#endif
}

template <int P, int MODE>
hipError_t line_z_launch(int shape, const PassGeom& g, const ZLineArgs& a, int nblocks,
                         hipStream_t st) {
#define WVL_ZLINE(S)                                                                                \
  case S: {                                                                                         \
    using K = ZLine<P, kZShapes[S].U, kZShapes[S].mi, MODE>;                                        \
    const size_t lds = (size_t)a.rows * K::ST * sizeof(typename K::C);                         \
    hipLaunchKernelGGL((k_line_z<P, kZShapes[S].U, kZShapes[S].mi, MODE, kZShapes[S].wpe>),         \
                       dim3(nblocks), dim3(64 * kZWaves), lds, st, g, a);                                \
    break;                                                                                          \
  }
  switch (shape) {
    WVL_ZLINE(0) WVL_ZLINE(1) WVL_ZLINE(2) WVL_ZLINE(3) WVL_ZLINE(4) WVL_ZLINE(5)
    default: return hipErrorInvalidValue;
  }
#undef WVL_ZLINE
  return hipGetLastError();
}

}  // namespace wvl
