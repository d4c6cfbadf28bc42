// The in-plane part of the local Hamiltonian, one z-plane at a time per
// workgroup, float64 and float32 FMA, gfx950.
//
// The 3D operators are tensor products of 1D operators (Sec. 3.1), so the
// local Hamiltonian of one orbital factorises along z:
//     psi = W_x W_y u,            u  = W_z c            (W = magic filter o synthesis)
//     Hc  = W_z^T t + K_z c + kxy, t = W_y^T W_x^T (V psi), kxy = (K_x + K_y) c
// with W^T = analysis o transposed magic filter and K = analysis o kinetic o
// synthesis (the combined filters of Sec. 2.4, last paragraph; the kinetic
// part uses A_a S_a = I on the other axes).  This kernel does everything that
// stays inside one z-plane, so a plane crosses HBM twice in and twice out.
//
// What bounds it: the FMA units.  A point takes 246 multiply-adds (4 x 32 taps
// of W and W^T, 2 x 59 of K) and about 85 other vector instructions.  Float64
// matrix instructions run on the same units at the same rate, block every
// other vector instruction of their SIMD while they run, and spend a third of
// their work on the zeros beside the band (and all of it on the padding of a
// ragged plane), so the passes are plain FMAs: 256 orbitals of 96^3 take 2.8 ms
// (40 TFLOP/s, the units busy 80% of the cycles) against 4.4 ms
// on the matrix instructions; 45 orbitals of 74 x 58 x 86 points 0.36 against
// 0.51 ms; float32, 64 orbitals of 64^3: 0.19 against 0.31 ms (vector passes
// of four outputs an item); 512 uneven orbitals of float pairs 5.2 against
// 27.2 ms.
#pragma once

#include <type_traits>
#include <utility>

#include "wvl_plane.h"

namespace wvl {

// Storage of a plane's values in memory and their type in LDS and registers:
// float pairs are widened to float64 on the way in (one FMA per tap; this
// chip's float64 FMA rate equals its float32 one, while pair arithmetic takes
// twelve float32 operations a tap) and split again on the way out.  Elements
// are addressed as a uniform base and a 32-bit byte offset; the vector types
// carry the alignment of one element, since an orbital may start anywhere.
template <int P> struct LineIO;
template <> struct LineIO<F64> {
  using C = double;
  struct Raw { d2u v; };
  __device__ static void pin(Raw& r) { asm volatile("" : "+v"(r.v)); }
  __device__ static const char* at(const void* p, int64_t i) { return (const char*)p + 8 * i; }
  __device__ static char* at(void* p, int64_t i) { return (char*)p + 8 * i; }
  __device__ static Raw ld2(const char* p, uint32_t i, int64_t) {
    return Raw{*reinterpret_cast<const d2u*>(p + 8u * i)};
  }
  __device__ static void cvt(const Raw& r, C& a, C& b) { a = r.v.x; b = r.v.y; }
  __device__ static void st2(char* p, uint32_t i, int64_t, C a, C b) {
    stream_st(reinterpret_cast<d2u*>(p + 8u * i), d2u{a, b});
  }
  __device__ static C ld(const char* p, uint32_t i, int64_t) {
    return *reinterpret_cast<const double*>(p + 8u * i);
  }
  __device__ static void st(char* p, uint32_t i, int64_t, C v) {
    stream_st(reinterpret_cast<double*>(p + 8u * i), v);
  }
  __device__ static void st_keep(char* p, uint32_t i, int64_t, C v) {
    *reinterpret_cast<double*>(p + 8u * i) = v;
  }
};
template <> struct LineIO<F32> {
  using C = float;
  struct Raw { f2u v; };
  __device__ static void pin(Raw& r) { asm volatile("" : "+v"(r.v)); }
  __device__ static const char* at(const void* p, int64_t i) { return (const char*)p + 4 * i; }
  __device__ static char* at(void* p, int64_t i) { return (char*)p + 4 * i; }
  __device__ static Raw ld2(const char* p, uint32_t i, int64_t) {
    return Raw{*reinterpret_cast<const f2u*>(p + 4u * i)};
  }
  __device__ static void cvt(const Raw& r, C& a, C& b) { a = r.v.x; b = r.v.y; }
  __device__ static void st2(char* p, uint32_t i, int64_t, C a, C b) {
    *reinterpret_cast<f2u*>(p + 4u * i) = f2u{a, b};
  }
  __device__ static C ld(const char* p, uint32_t i, int64_t) {
    return *reinterpret_cast<const float*>(p + 4u * i);
  }
  __device__ static void st(char* p, uint32_t i, int64_t, C v) {
    *reinterpret_cast<float*>(p + 4u * i) = v;
  }
  __device__ static void st_keep(char* p, uint32_t i, int64_t, C v) { st(p, i, 0, v); }
};
template <> struct LineIO<F32C> {
  using C = double;
  using S = LineIO<F32>;
  struct Raw { f2u h, l; };
  __device__ static void pin(Raw& r) { asm volatile("" : "+v"(r.h), "+v"(r.l)); }
  __device__ static const char* at(const void* p, int64_t i) { return S::at(p, i); }
  __device__ static char* at(void* p, int64_t i) { return S::at(p, i); }
  __device__ static Raw ld2(const char* p, uint32_t i, int64_t plane) {
    return Raw{S::ld2(p, i, 0).v, S::ld2(p + 4 * plane, i, 0).v};
  }
  __device__ static void cvt(const Raw& r, C& a, C& b) {
    a = (double)r.h.x + (double)r.l.x;
    b = (double)r.h.y + (double)r.l.y;
  }
  __device__ static void st2(char* p, uint32_t i, int64_t plane, C a, C b) {
    const float ha = (float)a, hb = (float)b;
    S::st2(p, i, 0, ha, hb);
    S::st2(p + 4 * plane, i, 0, (float)(a - (double)ha), (float)(b - (double)hb));
  }
  __device__ static C ld(const char* p, uint32_t i, int64_t plane) {
    return (double)S::ld(p, i, 0) + (double)S::ld(p + 4 * plane, i, 0);
  }
  __device__ static void st(char* p, uint32_t i, int64_t plane, C v) {
    const float h = (float)v;
    S::st(p, i, 0, h);
    S::st(p + 4 * plane, i, 0, (float)(v - (double)h));
  }
  __device__ static void st_keep(char* p, uint32_t i, int64_t plane, C v) { st(p, i, plane, v); }
};

// f(integral constant) for 0 .. N - 1: filter taps and window offsets are
// compile-time constants without a limit on the loop's size
template <typename F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
  static_for_(f, std::make_integer_sequence<int, N>{});
}

// LDS pointers (32-bit, so that window offsets become instruction offsets)
template <typename C> using Lds = __attribute__((address_space(3))) C*;

// which taps WO + 16 .. WO - 128 of an operator are not zero, per output parity
template <int OP>
struct LineTap {
  static constexpr int WO = (OpWin<OP>::OHI + 1) & ~1;    // window starts WO before the outputs
  static constexpr int NT = 128;
  bool on[2][NT + 16];
  constexpr LineTap() : on() {
    for (int p = 0; p < 2; ++p)
      for (int i = 0; i < NT + 16; ++i) {
        const int o = WO + i - NT;
        on[p][i] = o >= OpWin<OP>::OLO && o <= OpWin<OP>::OHI && coef<OP>(p, o, 0) != 0.0;
      }
  }
};
template <int OP> constexpr LineTap<OP> kLineTap = LineTap<OP>();

// Filter coefficients in the order line_conv takes them up: four per input
// pair, by one scalar load.  As literals they take two scalar moves each, a
// third of all instructions, and more of them are kept (and spilled) between
// passes: 3.10 against 3.04 ms on 256 orbitals of 96^3.
template <int OP, typename C>
struct LineCoef {
  static constexpr int OLO = OpWin<OP>::OLO, OHI = OpWin<OP>::OHI;
  static constexpr int WO = LineTap<OP>::WO, NT = LineTap<OP>::NT;
  static constexpr int NC = (WO - OLO + 3) / 2;        // groups that hold taps
  C v[NC][4];
  static constexpr C at(int p, int o) { return (C)coef<OP>(p, o, sizeof(C) == 4 ? 1 : 0); }
  constexpr LineCoef() : v() {
    for (int g = 0; g < NC; ++g) {
      v[g][0] = at(0, WO - 2 * g);
      v[g][1] = at(1, WO - 2 * g);
      v[g][2] = at(0, WO - 2 * g - 1);
      v[g][3] = at(1, WO - 2 * g + 1);
    }
  }
};
template <int OP, typename C> static __device__ const LineCoef<OP, C> kLineCoef = LineCoef<OP, C>();

__device__ __forceinline__ double line_fma(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float line_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// U consecutive outputs k0 .. k0 + U - 1 (k0 even) of operator OP on one
// periodic line of mc values in LDS (neighbours ST values apart).  The
// inputs k0 - WO ... are streamed in pairs; each is used by every output in
// its reach at once, so only the U sums stay in registers.  Pair g meets the
// taps WO - 2 g - 1 .. WO - 2 g + U - 1, of which it brings the lowest ones;
// the others have been loaded for earlier pairs.  mc and the start of the
// window are even: a pair never straddles the periodic wrap.
// PRIO: the wave's issue priority, one lower in the second half.
// FREE: an isolated line of mc inputs, output k at input position k + d (d
// even), zero outside: pairs outside read zeros at `zero` (and zero + ST);
// the value after a line of odd length is zero in LDS.
template <int OP, int U, int ST, int PRIO, bool FREE, typename C>
__device__ __forceinline__ void line_conv(Lds<C> line, int mc, int d, int k0, Lds<C> zero, C (&acc)[U]) {
  using K = LineCoef<OP, C>;
  constexpr int OLO = K::OLO, WO = K::WO;
  constexpr int NP = (WO + U - OLO + 1) / 2;      // pairs
  const __attribute__((address_space(4))) C* tab =
      (const __attribute__((address_space(4))) C*)&kLineCoef<OP, C>.v[0][0];
  asm volatile("" : "+s"(tab));      // loaded in this pass, not kept from another
  #pragma unroll
  for (int u = 0; u < U; ++u) acc[u] = C(0);
  __builtin_amdgcn_s_setprio(PRIO);
  C x0[2], x1[2];
  C cf[K::NC][4];
  auto coefs = [&](auto g) {
    if constexpr (g < K::NC) {
      #pragma unroll
      for (int j = 0; j < 4; ++j) cf[g][j] = tab[4 * g + j];
    }
  };
  auto run = [&](auto&& read) {
    // the next pair's inputs and coefficients are in flight while a pair is used
    read(std::integral_constant<int, 0>{});
    coefs(std::integral_constant<int, 0>{});
    static_for<NP>([&](auto g) {
      if constexpr (PRIO > 0 && g == NP / 2) __builtin_amdgcn_s_setprio(PRIO - 1);
      if constexpr (g + 1 < NP) {
        read(std::integral_constant<int, g + 1>{});
        coefs(std::integral_constant<int, g + 1>{});
      }
      // output u takes the tap WO - 2 g + u (one less for the second input),
      // whose group came u / 2 pairs ago
      #pragma unroll
      for (int u = 0; u < U; ++u)
        if (kLineTap<OP>.on[u & 1][u + K::NT - 2 * g])
          acc[u] = line_fma(cf[g - u / 2][u & 1 ? 3 : 0], x0[g % 2], acc[u]);
      #pragma unroll
      for (int u = 0; u < U; ++u)
        if (kLineTap<OP>.on[u & 1][u + K::NT - 2 * g - 1])
          acc[u] = line_fma(cf[g - u / 2][u & 1 ? 1 : 2], x1[g % 2], acc[u]);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  if constexpr (FREE) {
    const int s0 = k0 + d - WO;
    const Lds<C> A = line + s0 * ST;
    run([&](auto g) {
      const Lds<C> p = (unsigned)(s0 + 2 * g) < (unsigned)mc ? A + 2 * g * ST : zero;
      x0[g % 2] = p[0];
      x1[g % 2] = p[ST];
    });
  } else if (mc >= 2 * NP) {
    // at most one wrap: two bases, the pair index decides
    const int s0 = k0 < WO ? k0 - WO + mc : k0 - WO;
    const Lds<C> A = line + s0 * ST;
    const Lds<C> B = A - mc * ST;
    const int gs = (mc - s0) >> 1;
    run([&](auto g) {
      const Lds<C> p = g < gs ? A : B;
      x0[g % 2] = p[2 * g * ST];
      x1[g % 2] = p[2 * g * ST + ST];
    });
  } else {
    int s0 = k0 - WO;
    while (s0 < 0) s0 += mc;
    Lds<C> p = line + s0 * ST;
    const Lds<C> end = line + mc * ST;
    run([&](auto g) {
      x0[g % 2] = p[0];
      x1[g % 2] = p[ST];
      p += 2 * ST;
      p = p >= end ? p - mc * ST : p;
    });
  }
}

// ---------------------------------------------------------------------------
// The plane kernel.  A wave owns groups of whole rows in the x passes and of
// whole columns in the y passes; a line's segments of U outputs are lanes of
// that wave.  So a pass runs in place without a barrier (a wave reads all its
// inputs before it writes), a wave loads and stores its own rows, and the
// workgroup meets only where rows turn into columns and back.  Two plane
// buffers A (u, psi, y, t) and B (c, kxy):
//   rows:     u -> A, W_x;  c -> B, K_x c kept in registers
//   columns:  A: W_y, pointwise, W_y^T;  B: K_y c
//   rows:     A: W_x^T, t out;  B: + K_x c, kxy out;  then the next plane's rows
// Two barriers a plane.  Planes too large for two buffers use one, with c
// after t (four barriers).
//
// Isolated axes (FREE: 1 axis 1, 2 axis 2; Sec. 3.1): lines of m coefficients
// become m + 29 real-space points and back, so psi fills M1 x M2 = (m1 + 29) x
// (m2 + 29) points of the plane buffer, whose two rows after the last one stay
// zero (as does the value after each row).  u and t then have M3 planes and c m3,
// so K c is a launch of its own (HELM).
// ---------------------------------------------------------------------------
typedef const __attribute__((address_space(4))) OrbDev* OrbConst;

// what a plane needs of its orbital, read through the constant address space
// (scalar loads, which do not wait for the planes' memory operations in
// flight) once per plane
struct LineOrb {
  int64_t off, voff;
  double ks1, ks2, occ;
  __device__ __forceinline__ explicit LineOrb(OrbConst o)
      : off(o->off), voff(o->voff), ks1(o->kscale[0]), ks2(o->kscale[1]), occ(o->occ) {}
};

// lanes of one wave exchange values through LDS in program order: only the
// compiler has to keep that order
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int P, int PITCH, int U, int MI, bool TWO, int MODE, bool SHARED, int FREE>
struct LineKernel {
  using IO = LineIO<P>;
  using C = typename IO::C;
  using Raw = typename IO::Raw;
  // H*psi with K c beside u in the second buffer, or after t in the only one
  static constexpr bool KC = MODE == LINE_HPSI && TWO && !FREE, KC1 = MODE == LINE_HPSI && !TWO && !FREE;
  static constexpr bool UT = MODE == LINE_HPSI && !KC1;   // the next u is loaded before t goes out
  static constexpr int NPF = U / 2;        // pairs of a group of rows per lane at most
  static constexpr int NW = 16;            // waves at most

  const XyArgs& a;
  Lds<C> A, B;
  Lds<double> red;
  Lds<C> zero;
  int m1, m2, M1, M2, nw;
  // this lane's place in a group of rows (x) and of columns (y): line within
  // the group and first output; lines per group; this wave
  int xl, xk, yl, yk, rw, cw, w;
  int lo[NPF];

  __device__ __forceinline__ LineKernel(const XyArgs& a_, Lds<C> lds, Lds<double> r, OrbConst od)
      : a(a_), A(lds), red(r), m1(od->m[0]), m2(od->m[1]), nw(blockDim.x >> 6) {
    M1 = m1 + line_extra(MODE, FREE & 1);
    M2 = m2 + line_extra(MODE, FREE & 2);
    zero = lds + M2 * PITCH;
    B = TWO && !FREE ? lds + m2 * PITCH : lds;
    if (FREE) {
      for (int i = threadIdx.x; i < 2 * PITCH; i += blockDim.x) zero[i] = C(0);
      for (int i = threadIdx.x; i < M2; i += blockDim.x) lds[i * PITCH + M1] = C(0);   // M1 < PITCH
      __syncthreads();
    }
    w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int nsx = (M1 + U - 1) / U, nsy = (M2 + U - 1) / U;
    rw = line_lines(U, nsx);
    cw = line_lines(U, nsy);
    constexpr int SB = line_sub(U);
    if constexpr (SB > 0) {     // lane = (line sub-block, segment, line in it)
      const int r = lane / SB, l = lane - r * SB;
      const int bx = r / nsx, by = r / nsy;
      xl = bx * SB + l;
      xk = xl < rw ? r - bx * nsx : nsx;
      yl = by * SB + l;
      yk = yl < cw ? r - by * nsy : nsy;
    } else {                    // lane = (segment, line)
      xk = lane / rw;
      xl = lane - xk * rw;
      yk = lane / cw;
      yl = lane - yk * cw;
    }
    // idle lanes (past the last segment): a line outside every group
    if (xk >= nsx) { xl = 1 << 20; xk = 0; }
    if (yk >= nsy) { yl = 1 << 20; yk = 0; }
    xk *= U;
    yk *= U;
    const int h = m1 >> 1;
    int r0 = lane / h, c0 = lane - r0 * h;
    const int dr = 64 / h, dc = 64 - dr * h;
    #pragma unroll
    for (int n = 0; n < NPF; ++n) {
      lo[n] = r0 * PITCH + 2 * c0;
      r0 += dr;
      c0 += dc;
      if (c0 >= h) { c0 -= h; ++r0; }
    }
  }
  // Group i of this wave along axis AX: first line, and the number of lines
  // (0: none).
  template <int AX> __device__ __forceinline__ int first(int i) const { return (w + i * nw) * (AX == 1 ? rw : cw); }
  template <int AX> __device__ __forceinline__ int count(int i) const {
    return max(0, min(AX == 1 ? rw : cw, (AX == 1 ? m2 : M1) - first<AX>(i)));
  }
  // This lane's line (or -1) and first output in group i.  Opaque to the
  // optimiser: window offsets and wrap conditions are computed inside each
  // pass instead of being hoisted out of the loop over a group's orbitals
  // (and kept live, or spilled, across it).
  struct Item { int line, k0; bool on; };
  template <int AX> __device__ __forceinline__ Item item(int i) const {
    int l = AX == 1 ? xl : yl, k0 = AX == 1 ? xk : yk;
    asm volatile("" : "+v"(l), "+v"(k0));
    return Item{first<AX>(i) + l, k0, l < count<AX>(i)};
  }

  // first row of group i in a plane buffer (opaque: as in item())
  __device__ __forceinline__ Lds<C> rows(Lds<C> buf, int i) const {
    int r = first<1>(i) * PITCH;
    asm volatile("" : "+s"(r));
    return buf + r;
  }
  // Pairs of a group of rows: lane l takes pairs l + 64 n, addressed as a
  // uniform base per n and the lane's offset, clamped to the last pair (no
  // branch around a load; !any: one pair for everybody, nothing to load).
  __device__ __forceinline__ void load(const void* src, int64_t plane, int64_t gp, int i, Raw (&r)[NPF],
                                       bool any) const {
    int t = threadIdx.x & 63;
    asm volatile("" : "+v"(t));      // offsets are not kept across the loop
    const int lim = any ? max(0, (count<1>(i) * m1 >> 1) - 1) : 0;
    const int64_t g0 = gp + (any ? min(first<1>(i), m2 - 1) * m1 : 0);
    #pragma unroll
    for (int n = 0; n < NPF; ++n) {
      const int s = min(n * 64, lim);
      r[n] = IO::ld2(IO::at(src, g0 + 2 * s), 2u * min(t, lim - s), plane);
    }
  }
  __device__ __forceinline__ void put(Lds<C> buf, int i, const Raw (&r)[NPF]) const {
    const int np = count<1>(i) * m1 >> 1;
    const Lds<C> d = rows(buf, i);
    const int t = threadIdx.x & 63;
    #pragma unroll
    for (int n = 0; n < NPF; ++n)
      if (t < np - n * 64) {
        C v0, v1;
        IO::cvt(r[n], v0, v1);
        d[lo[n]] = v0;
        d[lo[n] + 1] = v1;
      }
  }
  __device__ __forceinline__ void copy_out(Lds<C> buf, int i, void* dst, int64_t plane, int64_t gp) const {
    int t = threadIdx.x & 63;
    asm volatile("" : "+v"(t));
    const int np = count<1>(i) * m1 >> 1;
    const Lds<C> d = rows(buf, i);
    const int64_t g0 = gp + first<1>(i) * m1;
    #pragma unroll
    for (int n = 0; n < NPF; ++n)
      if (t < np - n * 64) IO::st2(IO::at(dst, g0 + 128 * n), 2u * t, plane, d[lo[n]], d[lo[n] + 1]);
  }
  // wait for loaded pairs here
  __device__ __forceinline__ static void arrive(Raw (&r)[MI][NPF]) {
    #pragma unroll
    for (int i = 0; i < MI; ++i)
      #pragma unroll
      for (int n = 0; n < NPF; ++n) IO::pin(r[i][n]);
  }

  // lengths along AX of the inputs and outputs of OP
  template <int OP, int AX> __device__ __forceinline__ int len_in() const {
    return AX == 1 ? (OP == OP_CWT ? M1 : m1) : (OP == OP_CWT ? M2 : m2);
  }
  template <int OP, int AX> __device__ __forceinline__ int len_out() const {
    return AX == 1 ? (OP == OP_CW ? M1 : m1) : (OP == OP_CW ? M2 : m2);
  }
  template <int OP, int AX> __device__ __forceinline__ void conv(Lds<C> src, int i, C (&r)[U]) const {
    // idle lanes repeat the group's first line (their results are not used):
    // no branch, so that nothing has to be kept for the lanes around it
    const Item m = item<AX>(i);
    const int line = m.on ? m.line : first<AX>(i);
    // The SIMD issues its oldest wave first; left alone, the waves of a
    // workgroup reach the barrier one after the other and the last one runs
    // by itself, with every latency exposed.  Priorities fall along a phase
    // (W^T then W then K by rows, W then W^T then K by columns), so that waves
    // behind catch up.
    constexpr int prio = OP == OP_CK ? 1 : (OP == OP_CW) == (AX == 2) ? 3 : 2;
    constexpr bool fr = (FREE & AX) != 0;
    constexpr int d = !fr || OP == OP_CK ? 0 : OP == OP_CW ? -14 : 14;
    const int n = len_in<OP, AX>();
    if (AX == 1) line_conv<OP, U, 1, prio, fr>(src + line * PITCH, n, d, m.k0, zero, r);
    else line_conv<OP, U, PITCH, prio, fr>(src + line, n, d, m.k0, zero, r);
  }
  // f(u, position in the plane buffer, row, column) for this lane's outputs of OP
  template <int OP, int AX, typename F> __device__ __forceinline__ void each(int i, F&& f) const {
    const Item m = item<AX>(i);
    if (!m.on || (FREE && OP == OP_CK && AX == 2 && m.line >= m1)) return;
    const int mc = len_out<OP, AX>();
    const int p0 = AX == 1 ? m.line * PITCH + m.k0 : m.k0 * PITCH + m.line;
    constexpr int es = AX == 1 ? 1 : PITCH;
    if (m.k0 + U <= mc) {
      #pragma unroll
      for (int u = 0; u < U; ++u) f(u, p0 + u * es, AX == 1 ? m.line : m.k0 + u, AX == 1 ? m.k0 + u : m.line);
    } else {
      #pragma unroll
      for (int u = 0; u < U; ++u)
        if (m.k0 + u < mc) f(u, p0 + u * es, AX == 1 ? m.line : m.k0 + u, AX == 1 ? m.k0 + u : m.line);
    }
  }
  template <int OP, int AX>
  __device__ __forceinline__ void store(Lds<C> dst, int i, const C (&r)[U]) const {
    wave_sync();
    each<OP, AX>(i, [&](int u, int pos, int, int) { dst[pos] = r[u]; });
    wave_sync();
  }
  // one pass in place
  template <int OP, int AX> __device__ __forceinline__ void pass(Lds<C> buf, int i) const {
    C r[U];
    conv<OP, AX>(buf, i, r);
    store<OP, AX>(buf, i, r);
  }
  // r = s K x along AX for group i, and e += <x, r>
  template <int AX>
  __device__ __forceinline__ void kinetic(Lds<C> buf, int i, C s, C (&r)[U], double& e) const {
    conv<OP_CK, AX>(buf, i, r);
    #pragma unroll
    for (int u = 0; u < U; ++u) r[u] *= s;
    each<OP_CK, AX>(i, [&](int u, int pos, int, int) { e = __builtin_fma((double)buf[pos], (double)r[u], e); });
  }
  // the potential at the outputs of group i of columns (zero past the plane
  // and for idle lanes)
  __device__ __forceinline__ void load_v(const char* Vp, int i, double (&v)[U]) const {
    const Item m = item<2>(i);
    const int x = m.on ? m.line : 0, mc = m.on ? M2 : 0;
    #pragma unroll
    for (int u = 0; u < U; ++u) {
      const double q = *reinterpret_cast<const double*>(Vp + 8u * (uint32_t)(min(m.k0 + u, M2 - 1) * M1 + x));
      v[u] = m.k0 + u < mc ? q : 0.0;
    }
  }

  __device__ __forceinline__ static double wave_sum(double v) {
    #pragma unroll
    for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s, 64);
    return v;
  }
  // the plane's two energies: sums per wave now (slot of the plane's parity),
  // over the waves in index order after the next barrier
  __device__ __forceinline__ void energies(double ep, double ek, int par) const {
    ep = wave_sum(ep);
    ek = wave_sum(ek);
    if ((threadIdx.x & 63) == 0) {
      red[(2 * par) * NW + w] = ep;
      red[(2 * par + 1) * NW + w] = ek;
    }
  }
  __device__ __forceinline__ void write_energies(int b, int z, int par) const {
    if (threadIdx.x != 0) return;
    const int64_t slot = ((const __attribute__((address_space(4))) int32_t*)a.pq)[b] + z;
    double p = 0.0, k = 0.0;
    for (int i = 0; i < nw; ++i) {
      p += red[(2 * par) * NW + i];
      k += red[(2 * par + 1) * NW + i];
    }
    if (MODE == LINE_HPSI) a.epot[FREE ? (int64_t)b * a.m3_rs + z : slot] = p;
    if (MODE == LINE_HELM || !FREE) a.ekin[slot] = k;
  }

  // The planes z of orbitals b0 .. b1 - 1 in turn (one orbital at least).
  __device__ __forceinline__ void planes(int b0, int b1, int z, double (&rho)[MI][U]) const {
    const int64_t zo = (int64_t)z * (m1 * m2);
    const OrbConst orbs = (OrbConst)a.orbs;
    // u and t of orbital b (isolated axes: m3_rs planes an orbital)
    auto uoff = [&](int b) {
      return FREE && MODE != LINE_HELM ? (int64_t)b * a.m3_rs * (m1 * m2) + zo : orbs[b].off + zo;
    };
    const int64_t plane_u = FREE && MODE != LINE_HELM ? a.plane_u : a.plane;
    Raw ru[MI][NPF], rc[MI][NPF];   // (HELM: ru is kq)
    #pragma unroll
    for (int i = 0; i < MI; ++i) {
      if (MODE == LINE_HELM) load(a.c, a.plane, orbs[b0].off + zo, i, rc[i], true);
      else load(a.u, plane_u, uoff(b0), i, ru[i], true);
    }
    if (MODE != LINE_HELM) arrive(ru);
    #pragma nounroll
    for (int b = b0; b < b1; ++b) {
      const LineOrb o(orbs + b);
      const int64_t gp = o.off + zo;
      const bool more = b + 1 < b1;
      const int64_t gu = uoff(b), gn = uoff(more ? b + 1 : b);
      const double pot_scale = a.occ_weight ? a.pot_scale * o.occ : a.pot_scale;
      const C km = (C)(a.occ_weight ? a.kin_mul * o.occ : a.kin_mul);
      const int par = b & 1;
      double ep = 0.0, ek = 0.0;
      C kx[MI][U];
      // ---- rows: W_x u, K_x c
      #pragma unroll
      for (int i = 0; i < MI; ++i) {
        if (count<1>(i) == 0) break;
        wave_sync();
        if (MODE != LINE_HELM) {
          put(A, i, ru[i]);
          wave_sync();
          if (KC) load(a.c, a.plane, gp, i, rc[i], true);
          pass<OP_CW, 1>(A, i);
        }
        if (MODE == LINE_HELM || KC) {
          put(B, i, rc[i]);
          wave_sync();
          kinetic<1>(B, i, (C)o.ks1, kx[i], ek);
          if (MODE == LINE_HELM && P != F32 && a.eps) {   // p is still in B
            const C ep = (C)((const __attribute__((address_space(4))) double*)a.eps)[b];
            each<OP_CK, 1>(i, [&](int u, int pos, int, int) { kx[i][u] -= ep * B[pos]; });
          }
        }
      }
      if (MODE == LINE_HELM) {   // kq and the next plane arrive behind the columns
        #pragma unroll
        for (int i = 0; i < MI; ++i) {
          load(a.kxy, a.plane, gp, i, ru[i], true);
          load(a.c, a.plane, gn, i, rc[i], more);
        }
      }
      __syncthreads();
      // ---- columns: W_y; rho (in orbital order), e_pot, y = pot_scale V psi;
      //      W_y^T; K_y c
      #pragma unroll
      for (int i = 0; i < MI; ++i) {
        if (count<2>(i) == 0) break;
        if (MODE != LINE_HELM) {
          C r[U];
          double v[U];
          if (MODE == LINE_HPSI)
            load_v((const char*)(a.V + o.voff + (int64_t)z * (M1 * M2)), i, v);
          conv<OP_CW, 2>(A, i, r);
          const bool fst = b == b0;
          #pragma unroll
          for (int u = 0; u < U; ++u) {
            const double pd = (double)r[u];
            if (SHARED) rho[i][u] = __builtin_fma(o.occ * pd, pd, fst ? 0.0 : rho[i][u]);
            if (MODE == LINE_HPSI) {
              ep = __builtin_fma(v[u] * pd, pd, ep);
              r[u] *= (C)(v[u] * pot_scale);
            }
          }
          if (MODE == LINE_HPSI) {
            store<OP_CW, 2>(A, i, r);
            pass<OP_CWT, 2>(A, i);
          }
        }
        if (MODE == LINE_HELM || KC) {
          C r[U];
          kinetic<2>(B, i, (C)o.ks2, r, ek);
          store<OP_CK, 2>(B, i, r);
        }
      }
      // (the next plane's rows are loaded as late as the registers allow)
      if (MODE == LINE_RHO || UT) {
        #pragma unroll
        for (int i = 0; i < MI; ++i) load(a.u, plane_u, gn, i, ru[i], more);
      }
      if (MODE == LINE_HELM || UT) energies(ep, ek, par);
      __syncthreads();
      if (MODE == LINE_RHO) continue;
      if (MODE == LINE_HELM || UT) write_energies(b, z, par);
      // ---- rows: W_x^T, t out; kxy out
      if (MODE == LINE_HPSI) {
        if (KC1) {
          #pragma unroll
          for (int i = 0; i < MI; ++i) load(a.c, a.plane, gp, i, rc[i], true);
        }
        #pragma unroll
        for (int i = 0; i < MI; ++i)
          if (count<1>(i) > 0) pass<OP_CWT, 1>(A, i);
        // the pairs in flight arrive before the stores (whose completion their
        // first use would otherwise wait for: memory operations are counted
        // in order)
        arrive(KC1 ? rc : ru);
      }
      if (MODE == LINE_HELM) {
        arrive(ru);
        arrive(rc);
      }
      #pragma unroll
      for (int i = 0; i < MI; ++i) {
        if (count<1>(i) == 0) break;
        if (MODE == LINE_HPSI) {
          copy_out(A, i, a.t, plane_u, gu);
          if (KC) kxy_out(i, kx[i], km, gp);
        } else {
          helm_out(i, kx[i], km, gp, ru[i]);
        }
      }
      if (KC1) {
        // one buffer: c after t
        #pragma unroll
        for (int i = 0; i < MI; ++i) {
          if (count<1>(i) == 0) break;
          wave_sync();
          put(A, i, rc[i]);
          wave_sync();
          kinetic<1>(A, i, (C)o.ks1, kx[i], ek);
        }
        __syncthreads();
        #pragma unroll
        for (int i = 0; i < MI; ++i) {
          if (count<2>(i) == 0) break;
          C r[U];
          kinetic<2>(A, i, (C)o.ks2, r, ek);
          store<OP_CK, 2>(A, i, r);
        }
        energies(ep, ek, par);
        __syncthreads();
        write_energies(b, z, par);
        #pragma unroll
        for (int i = 0; i < MI; ++i) {
          load(a.u, plane_u, gn, i, ru[i], more);
          if (count<1>(i) == 0) continue;
          kxy_out(i, kx[i], km, gp);
        }
      }
    }
  }
  // kxy = km (K_x c + K_y c), the latter in B
  __device__ __forceinline__ void kxy_out(int i, const C (&kx)[U], C km, int64_t gp) const {
    each<OP_CK, 1>(i, [&](int u, int pos, int, int) { B[pos] = km * (kx[u] + B[pos]); });
    wave_sync();
    copy_out(B, i, a.kxy, a.plane, gp);
  }
  // kq = km (kq + (K_x + K_y) p)
  __device__ __forceinline__ void helm_out(int i, const C (&kx)[U], C km, int64_t gp,
                                           const Raw (&q)[NPF]) const {
    each<OP_CK, 1>(i, [&](int u, int pos, int, int) { B[pos] += kx[u]; });
    wave_sync();
    const int np = count<1>(i) * m1 >> 1;
    const Lds<C> d = rows(B, i);
    const int64_t g0 = gp + first<1>(i) * m1;
    const int t = threadIdx.x & 63;
    #pragma unroll
    for (int n = 0; n < NPF; ++n)
      if (t < np - n * 64) {
        C v0, v1;
        IO::cvt(q[n], v0, v1);
        IO::st2(IO::at(a.kxy, g0 + 128 * n), 2u * t, a.plane, km * (v0 + d[lo[n]]), km * (v1 + d[lo[n] + 1]));
      }
  }
};

// Grid: shared potential: blockIdx.x = z * ngroups + g, the orbitals of group
// g in turn (the density of the group's plane stays in registers and is
// written once; HELM: the next orbital's plane is loaded behind this one's
// columns); otherwise one (orbital, plane) per tile of the prefix pq.
template <int P, int PITCH, int U, int MI, bool TWO, int MODE, bool SHARED, int FREE, int NT, int WPE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
void k_line(XyArgs a) {
#ifdef __HIP_DEVICE_COMPILE__   // (the host pass would instantiate all of it for nothing)
  using K = LineKernel<P, PITCH, U, MI, TWO, MODE, SHARED, FREE>;
  using C = typename K::C;
  extern __shared__ __align__(16) unsigned char line_lds[];
  __shared__ double red[4 * K::NW];
  const Lds<C> lds = (Lds<C>)reinterpret_cast<C*>(line_lds);
  const Lds<double> rd = (Lds<double>)red;
  double rho[MI][U];
  if (SHARED) {
    const int g = blockIdx.x % a.ngroups, z = blockIdx.x / a.ngroups;
    const int b0 = g * a.G, b1 = min(b0 + a.G, a.norb);
    const K k(a, lds, rd, (OrbConst)a.orbs + b0);
    k.planes(b0, b1, z, rho);
    if (MODE == LINE_HELM) return;
    double* rp = a.rho_part + (int64_t)g * a.M + (int64_t)z * (k.M1 * k.M2);
    #pragma unroll
    for (int i = 0; i < MI; ++i)
      k.template each<OP_CW, 2>(i, [&](int u, int, int y, int x) { rp[y * k.M1 + x] = rho[i][u]; });
  } else {
    __shared__ int s_tile;
    for (int vt = blockIdx.x;;) {
      if (a.queue != nullptr) {
        __syncthreads();   // the previous tile is finished and s_tile has been read
        if (threadIdx.x == 0) s_tile = atomicAdd(a.queue, 1);
        __syncthreads();
        vt = s_tile;
        if (vt >= a.ntiles) break;
      }
      int r, z;
      find_tile(a.order, a.norb, vt + a.order[0], r, z);
      const int b = __builtin_amdgcn_readfirstlane(a.perm[r]);
      const K k(a, lds, rd, (OrbConst)a.orbs + b);
      k.planes(b, b + 1, __builtin_amdgcn_readfirstlane(z), rho);
      if (a.queue == nullptr) break;
    }
  }
#endif
}

template <int P, int MODE, bool SH, int FREE>
hipError_t line_launch(int shape, const XyArgs& a, int nblocks, int nt, size_t lds, hipStream_t st) {
  const dim3 g(nblocks), b(nt);
#define WVL_LINE(S)                                                                              \
  case S:                                                                                        \
    hipLaunchKernelGGL((k_line<P, kLineShapes[S].pitch, kLineShapes[S].U, kLineShapes[S].mi,      \
                               kLineShapes[S].two != 0, MODE, SH, FREE, kLineShapes[S].nt,       \
                               kLineShapes[S].wpe>), g, b, lds, st, a);                          \
    break;
  switch (shape) {
    WVL_LINE(0) WVL_LINE(1) WVL_LINE(2) WVL_LINE(3) WVL_LINE(4)
    default: return hipErrorInvalidValue;
  }
#undef WVL_LINE
  return hipGetLastError();
}

}  // namespace wvl
