// Device helpers and launch shapes shared by the in-plane kernels.
#pragma once

#include "wvl_kernels.h"

namespace wvl {

// parts of a plane the plane kernel runs: the whole local H*psi, only the
// density, or the preconditioner's in-plane operator
enum { LINE_HPSI = 0, LINE_RHO = 1, LINE_HELM = 2 };
constexpr int kFreeExtra = 29;   // real-space points added along an isolated axis
// ... in the plane buffer of a launch (K alone stays on the coefficients)
__host__ __device__ constexpr int line_extra(int mode, int isolated) {
  return isolated && mode != LINE_HELM ? kFreeExtra : 0;
}

constexpr int kXyThreads = 512;   // threads of an in-plane workgroup (8 waves)
constexpr int kXyWaves = kXyThreads / 64;
constexpr int kU = 4;             // outputs per work item of the vector engine
constexpr int kMaxItems = 8;      // vector-engine work items per thread and pass (m <= 128)

// Points of the plane owned by this thread: e = threadIdx.x + k * kXyThreads,
// with its LDS position y * pitch + x stepped incrementally.
struct PtIter {
  int e, x, y, dx, dy, m1;
  __device__ PtIter(int m1_) : m1(m1_) {
    e = threadIdx.x;
    x = threadIdx.x % m1_;
    y = threadIdx.x / m1_;
    dx = kXyThreads % m1_;
    dy = kXyThreads / m1_;
  }
  __device__ int pos(int pitch) const { return y * pitch + x; }
  __device__ void next() {
    e += kXyThreads;
    x += dx;
    y += dy;
    if (x >= m1) { x -= m1; ++y; }
  }
};

// Visit the points of the plane owned by this thread in batches of B: the
// B global loads of a batch (load(e)) are issued before any of them is used
// (use(e, pos, value)), so their latencies overlap instead of adding up.
template <int B, typename L, typename U>
__device__ __forceinline__ void plane_batched(int m1, int npl, int pitch, L&& load, U&& use) {
  PtIter q(m1);
  while (q.e < npl) {
    decltype(load(0)) v[B];
    int e[B], pos[B];
    #pragma unroll
    for (int k = 0; k < B; ++k) {
      e[k] = q.e;
      pos[k] = q.pos(pitch);
      if (q.e < npl) v[k] = load(q.e);
      q.next();
    }
    #pragma unroll
    for (int k = 0; k < B; ++k)
      if (e[k] < npl) use(e[k], pos[k], v[k]);
  }
}
constexpr int kPlaneBatch = 8;

__device__ __forceinline__ double xy_block_sum(double v) {
  __shared__ double red[kXyThreads / 64];
  #pragma unroll
  for (int s = 32; s > 0; s >>= 1) v += __shfl_xor(v, s, 64);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  if (lane == 0) red[wid] = v;
  __syncthreads();
  double t = 0.0;
  #pragma unroll
  for (int w = 0; w < kXyThreads / 64; ++w) t += red[w];
  __syncthreads();
  return t;
}

// Launch shapes of the plane kernel: the first that fits.  A shape fits when
// its rows (pitch) hold m1 values, mi groups of lines per wave cover the
// plane with at most nt threads, and the plane buffers (two, or one) fit the
// LDS.  U, the outputs of a work item: 12 at 96 points a line (8 segments,
// 161 registers, 3 waves per SIMD), less for shorter lines so that they fill
// the lanes and registers allow 4 waves per SIMD (wpe).  16 outputs would
// need more coefficients in scalar registers than there are.
struct LineShape { int pitch, U, mi, two, nt, wpe; };
constexpr LineShape kLineShapes[] = {{33, 8, 1, 1, 512, 4}, {65, 8, 1, 1, 1024, 4}, {81, 10, 1, 1, 768, 4},
                                     {97, 12, 1, 1, 768, 3}, {129, 8, 2, 0, 1024, 4}};
// Lanes of a wave over `ns` segments a line and line_lines() lines: 16
// consecutive lanes (what the LDS serves at a time in float64) fall on
// distinct banks when they are 4 lines x 4 segments of 12, 2 lines x 8
// segments of 10, or 8 or 16 lines x segments of 8 (odd line pitch).
constexpr int line_sub(int U) { return U == 12 ? 4 : U == 10 ? 2 : 0; }
__host__ __device__ inline int line_lines(int U, int ns) {
  const int sb = line_sub(U);
  return sb > 0 ? sb * (64 / sb / ns) : 64 / ns;
}
constexpr int kNumLineShapes = sizeof(kLineShapes) / sizeof(kLineShapes[0]);

// z passes with whole lines in LDS (wvl_line_z.h): W, W^T and K along z, the
// last z step of H*psi, K with the preconditioner's direction update
enum { ZL_CW = 0, ZL_CWT = 1, ZL_CK = 2, ZL_FINAL = 3, ZL_CG = 4 };
// Shapes: lines of up to 4 U mi values (U outputs a segment, mi groups of four
// segments); the first that fits.  wpe: waves per SIMD that the registers and
// (last shape) the LDS allow.
constexpr int kZWaves = 4;   // waves of a workgroup, each 16 lines
constexpr int kZLines = 16 * kZWaves;   // a lane loads one of them
static_assert(kZLines == 64, "a wave loads a row of the tile");
struct ZShape { int U, mi, wpe; };
constexpr ZShape kZShapes[] = {{8, 1, 4}, {8, 2, 4}, {10, 2, 3}, {12, 2, 3}, {10, 3, 3},
                                {12, 3, 2}};
constexpr int kNumZShapes = sizeof(kZShapes) / sizeof(kZShapes[0]);
inline int line_z_shape(int m) {
  for (int s = 0; s < kNumZShapes; ++s)
    if (m <= 4 * kZShapes[s].U * kZShapes[s].mi) return s;
  return -1;
}
// Whether a uniform batch of lines of m values, `blocks` times kThreads of them,
// takes them rather than the strided passes, which read a line's first window
// twice but leave no lane idle and keep more waves in flight.  Times of the last
// z step, here / strided:
//   float pairs, any length: 0.84 .. 1.0 (W, W^T and K each);
//   float64: 64 orbitals of 36 x 20 cells and 82 values 118 / 137 us, 98 values
//   194 / 154; of 56^3 cells 892 / 686;
//   float32: 64 orbitals of 64^3 points 72 / 80 us, of 80^3 129 / 148; of 72 x 40
//   planes, 66 values 66 / 54 us, 82 values 75 / 63, 98 values 109 / 72; of
//   144 x 20 planes, 8 values 29 / 18, 40 values 52 / 37: seven of eight lanes
//   busy, and not the shapes of more than 80 values, whose registers leave fewer
//   waves.  The shortest shape also where the strided passes would cut their
//   lines (H*psi of 200 orbitals of 16^3 points 58 / 62 us; of 40 x 60 x 16,
//   where they would not, 228 / 208).
// (Batches of several lengths: 0.9 .. 1.1 either way; they take the classes.)
inline bool line_z_pays(int prec, int m, int64_t blocks) {
  const int s = line_z_shape(m);
  if (s < 0 || prec == F32C) return s >= 0;
  if (prec == F64) return m <= 96;
  if (s == 0) return m >= 24 || blocks < kZTiles;
  return m <= 80 && 8 * m >= 7 * 4 * kZShapes[s].U * kZShapes[s].mi;
}

}  // namespace wvl
