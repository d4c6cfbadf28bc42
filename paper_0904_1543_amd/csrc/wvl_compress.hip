// Compressed storage of the orbitals: unpack onto the whole grid and pack
// back (steps 1 and 7 of the local Hamiltonian, Sec. 2.4), gfx950.
//
// Sec. 2.1: an orbital stores its scaling coefficient only at the coarse
// points of the low-resolution region and its seven wavelet coefficients only
// at the points of the high-resolution region.  The compressed vector of one
// orbital is [coarse-region scaling coefficients][7 per fine-region point];
// regions are given as segments of consecutive points along axis 1.  Both
// kernels are gathers, so every store is coalesced:
//  * decompress: one thread per coarse point, whose position and place in the
//    two regions (per-point maps, -1: not stored, value 0) serve all orbitals;
//    the thread reads its scaling value and its seven adjacent wavelet values
//    and stores four pairs of neighbours (256 float64 orbitals of 48^3 cells:
//    0.47 ms where one thread per element, bound by its divisions and by one
//    load and store each, took 0.81);
//  * compress: one thread per compressed element; the region's point list
//    gives the full-grid position to read.

#include "wvl_kernels.h"

namespace wvl {

template <int P>
__global__ __launch_bounds__(kThreads) void k_decompress(const OrbDev* __restrict__ orbs, int norb,
                                                         const int32_t* __restrict__ map_c,
                                                         const int32_t* __restrict__ map_f,
                                                         int64_t nvc, int64_t L, const void* in,
                                                         int64_t plane_in, void* out,
                                                         int64_t plane_out) {
  using T = Prec<P>;
  const OrbDev o0 = orbs[0];
  const uint32_t m1 = o0.m[0], m2 = o0.m[1];
  const uint32_t n1 = m1 >> 1, n2 = m2 >> 1, n = n1 * n2 * ((uint32_t)o0.m[2] >> 1);
  const uint32_t pnt = blockIdx.x * kThreads + threadIdx.x;
  if (pnt >= n) return;
  const int kc = map_c[pnt], kf = map_f[pnt];
  const uint32_t row = pnt / n1, i1 = pnt - row * n1, i2 = row % n2, i3 = row / n2;
  const int64_t e = ((int64_t)(2 * i3) * m2 + 2 * i2) * m1 + 2 * i1;
  const int64_t jf = nvc + 7 * (int64_t)kf;
  for (int b = blockIdx.y; b < norb; b += gridDim.y) {
    const int64_t src = (int64_t)b * L;
    typename T::W v[8] = {};
    if (kc >= 0) v[0] = T::ldw(in, src + kc, plane_in);
    if (kf >= 0)
      #pragma unroll
      for (int mu = 1; mu < 8; ++mu) v[mu] = T::ldw(in, src + jf + mu - 1, plane_in);
    const int64_t d = orbs[b].off + e;
    #pragma unroll
    for (int q = 0; q < 4; ++q)
      T::stw2(out, d + (int64_t)(q & 1) * m1 + (int64_t)(q >> 1) * m1 * m2, plane_out, v[2 * q], v[2 * q + 1]);
  }
}

template <int P>
__global__ __launch_bounds__(kThreads) void k_compress(const OrbDev* __restrict__ orbs, int norb,
                                                       const int32_t* __restrict__ list_c,
                                                       const int32_t* __restrict__ list_f,
                                                       int64_t nvc, int64_t L, const void* in,
                                                       int64_t plane_in, void* out,
                                                       int64_t plane_out) {
  using T = Prec<P>;
  const OrbDev o0 = orbs[0];
  const int m1 = o0.m[0], m2 = o0.m[1];
  const int n1 = m1 >> 1, n2 = m2 >> 1;
  const int64_t total = L * norb;
  for (int64_t g = (int64_t)blockIdx.x * kThreads + threadIdx.x; g < total;
       g += (int64_t)gridDim.x * kThreads) {
    const int b = (int)(g / L);
    const int64_t j = g - (int64_t)b * L;
    int pnt, mu;
    if (j < nvc) {
      pnt = list_c[j];
      mu = 0;
    } else {
      const int64_t k = (j - nvc) / 7;
      mu = (int)(j - nvc - 7 * k) + 1;
      pnt = list_f[k];
    }
    const int i1 = pnt % n1, r = pnt / n1;
    const int i2 = r % n2, i3 = r / n2;
    const int64_t e = ((int64_t)(2 * i3 + ((mu >> 2) & 1)) * m2 + (2 * i2 + ((mu >> 1) & 1))) * m1 +
                      2 * i1 + (mu & 1);
    T::stw(out, g, plane_out, T::ldw(in, orbs[b].off + e, plane_in));
  }
}

static unsigned grid_for(int64_t n) {
  int64_t blocks = (n + kThreads - 1) / kThreads;
  return (unsigned)(blocks > 65536 ? 65536 : (blocks < 1 ? 1 : blocks));
}

hipError_t launch_decompress(int prec, const OrbDev* orbs, int norb, int64_t M,
                             const int32_t* map_c, const int32_t* map_f, int64_t nvc, int64_t L,
                             const void* in, int64_t plane_in, void* out, int64_t plane_out,
                             hipStream_t st) {
  // orbitals in turn per thread, while 16 workgroups per compute unit remain
  const unsigned nb = (unsigned)((M / 8 + kThreads - 1) / kThreads);
  const dim3 g(nb, (unsigned)std::max<int64_t>(1, std::min<int64_t>(std::min(norb, 65535), 4096 / nb))), b(kThreads);
  switch (prec) {
    case F64: hipLaunchKernelGGL((k_decompress<F64>), g, b, 0, st, orbs, norb, map_c, map_f, nvc, L, in, plane_in, out, plane_out); break;
    case F32: hipLaunchKernelGGL((k_decompress<F32>), g, b, 0, st, orbs, norb, map_c, map_f, nvc, L, in, plane_in, out, plane_out); break;
    default:  hipLaunchKernelGGL((k_decompress<F32C>), g, b, 0, st, orbs, norb, map_c, map_f, nvc, L, in, plane_in, out, plane_out); break;
  }
  return hipGetLastError();
}

hipError_t launch_compress(int prec, const OrbDev* orbs, int norb, const int32_t* list_c,
                           const int32_t* list_f, int64_t nvc, int64_t L, const void* in,
                           int64_t plane_in, void* out, int64_t plane_out, hipStream_t st) {
  if (L == 0) return hipSuccess;
  const dim3 g(grid_for(L * norb)), b(kThreads);
  switch (prec) {
    case F64: hipLaunchKernelGGL((k_compress<F64>), g, b, 0, st, orbs, norb, list_c, list_f, nvc, L, in, plane_in, out, plane_out); break;
    case F32: hipLaunchKernelGGL((k_compress<F32>), g, b, 0, st, orbs, norb, list_c, list_f, nvc, L, in, plane_in, out, plane_out); break;
    default:  hipLaunchKernelGGL((k_compress<F32C>), g, b, 0, st, orbs, norb, list_c, list_f, nvc, L, in, plane_in, out, plane_out); break;
  }
  return hipGetLastError();
}

}  // namespace wvl
