// Shared by the orthogonalisation kernels of the one-vector Arnoldi step
// (krylov_dot.hip, krylov_axpy.hip): launch shapes, and the coefficients that
// a kernel sums from its predecessor's partials.
#pragma once

#include "krylov_common.hpp"

namespace rsfde {

// Two shapes, chosen by the vector length:
//   up to kOrthSmallN values: one value per load, up to 128 blocks, and every
//     block of a consumer sums the producer's partials itself (at most 128
//     per coefficient), so a Gram-Schmidt pass has no finishing kernel;
//   beyond: two values per load, up to kMaxRedBlocks blocks, and a finishing
//     kernel sums the partials once (512 blocks each reading 512 partials per
//     coefficient cost 19 us a step at 2047^2).
// A two-pass step takes four launches in the first shape and six in the second
// (seven before, with one more read of the basis).  At 63^2 its kernel time went
// from 48 to 22 us, one implicit step there 2.75 -> 2.08 ms.
constexpr size_t kOrthSmallN = (size_t)1 << 18;
constexpr int kOrthSmallBlocks = 128;
inline bool orth_small(size_t N) { return N <= kOrthSmallN; }
inline int orth_blocks(size_t N) {
  if (!orth_small(N)) return red_blocks(N);
  const size_t b = (N + kRedThreads - 1) / kRedThreads;
  return b < 1 ? 1 : (b > (size_t)kOrthSmallBlocks ? kOrthSmallBlocks : (int)b);
}

// Partials of the two Gram-Schmidt passes.
static_assert(kRedSecond >= kChunk && kRedRows >= kRedSecond + kChunk,
              "two regions of kChunk rows in the reduction workspace");
__device__ __forceinline__ double* orth_partials(const RedWork& rw, bool second) {
  return rw.partial + (second ? (size_t)kRedSecond * kMaxRedBlocks : 0);
}

// W consecutive values of a vector.
template <int W>
struct Vals;
template <>
struct Vals<1> {
  double v[1];
  __device__ __forceinline__ void load(const double* p, size_t i) { v[0] = p[i]; }
  __device__ __forceinline__ void store(double* p, size_t i) const { p[i] = v[0]; }
};
template <>
struct Vals<2> {
  double v[2];
  __device__ __forceinline__ void load(const double* p, size_t i) {
    const double2 q = reinterpret_cast<const double2*>(p)[i];
    v[0] = q.x;
    v[1] = q.y;
  }
  __device__ __forceinline__ void store(double* p, size_t i) const {
    reinterpret_cast<double2*>(p)[i] = double2{v[0], v[1]};
  }
};

// c[v] = vscale[v]^2 * (sum of the nb <= 128 partials of value v), v < NV, in
// LDS for the whole block (8 lanes per value, fixed order); block 0 also stores
// the coefficient vscale[v] * sum to hout[v].  Ends with a barrier.
template <int NV>
__device__ __forceinline__ void gather_coefs(const double* part, int nb, const double* vscale,
                                             double* hout, double* c) {
  static_assert(8 * NV <= kRedThreads, "eight lanes per value");
  const int v = threadIdx.x >> 3, l = threadIdx.x & 7;
  double s = 0.0;
  if (v < NV) {
    double q[kOrthSmallBlocks / 8];
#pragma unroll
    for (int k = 0; k < kOrthSmallBlocks / 8; ++k) {
      const int b = l + 8 * k;
      q[k] = b < nb ? part[(size_t)v * kMaxRedBlocks + b] : 0.0;
    }
#pragma unroll
    for (int k = 0; k < kOrthSmallBlocks / 8; ++k) s += q[k];
  }
#pragma unroll
  for (int o = 4; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if (v < NV && l == 0) {
    const double sc = vscale[v], h = s * sc;
    c[v] = h * sc;
    if (blockIdx.x == 0) hout[v] = h;
  }
  __syncthreads();
}

}  // namespace rsfde
