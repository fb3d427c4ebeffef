// Device helpers shared by the streaming Krylov kernels: wavefront and block
// sums and the deterministic "last block finishes" grid reduction.
#pragma once

#include <math.h>

#include <array>
#include <utility>

#include "internal.hpp"

namespace rsfde {

// ------------------------------ helpers -----------------------------------

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Sum NV per-thread values over the block and publish them as the block's
// partials, part[v * kMaxRedBlocks + blockIdx.x] (plain stores; the kernel that
// reads them runs after this one, so the kernel boundary orders them and no
// device-scope fence is needed).  Within a wavefront the values are reduced
// together: each of the first log2 NV butterfly steps halves the values a lane
// still carries (it sends one half and keeps the other), so NV values take
// about NV shuffles instead of 6 NV.
template <int NV>
__device__ __forceinline__ void publish_partials(const double (&acc)[NV], double* part,
                                                 double* sh /* [16 * NV] */) {
  constexpr int LG = NV <= 1 ? 0 : NV <= 2 ? 1 : NV <= 4 ? 2 : NV <= 8 ? 3 : NV <= 16 ? 4 : 5;
  constexpr int P2 = 1 << LG;
  static_assert(NV <= P2, "at most 32 values");
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  double a[P2];
#pragma unroll
  for (int v = 0; v < P2; ++v) a[v] = v < NV ? acc[v < NV ? v : 0] : 0.0;
#pragma unroll
  for (int k = 0; k < LG; ++k) {
    const int n = P2 >> (k + 1);
    const bool up = (lane & (32 >> k)) != 0;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double send = up ? a[i] : a[i + n], keep = up ? a[i + n] : a[i];
      a[i] = keep + __shfl_xor(send, 32 >> k, 64);
    }
  }
  double s = a[0];  // value lane >> (6 - LG), summed over the steps so far
#pragma unroll
  for (int o = 32 >> LG; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  const int v = lane >> (6 - LG);
  if ((lane & ((64 >> LG) - 1)) == 0 && v < NV) sh[wid * NV + v] = s;
  __syncthreads();
  const int nw = blockDim.x >> 6;
  if (threadIdx.x < NV) {
    double t = 0.0;
    for (int w = 0; w < nw; ++w) t += sh[w * NV + threadIdx.x];
    part[(size_t)threadIdx.x * kMaxRedBlocks + blockIdx.x] = t;
  }
}

// In a finishing kernel: the calling wavefront adds partials[v][0..nb) in a
// fixed order (lane-strided, then a butterfly) and returns the total in every lane.
__device__ __forceinline__ double wave_total(const RedWork& rw, int v, int nb) {
  const int lane = threadIdx.x & 63;
  const double* p = rw.partial + (size_t)v * kMaxRedBlocks;
  // all loads first (independent addresses), then the fixed-order sum
  double x[kMaxRedBlocks / 64];
#pragma unroll
  for (int q = 0; q < kMaxRedBlocks / 64; ++q) {
    const int k = lane + 64 * q;
    x[q] = k < nb ? p[k] : 0.0;
  }
  double s = 0.0;
#pragma unroll
  for (int q = 0; q < kMaxRedBlocks / 64; ++q) s += x[q];
  return wave_sum(s);
}

constexpr int kFinishThreads = 1024;  // 16 wavefronts: one value per wavefront

}  // namespace rsfde
