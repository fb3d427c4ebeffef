// Fused multi-dot of the Arnoldi step (classical Gram-Schmidt projections):
// h_i = vscale[i] * <V_i, w> for i < nv in one pass over the basis.  The vector
// count is a template parameter, so every basis load is unconditional and the
// loop unrolls: all NV + 1 streams are in flight at once.  nv > kChunk runs in
// chunks.  Short vectors leave their partials to the next kernel (krylov_orth.hpp);
// long ones and chunks are finished into column j of the Hessenberg matrix.
#include "krylov_orth.hpp"

namespace rsfde {

// Long vectors (W = 2) run 512 blocks, two wavefronts per SIMD, and are bound by
// reading the basis: scheduled for that occupancy, all NV + 1 streams' loads are
// in flight; scheduled for more wavefronts they go out in batches (2047^2: 24
// vectors 213 -> 158 us, 32 vectors 283 -> 206 us, 5.4 TB/s; up to 16 the same).
template <int NV, int W>
__global__ __launch_bounds__(kRedThreads)
__attribute__((amdgpu_waves_per_eu(W == 2 ? 2 : 1, W == 2 ? 2 : 8)))
void k_multidot(const double* __restrict__ V, size_t ldv, const double* __restrict__ w, size_t N,
                RedWork rw, bool second, const Members mb) {
  __shared__ double sh[16 * NV];
  {  // member of a batched launch (grid dimension y)
    const size_t mo = mb.off(blockIdx.y);
    V += mo;
    w += mo;
    rw.partial += mo;
  }
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N / W;
       i += (size_t)gridDim.x * blockDim.x) {
    Vals<W> wv, x[NV];
    wv.load(w, i);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v].load(V + (size_t)v * ldv, i);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int k = 0; k < W; ++k) acc[v] += x[v].v[k] * wv.v[k];
  }
  if (W == 2 && (N & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
    const double wl = w[N - 1];
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += V[(size_t)v * ldv + N - 1] * wl;
  }
  publish_partials<NV>(acc, orth_partials(rw, second), sh);
}

// dst[v0 + v] = vscale[v0 + v] * (sum of the partials of value v), v < nv;
// dst is column j of H or the reorthogonalisation vector h2.
__global__ __launch_bounds__(kFinishThreads) void k_multidot_finish(RedWork rw, int nb, int nv,
                                                                    KrylovState* ks, double* dst,
                                                                    int v0, bool second,
                                                                    const Members mb) {
  {
    const size_t mo = mb.off(blockIdx.y);
    rw.partial += mo;
    ks = (KrylovState*)((double*)ks + mo);
    dst += mo;
  }
  const int lane = threadIdx.x & 63;
  const RedWork part{orth_partials(rw, second)};
  for (int v = threadIdx.x >> 6; v < nv; v += kFinishThreads / 64) {
    const double t = wave_total(part, v, nb);
    if (lane == 0) dst[v0 + v] = ks->vscale[v0 + v] * t;
  }
}

using MultidotFn = void (*)(const double*, size_t, const double*, size_t, RedWork, bool,
                            const Members&, dim3, hipStream_t);

template <int NV, int W>
static void run_multidot(const double* V, size_t ldv, const double* w, size_t N, RedWork rw,
                         bool second, const Members& mb, dim3 g, hipStream_t s) {
  hipLaunchKernelGGL((k_multidot<NV, W>), g, dim3(kRedThreads), 0, s, V, ldv, w, N, rw, second, mb);
}
template <int W, int... I>
static constexpr std::array<MultidotFn, sizeof...(I)> multidot_table(std::integer_sequence<int, I...>) {
  return {&run_multidot<I + 1, W>...};
}
static const auto kMultidot1 = multidot_table<1>(std::make_integer_sequence<int, kChunk>{});
static const auto kMultidot2 = multidot_table<2>(std::make_integer_sequence<int, kChunk>{});

hipError_t launch_multidot(const double* V, size_t ldv, int nv, const double* w, size_t N,
                           RedWork rw, KrylovState* ks, int j, bool second, bool finish,
                           hipStream_t s, const Members& mb) {
  if (nv < 1 || nv > kMaxRestart || (!finish && nv > kChunk)) return hipErrorInvalidValue;
  if (mb.n < 1 || mb.n > kMaxBatch) return hipErrorInvalidValue;
  double* dst = second ? ks->h2 : ks->H + (size_t)j * kLdH;
  const int nb = orth_blocks(N);
  for (int v0 = 0; v0 < nv; v0 += kChunk) {
    const int n = nv - v0 < kChunk ? nv - v0 : kChunk;
    (orth_small(N) ? kMultidot1 : kMultidot2)[n - 1](V + (size_t)v0 * ldv, ldv, w, N, rw, second,
                                                     mb, dim3(nb, mb.n), s);
    if (finish)
      if (hipError_t e = launch_multidot_finish(nb, n, rw, ks, dst, v0, second, s, mb)) return e;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_multidot_finish(int nb, int nv, RedWork rw, KrylovState* ks, double* dst, int v0,
                                  bool second, hipStream_t s, const Members& mb) {
  hipLaunchKernelGGL(k_multidot_finish, dim3(1, mb.n), dim3(kFinishThreads), 0, s, rw, nb, nv, ks,
                     dst, v0, second, mb);
  return hipGetLastError();
}

}  // namespace rsfde
