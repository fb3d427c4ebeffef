// Updates of the Arnoldi step: V_{j+1} = w - sum_i h_i v_i (stored
// unnormalised) in one pass over the basis, with what the step needs next in
// the same pass: the dots <V_i, V_{j+1}> of the second Gram-Schmidt pass
// (k_axpy_dot), or ||V_{j+1}||^2 (k_axpy_givens, FINAL).  The Givens kernel then
// sets vscale[j+1] = 1/beta (beta = ||V_{j+1}||), applies the previous Givens
// rotations to column j, forms rotation j from its last entry and beta (Section 5:
// GMRES), stores the rotated column with 0 below the diagonal and publishes the
// residual estimate |g_{j+1}| for the host.
//
// All are bound by reading the basis; on short vectors, by the launches and
// the latency of one load round each (krylov_orth.hpp).
#include "krylov_orth.hpp"

namespace rsfde {

// GATHER: the coefficients are summed here from the dots' partials (short
// vectors) and stored to hout by block 0; otherwise they are read from coef.
template <int NV, int W, bool GATHER>
__device__ __forceinline__ void coefs(double* c, const RedWork& rw, int nb, bool second,
                                      const double* coef, const double* vscale, double* hout) {
  if constexpr (GATHER) {
    gather_coefs<NV>(orth_partials(rw, second), nb, vscale, hout, c);
  } else {
    if (threadIdx.x < NV) c[threadIdx.x] = coef[threadIdx.x] * vscale[threadIdx.x];
    __syncthreads();
  }
}

// W = 2: scheduled for the two wavefronts per SIMD that its grid gives, as
// k_multidot is.  Left to itself the compiler's batches of loads suit some counts
// and not others (2047^2: 21, 22, 25, 26, 29 and 30 vectors 195 to 273 us, now 148
// to 202; the counts between lose 2 to 3 %: 20 136 -> 140, 28 186 -> 191).
template <int NV, int W, bool FINAL, bool GATHER>
__global__ __launch_bounds__(kRedThreads)
__attribute__((amdgpu_waves_per_eu(W == 2 ? 2 : 1, W == 2 ? 2 : 8)))
void k_axpy_givens(const double* __restrict__ V, size_t ldv, const double* win, double* vout,
                   size_t N, RedWork rw, double* coef, const double* vscale, bool second,
                   const Members mb) {
  __shared__ double sh[16], c[NV];
  {  // member of a batched launch (grid dimension y)
    const size_t mo = mb.off(blockIdx.y);
    V += mo;
    win += mo;
    vout += mo;
    rw.partial += mo;
    coef += mo;
    vscale += mo;
  }
  const size_t n = N / W, stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  Vals<W> u, x[NV];
  auto load = [&] {
    u.load(win, i);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v].load(V + (size_t)v * ldv, i);
  };
  if constexpr (GATHER)
    if (i < n) load();  // in flight while the coefficients are summed
  coefs<NV, W, GATHER>(c, rw, gridDim.x, second, coef, vscale, coef);
  double acc[1] = {0.0};
  while (i < n) {
    if constexpr (!GATHER) load();
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int k = 0; k < W; ++k) u.v[k] -= c[v] * x[v].v[k];
    u.store(vout, i);
    if (FINAL)
#pragma unroll
      for (int k = 0; k < W; ++k) acc[0] += u.v[k] * u.v[k];
    i += stride;
    if constexpr (GATHER)
      if (i < n) load();
  }
  if (W == 2 && (N & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
    double t = win[N - 1];
#pragma unroll
    for (int v = 0; v < NV; ++v) t -= c[v] * V[(size_t)v * ldv + N - 1];
    vout[N - 1] = t;
    if (FINAL) acc[0] += t * t;
  }
  // (row 0 of the partials: the first pass's, read by no block of this launch
  // unless it is itself the first pass; then each block's own norm partial goes
  // to the second pass's rows)
  if constexpr (FINAL) publish_partials<1>(acc, orth_partials(rw, !second), sh);
}

// vout = w - sum_i c_i V_i and the partials of <V_i, vout>, i < NV: the first
// pass's update and the second pass's dots read the basis once.
template <int NV, int W, bool GATHER>
__global__ __launch_bounds__(kRedThreads) void k_axpy_dot(const double* __restrict__ V, size_t ldv,
                                                          const double* __restrict__ w,
                                                          double* __restrict__ vout, size_t N,
                                                          RedWork rw, double* coef,
                                                          const double* vscale, const Members mb) {
  __shared__ double sh[16 * NV], c[NV];
  {  // member of a batched launch (grid dimension y)
    const size_t mo = mb.off(blockIdx.y);
    V += mo;
    w += mo;
    vout += mo;
    rw.partial += mo;
    coef += mo;
    vscale += mo;
  }
  const size_t n = N / W, stride = (size_t)gridDim.x * blockDim.x;
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  Vals<W> u, x[NV];
  auto load = [&] {
    u.load(w, i);
#pragma unroll
    for (int v = 0; v < NV; ++v) x[v].load(V + (size_t)v * ldv, i);
  };
  if constexpr (GATHER)
    if (i < n) load();
  coefs<NV, W, GATHER>(c, rw, gridDim.x, false, coef, vscale, coef);
  double acc[NV];
#pragma unroll
  for (int v = 0; v < NV; ++v) acc[v] = 0.0;
  while (i < n) {
    if constexpr (!GATHER) load();
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int k = 0; k < W; ++k) u.v[k] -= c[v] * x[v].v[k];
    u.store(vout, i);
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
      for (int k = 0; k < W; ++k) acc[v] += x[v].v[k] * u.v[k];
    i += stride;
    if constexpr (GATHER)
      if (i < n) load();
  }
  if (W == 2 && (N & 1) && blockIdx.x == 0 && threadIdx.x == 0) {
    double t = w[N - 1];
#pragma unroll
    for (int v = 0; v < NV; ++v) t -= c[v] * V[(size_t)v * ldv + N - 1];
    vout[N - 1] = t;
#pragma unroll
    for (int v = 0; v < NV; ++v) acc[v] += V[(size_t)v * ldv + N - 1] * t;
  }
  publish_partials<NV>(acc, orth_partials(rw, true), sh);
}

// beta = ||V_{j+1}||, vscale[j+1] = 1/beta, the previous Givens rotations applied
// to column j, rotation j of (H[j][j], beta) to (den, 0), and |g_{j+1}| for the host.
// One wavefront: the column and the rotations are loaded at once (one lane per
// entry) and the recurrence runs from LDS; reading them one dependent global
// load after the other took 6.2 us at j = 20.
__global__ __launch_bounds__(64) void k_givens(RedWork rw, int nb, KrylovState* ks, int j,
                                               int add_h2, bool second, HostStatus* hs,
                                               const Members mb) {
  __shared__ double h[kMaxRestart + 1], cs[kMaxRestart], sn[kMaxRestart];
  rw.partial += mb.off(blockIdx.y);
  ks = (KrylovState*)((double*)ks + mb.off(blockIdx.y));
  hs += mb.m[blockIdx.y];
  double* Hj = ks->H + (size_t)j * kLdH;
  const int lane = threadIdx.x;  // j < kMaxRestart = 64: one lane per entry 0..j
  const double gj = ks->g[j];
  if (lane <= j) {
    h[lane] = Hj[lane] + (add_h2 ? ks->h2[lane] : 0.0);
    if (lane < j) {
      cs[lane] = ks->cs[lane];
      sn[lane] = ks->sn[lane];
    }
  }
  const double uu = wave_total(RedWork{orth_partials(rw, !second)}, 0, nb);
  __syncthreads();
  if (lane == 0) {
    const double beta = sqrt(uu);
    ks->vscale[j + 1] = beta > 0.0 ? 1.0 / beta : 0.0;
    double a = h[0];
#pragma unroll 4
    for (int i = 0; i < j; ++i) {
      const double bb = h[i + 1];
      h[i] = cs[i] * a + sn[i] * bb;
      a = -sn[i] * a + cs[i] * bb;
    }
    const double den = hypot(a, beta);
    const double c = den > 0.0 ? a / den : 1.0;
    const double s = den > 0.0 ? beta / den : 0.0;
    ks->cs[j] = c;
    ks->sn[j] = s;
    h[j] = den;
    Hj[j + 1] = 0.0;
    ks->g[j] = c * gj;
    const double gn = -s * gj;
    ks->g[j + 1] = gn;
    hs->est[j] = fabs(gn);
    if (!isfinite(beta) || !isfinite(den) || !isfinite(gj)) hs->flags |= kFlagNonFinite;
    __threadfence_system();
  }
  __syncthreads();
  if (lane <= j) Hj[lane] = h[lane];
}

using AxpyFn = void (*)(const double*, size_t, const double*, double*, size_t, RedWork, double*,
                        const double*, bool, const Members&, dim3, hipStream_t);

template <int NV, int W, bool FINAL, bool GATHER>
static void run_axpy(const double* V, size_t ldv, const double* win, double* vout, size_t N,
                     RedWork rw, double* coef, const double* vscale, bool second, const Members& mb,
                     dim3 g, hipStream_t s) {
  hipLaunchKernelGGL((k_axpy_givens<NV, W, FINAL, GATHER>), g, dim3(kRedThreads), 0, s, V, ldv, win,
                     vout, N, rw, coef, vscale, second, mb);
}
template <int NV, int W, bool GATHER>
static void run_axpy_dot(const double* V, size_t ldv, const double* win, double* vout, size_t N,
                         RedWork rw, double* coef, const double* vscale, bool, const Members& mb,
                         dim3 g, hipStream_t s) {
  hipLaunchKernelGGL((k_axpy_dot<NV, W, GATHER>), g, dim3(kRedThreads), 0, s, V, ldv, win, vout, N,
                     rw, coef, vscale, mb);
}
template <int W, bool FINAL, bool GATHER, int... I>
static constexpr std::array<AxpyFn, sizeof...(I)> axpy_table(std::integer_sequence<int, I...>) {
  return {&run_axpy<I + 1, W, FINAL, GATHER>...};
}
template <int W, bool GATHER, int... I>
static constexpr std::array<AxpyFn, sizeof...(I)> axpy_dot_table(std::integer_sequence<int, I...>) {
  return {&run_axpy_dot<I + 1, W, GATHER>...};
}
using Counts = std::make_integer_sequence<int, kChunk>;
// short vectors: one chunk, coefficients summed by the consumer
static const auto kFinalSmall = axpy_table<1, true, true>(Counts{});
static const auto kDotSmall = axpy_dot_table<1, true>(Counts{});
// long vectors, and chunks of more than kChunk basis vectors
static const auto kFinal = axpy_table<2, true, false>(Counts{});
static const auto kPart = axpy_table<2, false, false>(Counts{});
static const auto kDot = axpy_dot_table<2, false>(Counts{});

// One chunk of a short vector's basis: its consumers gather the partials.
static bool gathers(int nv, size_t N) { return nv <= kChunk && orth_small(N); }

hipError_t launch_orth_dots(const double* V, size_t ldv, int nv, const double* w, size_t N,
                            RedWork rw, KrylovState* ks, int j, hipStream_t s, const Members& mb) {
  return launch_multidot(V, ldv, nv, w, N, rw, ks, j, false, !gathers(nv, N), s, mb);
}

hipError_t launch_orth_update(const double* V, size_t ldv, int nv, const double* w, double* vout,
                              size_t N, RedWork rw, KrylovState* ks, int j, bool reorth,
                              HostStatus* hs, hipStream_t s, const Members& mb) {
  if (nv < 1 || nv > kMaxRestart || j < 0 || j >= kMaxRestart) return hipErrorInvalidValue;
  if (mb.n < 1 || mb.n > kMaxBatch) return hipErrorInvalidValue;
  double* const Hj = ks->H + (size_t)j * kLdH;
  const bool one = nv <= kChunk, small = gathers(nv, N);
  const int nb = orth_blocks(N);
  const dim3 g(nb, mb.n);
  hipError_t e;
  const double* win = w;
  if (reorth && one) {  // the first pass's update with the second pass's dots
    (small ? kDotSmall : kDot)[nv - 1](V, ldv, w, vout, N, rw, Hj, ks->vscale, false, mb, g, s);
    if (!small && (e = launch_multidot_finish(nb, nv, rw, ks, ks->h2, 0, true, s, mb)) != hipSuccess)
      return e;
    win = vout;
  } else if (reorth) {  // more than kChunk vectors: every chunk's update before any dot
    for (int v0 = 0; v0 < nv; v0 += kChunk) {
      const int n = nv - v0 < kChunk ? nv - v0 : kChunk;
      kPart[n - 1](V + (size_t)v0 * ldv, ldv, win, vout, N, rw, Hj + v0, ks->vscale + v0, false, mb,
                   g, s);
      win = vout;
    }
    if ((e = launch_multidot(V, ldv, nv, vout, N, rw, ks, j, true, true, s, mb)) != hipSuccess)
      return e;
  }
  double* const coef = reorth ? ks->h2 : Hj;
  for (int v0 = 0; v0 < nv; v0 += kChunk) {
    const int n = nv - v0 < kChunk ? nv - v0 : kChunk;
    const bool last = v0 + n == nv;
    (small ? kFinalSmall : last ? kFinal : kPart)[n - 1](V + (size_t)v0 * ldv, ldv, win, vout, N, rw,
                                                         coef + v0, ks->vscale + v0, reorth, mb, g,
                                                         s);
    win = vout;
  }
  hipLaunchKernelGGL(k_givens, dim3(1, mb.n), dim3(64), 0, s, rw, nb, ks, j, reorth ? 1 : 0, reorth,
                     hs, mb);
  return hipGetLastError();
}

}  // namespace rsfde
