// The sine-transform preconditioner of Section 4.1 for grids whose n + 1 is not
// a power of two.  P_hat^{-1} is the same operator as in pc_kernels.hpp:
//   z = mask * S_y (W / E1) S_x + (1 - mask) * S_y (W / E2) S_x,  W = S_y V S_x,
// E1 = 1 - kx lx_i - ky ly_j, E2 = E1 + dt/eta, S the orthonormal DST-I
// sqrt(2/(n+1)) sin(pi j k / (n+1)) (Section 4.1).  Only the way a length-n
// DST-I is computed differs.
//
// Chirp form of the DST-I (Bluestein's identity jk = (j^2 + k^2 - (k-j)^2)/2):
//   sum_j x_j sin(pi j k / M) = Im( c_k sum_j (c_j x_j) conj(c_{k-j}) ),
//   c_j = exp(i pi j^2 / (2M)),  M = n + 1,
// i.e. a chirp premultiply, a Toeplitz convolution with the even kernel
// exp(-i pi m^2 / (2M)), |m| < n, and a chirp postmultiply.  The convolution
// is circular of power-of-two length L >= 2n - 1 (no wrap-around reaches
// outputs 0..n-1), done with the register-resident FFT of fft_engine.hpp; the
// kernel's spectrum `khat` (times sqrt(2/M) / L) is a set-up table in
// register-position order, so the pointwise product needs no reordering.
// Every line is one complex FFT pair (real lines cannot share one: the chirp
// mixes real and imaginary parts), about four times the work of the
// odd-extension form, which the library uses whenever n + 1 is a power of two.
//
// Passes (T = double or float internals; v and z are FP64):
//   rows:    W1 = rows of (sig * v) transformed along x
//   columns: W  = W1 transformed along y; Y1 = S_y(W / E1), Y2 = S_y(W / E2)
//   rows:    z  = S_x of Y1 rows where mask = 1, of Y2 rows where mask = 0
// Layouts: [rows][n1] arrays (TL = false); where one direction of a
// two-dimensional grid takes the symmetric form (cd_sd.hpp), both use its layouts
// (TL = true): W1, Y1 and Y2 strip-tiled.
#pragma once
#include "cd_sd.hpp"

namespace rsfde {

template <int L>
struct CdCfg {
  using F = Fft<L, fft_pts(L)>;
  static constexpr int TPF = F::TPF;
  static constexpr bool CX = fft_cx(L);
  static constexpr int LEN = lds_len(L, CX);  // LDS scalars of one transform
  static constexpr int BR = row_ffts(TPF);  // lines per row block
  static constexpr int BCL = (256 / TPF) > 16 ? 16 : ((256 / TPF) > 0 ? (256 / TPF) : 1);
  static constexpr int BCS = L <= 512 && col_ffts_small(TPF) < BCL ? col_ffts_small(TPF) : BCL;
  static constexpr int THR_R = BR * TPF;
  // The column pass's three transforms written out instead of in a loop: where the
  // loop's reloads of the tables cost more than the shorter code gives.  Whole
  // preconditioner, loop / written out: FP64 1000^2 90.4 / 89.0 us, 2000 x 700 129.8
  // / 128.0 (L = 2048), 64 x 2049 61.1 / 59.9 (L = 8192); FP32 1400^2 128.5 / 125.2,
  // 2000^2 183.4 / 176.6 (L = 4096).  Elsewhere the loop: FP64 600 x 1800 132.9 /
  // 135.7 (L = 4096), FP32 2000 x 700 80.7 / 85.3 (L = 2048), 20 x 20 x 2100 122 /
  // 138 (L = 8192), and every tiled form (FP32 4000 x 1500 295 / 306).
  template <typename T, bool TL>
  static constexpr bool unrolled() {
    return !TL && (sizeof(T) == 8 ? L == 2048 || L == 8192 : L == 4096);
  }
  // A view that the large column blocks cannot spread over the CUs.
  static bool small_cols(long cols, long copies) {
    return BCS < BCL && (cols + BCL - 1) / BCL * copies < kSmallGridBlocks;
  }
};

// In: reg[e].re = x at sequence position pos(0, tau, e) (zero at positions >= n).
// Out: reg[e].re = (S x) at the same position (unspecified at positions >= n).
template <typename T, class F, bool CX, int ST = 1>
__device__ __forceinline__ void chirp_dst(cpx<T>* reg, int tau, const cpx<T>* __restrict__ chn,
                                          const cpx<T>* __restrict__ khat,
                                          const cpx<T>* __restrict__ tw, T* lds, int n) {
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    const cpx<T> c = p < n ? chn[p] : cpx<T>{T(0), T(0)};
    const T x = reg[e].re;
    reg[e].re = x * c.re;
    reg[e].im = x * c.im;
  });
  fft_forward<T, F, true, ST, CX>(reg, tau, tw, lds);
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    reg[e] = cmul(reg[e], khat[F::pos(F::NS - 1, tau, e)]);
  });
  fft_inverse<T, F, true, ST, CX>(reg, tau, tw, lds);
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    const cpx<T> c = p < n ? chn[p] : cpx<T>{T(0), T(0)};
    reg[e].re = c.re * reg[e].im + c.im * reg[e].re;  // Im(c * y)
  });
}

// Rows: W1[r] = S_x (sig * v[r]).
template <typename T, int L, bool TL>
__global__ __launch_bounds__(CdCfg<L>::THR_R) void k_cd_rows_fwd(
    const double* __restrict__ v, const double* __restrict__ sig, T* __restrict__ out,
    const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ tw, int n1, int n2) {
  using C = CdCfg<L>;
  using F = typename C::F;
  __shared__ T lds[C::BR * C::LEN];
  const int b = threadIdx.x / F::TPF, tau = threadIdx.x % F::TPF;
  const int r = blockIdx.x * C::BR + b;
  const bool vr = r < n2;
  const double sc = sig ? *sig : 1.0;
  cpx<T> reg[F::PP];
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    reg[e].re = (vr && p < n1) ? (T)(sc * v[(size_t)r * n1 + p]) : T(0);
    reg[e].im = T(0);
  });
  chirp_dst<T, F, C::CX>(reg, tau, chn, khat, tw, lds + b * C::LEN, n1);
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    if (vr && p < n1) out[TL ? tile_index(r, p, (n2 + 1) >> 1) : (size_t)r * n1 + p] = reg[e].re;
  });
}

// Columns: W = S_y W1 column, then Y1 = S_y(W / E1) and Y2 = S_y(W / E2).
// Thread layout (tau, b) with b fastest: a wavefront touches BC adjacent
// columns of each row it reads.
template <typename T, int L, int BC, bool TL>
__global__ __launch_bounds__(CdCfg<L>::TPF* BC) void k_cd_cols(
    const T* __restrict__ in, T* __restrict__ Y1, T* __restrict__ Y2,
    const double* __restrict__ lamx, const double* __restrict__ lamy,
    const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ tw, int n1, int n2, double kx, double ky, double dpen) {
  using C = CdCfg<L>;
  using F = typename C::F;
  __shared__ T lds[BC * C::LEN];
  const int b = threadIdx.x % BC, tau = threadIdx.x / BC;
  const int c = xcd_remap(blockIdx.x, gridDim.x) * BC + b;
  const bool vc = c < n1;
  T* my = lds + b * (C::CX ? 2 : 1);  // regions interleaved (stride BC)
  const int hp = (n2 + 1) >> 1;
  cpx<T> reg[F::PP];
  T w[F::PP];
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    reg[e].re = (vc && p < n2) ? in[TL ? tile_index(p, c, hp) : (size_t)p * n1 + c] : T(0);
    reg[e].im = T(0);
  });
  if constexpr (C::template unrolled<T, TL>()) {
    // (the denominators are formed before w: the other order held 256 VGPRs and
    // more at L = 2048 in FP64 where this one takes 218)
    chirp_dst<T, F, C::CX, BC>(reg, tau, chn, khat, tw, my, n2);
    const double ax = 1.0 - kx * (vc ? lamx[c] : 0.0);
    static_for<F::PP>([&](auto ee) {
      constexpr int e = decltype(ee)::value;
      const int p = F::pos(0, tau, e);
      const T e1 = (T)(ax - ky * (p < n2 ? lamy[p] : 0.0));
      w[e] = p < n2 ? reg[e].re : T(0);
      reg[e].re = w[e] / e1;
    });
    chirp_dst<T, F, C::CX, BC>(reg, tau, chn, khat, tw, my, n2);
    static_for<F::PP>([&](auto ee) {
      constexpr int e = decltype(ee)::value;
      const int p = F::pos(0, tau, e);
      if (vc && p < n2) Y1[TL ? tile_index(p, c, hp) : (size_t)p * n1 + c] = reg[e].re;
      const T e2 = (T)(ax + dpen - ky * (p < n2 ? lamy[p] : 0.0));
      reg[e].re = w[e] / e2;
    });
    chirp_dst<T, F, C::CX, BC>(reg, tau, chn, khat, tw, my, n2);
    static_for<F::PP>([&](auto ee) {
      constexpr int e = decltype(ee)::value;
      const int p = F::pos(0, tau, e);
      if (vc && p < n2) Y2[TL ? tile_index(p, c, hp) : (size_t)p * n1 + c] = reg[e].re;
    });
    return;
  }
  const double ax = 1.0 - kx * (vc ? lamx[c] : 0.0);
  // The three transforms by one copy of the code (half the instructions to
  // fetch; 256^2 13.9 -> 13.4 us): the forward one, then w / E1 and w / E2.
#pragma unroll 1
  for (int q = 0; q < 3; ++q) {
    // opaque thread index and tables: nothing per point is hoisted out of the loop
    int th = tau;
    asm volatile("" : "+v"(th));
    const int zo = opaque_zero();
    const double* ly = lamy + zo;
    chirp_dst<T, F, C::CX, BC>(reg, th, chn + zo, khat + zo, tw + zo, my, n2);
    static_for<F::PP>([&](auto ee) {
      constexpr int e = decltype(ee)::value;
      const int p = F::pos(0, th, e);
      const bool in_range = p < n2;
      if (q == 0) {
        w[e] = in_range ? reg[e].re : T(0);
      } else if (vc && in_range) {
        (q == 1 ? Y1 : Y2)[TL ? tile_index(p, c, hp) : (size_t)p * n1 + c] = reg[e].re;
      }
      reg[e].re = w[e] / (T)(ax + (q == 0 ? 0.0 : dpen) - ky * (in_range ? ly[p] : 0.0));
    });
  }
}

// Rows: line u = 2r + k transforms row r of Y1 (k = 0) or Y2 (k = 1) along x
// and writes z where the mask selects that branch; the two lines of a row
// write disjoint points, so no combine step is needed.
template <typename T, int L, bool TL>
__global__ __launch_bounds__(CdCfg<L>::THR_R) void k_cd_rows_inv(
    const T* __restrict__ Y1, const T* __restrict__ Y2, const uint8_t* __restrict__ mask,
    double* __restrict__ z, const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ tw, int n1, int n2) {
  using C = CdCfg<L>;
  using F = typename C::F;
  __shared__ T lds[C::BR * C::LEN];
  const int b = threadIdx.x / F::TPF, tau = threadIdx.x % F::TPF;
  const int u = blockIdx.x * C::BR + b;
  const int r = u >> 1, k = u & 1;
  const bool vr = r < n2;
  const T* src = k ? Y2 : Y1;
  cpx<T> reg[F::PP];
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    reg[e].re = (vr && p < n1) ? src[TL ? tile_index(r, p, (n2 + 1) >> 1) : (size_t)r * n1 + p] : T(0);
    reg[e].im = T(0);
  });
  chirp_dst<T, F, C::CX>(reg, tau, chn, khat, tw, lds + b * C::LEN, n1);
  const uint8_t want = k ? 0 : 1;
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    if (vr && p < n1) {
      const size_t i = (size_t)r * n1 + p;
      if ((mask[i] != 0) == (want != 0)) z[i] = (double)reg[e].re;
    }
  });
}

// Columns without scaling (the three-dimensional plans' y transforms): out =
// S_y in for the columns c < ncol of `batch` slices [rows][ncol], slice b at
// offset b * bstride; with inB given, grid dimension z = 1 transforms inB into
// outB in the same launch.  in and out must not overlap.
template <typename T, int L, int BC>
__global__ __launch_bounds__(CdCfg<L>::TPF* BC) void k_cd_dst_cols(
    const T* __restrict__ inA, T* __restrict__ outA, const T* __restrict__ inB,
    T* __restrict__ outB, const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ tw, int ncol, int rows, size_t bstride) {
  using C = CdCfg<L>;
  using F = typename C::F;
  __shared__ T lds[BC * C::LEN];
  const size_t off = (size_t)blockIdx.y * bstride;
  const T* in = (blockIdx.z ? inB : inA) + off;
  T* out = (blockIdx.z ? outB : outA) + off;
  const int b = threadIdx.x % BC, tau = threadIdx.x / BC;
  const int c = xcd_remap(blockIdx.x, gridDim.x) * BC + b;
  const bool vc = c < ncol;
  T* my = lds + b * (C::CX ? 2 : 1);  // regions interleaved (stride BC)
  cpx<T> reg[F::PP];
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    reg[e].re = (vc && p < rows) ? in[(size_t)p * ncol + c] : T(0);
    reg[e].im = T(0);
  });
  chirp_dst<T, F, C::CX, BC>(reg, tau, chn, khat, tw, my, rows);
  static_for<F::PP>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    const int p = F::pos(0, tau, e);
    if (vc && p < rows) out[(size_t)p * ncol + c] = reg[e].re;
  });
}

#define RSFDE_CD_CASES(X) \
  X(2) X(4) X(8) X(16) X(32) X(64) X(128) X(256) X(512) X(1024) X(2048) X(4096) X(8192)

// The symmetric form's lengths (cd_sd.hpp).
#define RSFDE_CDS_CASES(X) X(16384)

template <typename T>
hipError_t launch_cd_rows_fwd(const CdDir& d, const double* v, const double* sig, T* out, int n1,
                              int n2, bool tiled, hipStream_t s) {
  const cpx<T>*chn = (const cpx<T>*)d.chn, *khat = (const cpx<T>*)d.khat, *tw = (const cpx<T>*)d.tw;
  if (d.twS) {
    if (!tiled || 4 * n1 > d.L) return hipErrorInvalidValue;
    switch (d.L) {
#define X(LL)                                                                                   \
  case LL: {                                                                                    \
    using C = CdSd<LL>;                                                                         \
    hipLaunchKernelGGL((k_cds_rows_fwd<T, LL>), dim3((n2 + 1) / 2), dim3(C::THR), 0, s, v,       \
                       sig, out, chn, khat, tw, (const cpx<T>*)d.twS, n1, n2);         \
    return hipGetLastError();                                                                   \
  }
      RSFDE_CDS_CASES(X)
#undef X
      default:
        return hipErrorInvalidValue;
    }
  }
  switch (d.L) {
#define X(LL)                                                                                 \
  case LL: {                                                                                  \
    using C = CdCfg<LL>;                                                                      \
    const dim3 g((n2 + C::BR - 1) / C::BR), t(C::THR_R);                                      \
    if (tiled)                                                                                \
      hipLaunchKernelGGL((k_cd_rows_fwd<T, LL, true>), g, t, 0, s, v, sig, out, chn, khat, tw, n1, \
                         n2);                                                                 \
    else                                                                                      \
      hipLaunchKernelGGL((k_cd_rows_fwd<T, LL, false>), g, t, 0, s, v, sig, out, chn, khat, tw, n1, \
                         n2);                                                                 \
    return hipGetLastError();                                                                 \
  }
    RSFDE_CD_CASES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_cd_cols(const CdDir& d, const T* in, T* Y1, T* Y2, const double* lamx,
                          const double* lamy, int n1, int n2, double kx, double ky, double dpen,
                          bool tiled, hipStream_t s) {
  const cpx<T>*chn = (const cpx<T>*)d.chn, *khat = (const cpx<T>*)d.khat, *tw = (const cpx<T>*)d.tw;
  if (d.twS) {
    if (!tiled || 4 * n2 > d.L) return hipErrorInvalidValue;
    switch (d.L) {
#define X(LL)                                                                                    \
  case LL: {                                                                                     \
    using C = CdSd<LL>;                                                                          \
    hipLaunchKernelGGL((k_cds_cols<T, LL>), dim3((n1 + 1) / 2), dim3(C::THR), 0, s, in, Y1, Y2, \
                       lamx, lamy, chn, khat, tw, (const cpx<T>*)d.twS, n1, n2, kx, ky, dpen);         \
    return hipGetLastError();                                                                    \
  }
      RSFDE_CDS_CASES(X)
#undef X
      default:
        return hipErrorInvalidValue;
    }
  }
  switch (d.L) {
#define X(LL)                                                                                  \
  case LL: {                                                                                   \
    using C = CdCfg<LL>;                                                                       \
    auto go = [&](auto bc, auto tl) {                                                          \
      constexpr int BC = decltype(bc)::value;                                                  \
      constexpr bool TL = decltype(tl)::value;                                                 \
      hipLaunchKernelGGL((k_cd_cols<T, LL, BC, TL>), dim3((n1 + BC - 1) / BC), dim3(BC * C::TPF), 0, \
                         s, in, Y1, Y2, lamx, lamy, chn, khat, tw, n1, n2, kx, ky, dpen);      \
    };                                                                                         \
    using S = std::integral_constant<int, C::BCS>;                                             \
    using B = std::integral_constant<int, C::BCL>;                                             \
    if (C::small_cols(n1, 1)) tiled ? go(S{}, std::true_type{}) : go(S{}, std::false_type{});  \
    else tiled ? go(B{}, std::true_type{}) : go(B{}, std::false_type{});                       \
    return hipGetLastError();                                                                  \
  }
    RSFDE_CD_CASES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_cd_dst_cols(int L, const T* inA, T* outA, const T* inB, T* outB, const void* chn,
                              const void* khat, const void* tw, int ncol, int rows, int batch,
                              size_t bstride, hipStream_t s) {
  if (batch < 1 || batch > 65535 || ncol < 1 || rows < 1 || !inA || !outA || (!inB) != (!outB))
    return hipErrorInvalidValue;
  switch (L) {
#define X(LL)                                                                                  \
  case LL: {                                                                                   \
    using C = CdCfg<LL>;                                                                       \
    const int nz = inB ? 2 : 1;                                                                \
    auto go = [&](auto bc) {                                                                   \
      constexpr int BC = decltype(bc)::value;                                                  \
      hipLaunchKernelGGL((k_cd_dst_cols<T, LL, BC>), dim3((ncol + BC - 1) / BC, batch, nz),    \
                         dim3(BC * C::TPF), 0, s, inA, outA, inB, outB, (const cpx<T>*)chn,    \
                         (const cpx<T>*)khat, (const cpx<T>*)tw, ncol, rows, bstride);         \
    };                                                                                         \
    if (C::small_cols(ncol, (long)batch * nz)) go(std::integral_constant<int, C::BCS>{});      \
    else go(std::integral_constant<int, C::BCL>{});                                            \
    return hipGetLastError();                                                                  \
  }
    RSFDE_CD_CASES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_cd_rows_inv(const CdDir& d, const T* Y1, const T* Y2, const uint8_t* mask,
                              double* z, int n1, int n2, bool tiled, hipStream_t s) {
  const cpx<T>*chn = (const cpx<T>*)d.chn, *khat = (const cpx<T>*)d.khat, *tw = (const cpx<T>*)d.tw;
  if (d.twS) {
    if (!tiled || 4 * n1 > d.L) return hipErrorInvalidValue;
    switch (d.L) {
#define X(LL)                                                                                  \
  case LL: {                                                                                   \
    using C = CdSd<LL>;                                                                        \
    hipLaunchKernelGGL((k_cds_rows_inv<T, LL>), dim3((n2 + 1) / 2 * 2), dim3(C::THR), 0, s, Y1, Y2, \
                       mask, z, chn, khat, tw, (const cpx<T>*)d.twS, n1, n2);           \
    return hipGetLastError();                                                                  \
  }
      RSFDE_CDS_CASES(X)
#undef X
      default:
        return hipErrorInvalidValue;
    }
  }
  switch (d.L) {
#define X(LL)                                                                                     \
  case LL: {                                                                                      \
    using C = CdCfg<LL>;                                                                          \
    const dim3 g((2 * n2 + C::BR - 1) / C::BR), t(C::THR_R);                                      \
    if (tiled)                                                                                    \
      hipLaunchKernelGGL((k_cd_rows_inv<T, LL, true>), g, t, 0, s, Y1, Y2, mask, z, chn, khat, tw, n1, \
                         n2);                                                                     \
    else                                                                                          \
      hipLaunchKernelGGL((k_cd_rows_inv<T, LL, false>), g, t, 0, s, Y1, Y2, mask, z, chn, khat, tw, \
                         n1, n2);                                                                 \
    return hipGetLastError();                                                                     \
  }
    RSFDE_CD_CASES(X)
#undef X
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace rsfde
