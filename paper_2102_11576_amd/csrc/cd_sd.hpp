// Chirp form of the DST-I on the symmetric sweep, for the two-dimensional
// passes of long lines (n + 1 not a power of two).
//
// With M = n + 1, c_m = exp(i pi m^2 / (2M)) and x extended oddly to |j| <= n,
//   2i sum_{j=1..n} x_j sin(pi j k / M) = c_k sum_{|j| <= n} (x_j c_j) conj(c_{k-j}).
// x_j c_j is odd in j and the kernel conj(c_m) is even, so the convolution runs
// as a circular one of length L >= 4n on odd sequences: sd_engine.hpp's forward
// sweep, a product with the kernel's (even) spectrum, its inverse sweep.  Real
// and imaginary parts of x never mix (the identity is linear over complex x),
// so two real lines share one transform.  Against one real line per complex FFT
// of length 2n - 1 or more (pc_chirp.hpp), a pair of lines takes 9/16 of the
// sub-FFT work of one FFT of twice the length instead of two full FFTs, half
// the LDS traffic and half the threads.
//
// Only positions j <= n <= L/4 are read and written: of a group thread's 16
// register positions (Sd::nat) those with m in 0..4 and 12..15.
//
// Passes and layouts (as the power-of-two passes, with natural positions in
// place of slots):
//   rows fwd: rows 2r, 2r + 1 share a transform; W1 strip-tiled (tile_index)
//   columns:  columns 2c, 2c + 1 share the forward transform; then one transform
//             per column of (w/E1, w/E2), stored as pairs (pair_index)
//   rows inv: the pair (Y1, Y2) of a row is one transform; z = mask ? Y1 S : Y2 S
//
// Bound: at 1000 x 700 one round of blocks, so the serial time of a block's
// transforms; at 2000^2 and beyond the FP64 unit and LDS.  Measured, plain
// chirp form before: CDSD_NUMBERS
#pragma once

#include "sd_kernels.hpp"

namespace rsfde {

// Threads and transforms per block: as the symmetric power-of-two passes; the
// second and third transforms of a column pair run at once on two thread sets
// up to L = kCdConcL (grids too small to fill the GPU).
constexpr int kCdConcL = 4096;
template <int L>
struct CdSd {
  using S = Sd<L>;
  static constexpr int ND = S::TS >= 16 ? 1 : 16 / S::TS;
  static constexpr int THR_R = ND * S::TPD;
  static constexpr bool CONC = L <= kCdConcL;
  static constexpr int THR_C = (CONC ? 2 : 1) * S::TPD;
  // register positions that reach j <= L/4
  static constexpr bool used(int m) { return m <= 4 || m >= 12; }
};

// Position j (1-based) of register m of group p, 0 where it holds no value of
// the line; neg as in Sd::nat.
template <int L>
__device__ __forceinline__ int cd_pos(int p, int m, int n, bool& neg) {
  const int j = Sd<L>::nat(p, m, neg);
  return (j >= 1 && j <= n) ? j : 0;
}

// One transform: group-stage threads (g, group p) hold the chirped odd extension
// in v[] (zero where unused) and receive the convolution at the same positions.
template <typename T, int L, bool MAT>
__device__ __forceinline__ void cd_sd_conv(cpx<T>* v, bool g, int p, int r, int tau, cpx<T> w1,
                                           const cpx<T>* __restrict__ khat,
                                           const cpx<T>* __restrict__ twS, T* region, bool act) {
  using S = Sd<L>;
  using Fs = typename S::Fs;
  constexpr int TWs = sd_tw<L, 1>();
  {
    Roots<T, Fs> rs;
    rs.load_fwd(tau, twS);
    sd_forward<T, L, 1, TWs, MAT>(v, g, p, r, tau, w1, rs, region, act);
  }
  const cpx<T>* kr = khat + r * S::LS;
  static_for<16>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    v[e] = cmul(v[e], kr[Fs::pos(Fs::NS - 1, tau, e)]);
  });
  {
    Roots<T, Fs> rs;
    rs.load_inv(tau, twS);
    sd_inverse<T, L, 1, TWs, MAT>(v, g, p, r, tau, w1, rs, region, act);
  }
}

// v[m] *= c_j (premultiply, with the sign of the extension) for the used
// registers, 0 for the others.
template <typename T, int L>
__device__ __forceinline__ void cd_chirp_in(cpx<T>* v, int p, int n, const cpx<T>* __restrict__ chn) {
  static_for<16>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    if constexpr (CdSd<L>::used(m)) {
      bool neg;
      const int j = cd_pos<L>(p, m, n, neg);
      const cpx<T> c = chn[j ? j - 1 : 0];
      const T s = j ? (neg ? (T)-1 : (T)1) : (T)0;
      const cpx<T> q = cmul(v[m], c);
      v[m] = {s * q.re, s * q.im};
    } else {
      v[m] = {(T)0, (T)0};
    }
  });
}

// v[m] = c_j v[m] with the sign of the extension taken out.
template <typename T, int L>
__device__ __forceinline__ void cd_chirp_out(cpx<T>* v, int p, int n, const cpx<T>* __restrict__ chn) {
  static_for<16>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    if constexpr (CdSd<L>::used(m)) {
      bool neg;
      const int j = cd_pos<L>(p, m, n, neg);
      const cpx<T> c = chn[j ? j - 1 : 0];
      const cpx<T> q = cmul(v[m], c);
      v[m] = neg ? cpx<T>{-q.re, -q.im} : q;
    }
  });
}

// f(m, j) for the register positions that own an output (the self-mirrored
// groups 0 and LS/2 hold each position twice).
template <int L, class Fn>
__device__ __forceinline__ void cd_outputs(int p, int n, Fn&& f) {
  const bool self = p == 0 || p == Sd<L>::LS / 2;
  static_for<16>([&](auto mm) {
    constexpr int m = decltype(mm)::value;
    if constexpr (CdSd<L>::used(m)) {
      bool neg;
      const int j = cd_pos<L>(p, m, n, neg);
      if (j && (m < 8 || !self)) f(mm, j);
    }
  });
}

template <typename T, int L>
__global__ __launch_bounds__(CdSd<L>::THR_R) void k_cds_rows_fwd(
    const double* __restrict__ v, const double* __restrict__ sig, T* __restrict__ Q,
    const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ twL, const cpx<T>* __restrict__ twS, int n1, int n2) {
  using S = Sd<L>;
  using C = CdSd<L>;
  __shared__ T lds[C::ND * S::LEN];
  const int d = threadIdx.x / S::TPD, tg = threadIdx.x % S::TPD;
  const int ra = 2 * (blockIdx.x * C::ND + d), rb = ra + 1;
  const bool va = ra < n2, vb = rb < n2;
  const bool g = tg < S::NG;
  const int r = tg / S::TS, tau = tg % S::TS;
  const double sc = sig ? *sig : 1.0;
  const cpx<T> w1 = twL[g ? tg : 0];
  const double* xa = v + (size_t)(va ? ra : 0) * n1;
  const double* xb = v + (size_t)(vb ? rb : 0) * n1;
  cpx<T> reg[16];
  if (g) {  // loads from clamped addresses, all in flight at once
    static_for<16>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      if constexpr (C::used(m)) {
        bool neg;
        const int j = cd_pos<L>(tg, m, n1, neg);
        const int i = j ? j - 1 : 0;
        const double a = xa[i], b = xb[i];
        reg[m].re = va ? (T)(sc * a) : (T)0;
        reg[m].im = vb ? (T)(sc * b) : (T)0;
      }
    });
    cd_chirp_in<T, L>(reg, tg, n1, chn);
  }
  cd_sd_conv<T, L, true>(reg, g, tg, r, tau, w1, khat, twS, lds + d * S::LEN, true);
  if (!g || !va) return;
  cd_chirp_out<T, L>(reg, tg, n1, chn);
  const int hp = (n2 + 1) >> 1;
  cd_outputs<L>(tg, n1, [&](auto mm, int j) {
    constexpr int m = decltype(mm)::value;
    const size_t i = tile_index(ra, j - 1, hp);  // row b of an odd n2: the zeros loaded for it
    Q[i] = reg[m].re;
    Q[i + 4] = reg[m].im;
  });
}

template <typename T, int L>
__global__ __launch_bounds__(CdSd<L>::THR_C) void k_cds_cols(
    const T* __restrict__ Q, T* __restrict__ P, const double* __restrict__ lamx,
    const double* __restrict__ lamy, const cpx<T>* __restrict__ chn,
    const cpx<T>* __restrict__ khat, const cpx<T>* __restrict__ twL,
    const cpx<T>* __restrict__ twS, int n1, int n2, double kx, double ky, double dpen) {
  using S = Sd<L>;
  using C = CdSd<L>;
  using V2 = typename Vec2<T>::type;
  constexpr int NU = 9;  // registers used: m = 0..4, 12..15
  __shared__ T lds[(C::CONC ? 2 : 1) * S::LEN];
  __shared__ T stash[NU * S::NG];  // the second column's coefficients
  const int h = threadIdx.x / S::TPD, tg = threadIdx.x % S::TPD;
  const int c = xcd_remap(blockIdx.x, gridDim.x);
  const int ca = 2 * c, cb = ca + 1;
  const bool vb = cb < n1;  // ca < n1 always
  const int hp = (n2 + 1) >> 1;
  const bool f0 = h == 0, g = tg < S::NG;
  const int r = tg / S::TS, tau = tg % S::TS;
  const cpx<T> w1 = twL[g ? tg : 0];
  const double lxa = 1.0 - kx * lamx[ca], lxb = 1.0 - kx * lamx[vb ? cb : ca];
  T* region = lds + h * S::LEN;
  cpx<T> reg[16];
  if (g && f0) {
    static_for<16>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      if constexpr (C::used(m)) {
        bool neg;
        const int j = cd_pos<L>(tg, m, n2, neg);
        const V2 q = *(const V2*)(Q + tile_index(j ? j - 1 : 0, ca, hp));
        reg[m].re = q.x;
        reg[m].im = vb ? q.y : (T)0;  // (the strip's padding column is not written)
      }
    });
    cd_chirp_in<T, L>(reg, tg, n2, chn);
  }
  // Three transforms by one copy of the code: the forward one of the column
  // pair, then (w / E1, w / E2) of each column; the last two at once when CONC.
#pragma unroll 1
  for (int q = 0; q < (C::CONC ? 2 : 3); ++q) {
    cd_sd_conv<T, L, false>(reg, g && (f0 || q > 0), tg, r, tau, w1, khat, twS, region,
                            f0 || q > 0);
    if (g && (f0 || q > 0)) cd_chirp_out<T, L>(reg, tg, n2, chn);
    const bool first = q == 0;
    if (!first && g) {  // column 2c + h (CONC) or 2c + q - 1
      const int cw = ca + (C::CONC ? h : q - 1);
      if (cw < n1)
        cd_outputs<L>(tg, n2, [&](auto mm, int j) {
          constexpr int m = decltype(mm)::value;
          *(V2*)(P + pair_index<T>(j - 1, cw, n2)) = V2{reg[m].re, reg[m].im};
        });
    }
    if (first && g && f0) {
      static_for<16>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        if constexpr (C::used(m)) stash[(m <= 4 ? m : m - 7) * S::NG + tg] = reg[m].im;
      });
    }
    if constexpr (C::CONC) __syncthreads();
    if (g && q < (C::CONC ? 1 : 2)) {
      const bool second = C::CONC ? !f0 : q == 1;
      const double lx = second ? lxb : lxa;
      static_for<16>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        if constexpr (C::used(m)) {
          bool neg;
          const int j = cd_pos<L>(tg, m, n2, neg);
          const double e1 = lx - ky * lamy[j ? j - 1 : 0];
          const T w = second ? stash[(m <= 4 ? m : m - 7) * S::NG + tg] : reg[m].re;
          reg[m].re = w / (T)e1;
          reg[m].im = w / (T)(e1 + dpen);
        }
      });
      cd_chirp_in<T, L>(reg, tg, n2, chn);
    }
  }
}

template <typename T, int L>
__global__ __launch_bounds__(CdSd<L>::THR_R) void k_cds_rows_inv(
    const T* __restrict__ P, const uint8_t* __restrict__ mask, double* __restrict__ z,
    const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ twL, const cpx<T>* __restrict__ twS, int n1, int n2) {
  using S = Sd<L>;
  using C = CdSd<L>;
  using V2 = typename Vec2<T>::type;
  __shared__ T lds[C::ND * S::LEN];
  const int d = threadIdx.x / S::TPD, tg = threadIdx.x % S::TPD;
  const int row = blockIdx.x * C::ND + d;
  const bool vr = row < n2;
  const bool g = tg < S::NG;
  const int r = tg / S::TS, tau = tg % S::TS;
  const int rr = vr ? row : 0;
  const cpx<T> w1 = twL[g ? tg : 0];
  cpx<T> reg[16];
  if (g) {
    static_for<16>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      if constexpr (C::used(m)) {
        bool neg;
        const int j = cd_pos<L>(tg, m, n1, neg);
        const V2 q = *(const V2*)(P + pair_index<T>(rr, j ? j - 1 : 0, n2));
        reg[m].re = q.x;
        reg[m].im = q.y;
      }
    });
    cd_chirp_in<T, L>(reg, tg, n1, chn);
  }
  cd_sd_conv<T, L, true>(reg, g, tg, r, tau, w1, khat, twS, lds + d * S::LEN, true);
  if (!g || !vr) return;
  cd_chirp_out<T, L>(reg, tg, n1, chn);
  cd_outputs<L>(tg, n1, [&](auto mm, int j) {
    constexpr int m = decltype(mm)::value;
    const size_t i = (size_t)row * n1 + (j - 1);
    z[i] = mask[i] ? (double)reg[m].re : (double)reg[m].im;
  });
}

}  // namespace rsfde
