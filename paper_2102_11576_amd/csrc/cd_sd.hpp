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
// Passes, all intermediates strip-tiled (tile_index):
//   rows fwd: rows 2r, 2r + 1 share a transform
//   columns:  columns 2c, 2c + 1 share the forward transform, then one transform
//             of w / E1 -> Y1 and one of w / E2 -> Y2
//   rows inv: rows 2r, 2r + 1 of Y1 share one, of Y2 another; z from Y1 where
//             mask = 1, from Y2 where mask = 0
// The fields Y1 and Y2 never share a transform: Y1 is larger by up to dt/eta, and
// its rounding would reach the penalty region's values (1.5e-12 of their largest
// one on 2 x 4096 points, against 1e-15).
//
// Bound: the FP64 unit and LDS of one block per CU (its region and, in the column
// pass, the stash).  Whole preconditioner at 4000^2, plain form -> this one: FP64
// 1859 -> 1122 us, FP32 1092 -> 738; cd_sym_length says where it is used and why.
#pragma once

#include "sd_kernels.hpp"

namespace rsfde {

template <int L>
struct CdSd {
  using S = Sd<L>;
  static constexpr int THR = S::TPD;  // one transform per block
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
                                           const cpx<T>* __restrict__ twS, T* region) {
  using S = Sd<L>;
  using Fs = typename S::Fs;
  constexpr int TWs = sd_tw<S, 1>();
  {
    Roots<T, Fs> rs;
    rs.load_fwd(tau, twS);
    sd_forward<T, S, 1, TWs, MAT>(v, g, p, r, tau, w1, rs, region);
  }
  const cpx<T>* kr = khat + r * S::LS;
  static_for<S::PS>([&](auto ee) {
    constexpr int e = decltype(ee)::value;
    v[e] = cmul(v[e], kr[Fs::pos(Fs::NS - 1, tau, e)]);
  });
  {
    Roots<T, Fs> rs;
    rs.load_inv(tau, twS);
    sd_inverse<T, S, 1, TWs, MAT>(v, g, p, r, tau, w1, rs, region);
  }
}

// A zero that the optimiser cannot see through, added to a table's pointer where
// the table is read again later: the values are then loaded again instead of
// being held in registers across a transform (k_cds_cols spilled 360 registers; an
// opaque pointer would lose its global address space).
__device__ __forceinline__ int opaque_zero() {
  int z = 0;
  asm volatile("" : "+s"(z));
  return z;
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
__global__ __launch_bounds__(CdSd<L>::THR) void k_cds_rows_fwd(
    const double* __restrict__ v, const double* __restrict__ sig, T* __restrict__ Q,
    const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ twL, const cpx<T>* __restrict__ twS, int n1, int n2) {
  using S = Sd<L>;
  using C = CdSd<L>;
  __shared__ T lds[S::LEN];
  const int tg = threadIdx.x;
  const int ra = 2 * blockIdx.x, rb = ra + 1;
  const bool vb = rb < n2;  // ra < n2 always
  const bool g = tg < S::NG;
  const int r = tg / S::TS, tau = tg % S::TS;
  const double sc = sig ? *sig : 1.0;
  const cpx<T> w1 = twL[g ? tg : 0];
  const double* xa = v + (size_t)ra * n1;
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
        reg[m].re = (T)(sc * a);
        reg[m].im = vb ? (T)(sc * b) : (T)0;
      }
    });
    cd_chirp_in<T, L>(reg, tg, n1, chn);
  }
  cd_sd_conv<T, L, true>(reg, g, tg, r, tau, w1, khat, twS, lds);
  if (!g) return;
  int te = tg;  // the epilogue's positions are formed after the sweeps, not held across
  asm volatile("" : "+v"(te));
  cd_chirp_out<T, L>(reg, te, n1, chn + opaque_zero());
  const int hp = (n2 + 1) >> 1;
  cd_outputs<L>(te, n1, [&](auto mm, int j) {
    constexpr int m = decltype(mm)::value;
    const size_t i = tile_index(ra, j - 1, hp);  // row b of an odd n2: the zeros loaded for it
    Q[i] = reg[m].re;
    Q[i + 4] = reg[m].im;
  });
}

template <typename T, int L>
__global__ __launch_bounds__(CdSd<L>::THR) void k_cds_cols(
    const T* __restrict__ Q, T* __restrict__ Y1, T* __restrict__ Y2,
    const double* __restrict__ lamx, const double* __restrict__ lamy,
    const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ twL, const cpx<T>* __restrict__ twS, int n1, int n2, double kx,
    double ky, double dpen) {
  using S = Sd<L>;
  using C = CdSd<L>;
  using V2 = typename Vec2<T>::type;
  constexpr int NU = 9;  // registers used: m = 0..4, 12..15
  __shared__ T lds[S::LEN];
  __shared__ T stash[2 * NU * S::NG];  // the pair's coefficients, for the second scaling
  const int tg = threadIdx.x;
  const int c = xcd_remap(blockIdx.x, gridDim.x);
  const int ca = 2 * c, cb = ca + 1;
  const bool vb = cb < n1;  // ca < n1 always
  const int hp = (n2 + 1) >> 1;
  const double lxa = 1.0 - kx * lamx[ca], lxb = 1.0 - kx * lamx[vb ? cb : ca];
  cpx<T> reg[16];
  if (tg < S::NG) {
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
  // pair, then w / E1 and w / E2.
#pragma unroll 1
  for (int q = 0; q < 3; ++q) {
    // nothing per point is hoisted out of the loop: opaque thread index and tables
    int th = tg;
    asm volatile("" : "+v"(th));
    const int zo = opaque_zero();
    const bool g = th < S::NG;
    cd_sd_conv<T, L, false>(reg, g, th, th / S::TS, th % S::TS, twL[g ? th : 0], khat + zo,
                            twS + zo, lds);
    if (!g) continue;  // (no barrier follows in this round)
    cd_chirp_out<T, L>(reg, th, n2, chn + zo);
    if (q == 0) {
      static_for<16>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        constexpr int u = m <= 4 ? m : m - 7;
        if constexpr (C::used(m)) {
          stash[(2 * u) * S::NG + th] = reg[m].re;
          stash[(2 * u + 1) * S::NG + th] = reg[m].im;
        }
      });
    } else {
      T* Y = q == 1 ? Y1 : Y2;
      cd_outputs<L>(th, n2, [&](auto mm, int j) {  // (cb = n1: the padding column)
        constexpr int m = decltype(mm)::value;
        *(V2*)(Y + tile_index(j - 1, ca, hp)) = V2{reg[m].re, reg[m].im};
      });
    }
    if (q < 2) {
      const double pen = q == 0 ? 0.0 : dpen;
      const double* ly = lamy + zo;
      static_for<16>([&](auto mm) {
        constexpr int m = decltype(mm)::value;
        constexpr int u = m <= 4 ? m : m - 7;
        if constexpr (C::used(m)) {
          bool neg;
          const int j = cd_pos<L>(th, m, n2, neg);
          const double l = ky * ly[j ? j - 1 : 0];
          reg[m].re = stash[(2 * u) * S::NG + th] / (T)(lxa + pen - l);
          reg[m].im = stash[(2 * u + 1) * S::NG + th] / (T)(lxb + pen - l);
        }
      });
      cd_chirp_in<T, L>(reg, th, n2, chn + zo);
    }
  }
}

template <typename T, int L>
__global__ __launch_bounds__(CdSd<L>::THR) void k_cds_rows_inv(
    const T* __restrict__ Y1, const T* __restrict__ Y2, const uint8_t* __restrict__ mask,
    double* __restrict__ z, const cpx<T>* __restrict__ chn, const cpx<T>* __restrict__ khat,
    const cpx<T>* __restrict__ twL, const cpx<T>* __restrict__ twS, int n1, int n2) {
  using S = Sd<L>;
  using C = CdSd<L>;
  __shared__ T lds[S::LEN];
  const int tg = threadIdx.x;
  const int field = blockIdx.x & 1, ra = blockIdx.x & ~1, rb = ra + 1;
  const bool vb = rb < n2;  // ra < n2 always
  const bool g = tg < S::NG;
  const int r = tg / S::TS, tau = tg % S::TS;
  const int hp = (n2 + 1) >> 1;
  const T* Y = field ? Y2 : Y1;
  const cpx<T> w1 = twL[g ? tg : 0];
  cpx<T> reg[16];
  if (g) {
    static_for<16>([&](auto mm) {
      constexpr int m = decltype(mm)::value;
      if constexpr (C::used(m)) {
        bool neg;
        const int j = cd_pos<L>(tg, m, n1, neg);
        const size_t i = tile_index(ra, j ? j - 1 : 0, hp);
        const T a = Y[i], b = Y[i + 4];
        reg[m].re = a;
        reg[m].im = vb ? b : (T)0;
      }
    });
    cd_chirp_in<T, L>(reg, tg, n1, chn);
  }
  cd_sd_conv<T, L, true>(reg, g, tg, r, tau, w1, khat, twS, lds);
  if (!g) return;
  int te = tg;  // the epilogue's positions are formed after the sweeps, not held across
  asm volatile("" : "+v"(te));
  cd_chirp_out<T, L>(reg, te, n1, chn + opaque_zero());
  const bool want = field == 0;
  cd_outputs<L>(te, n1, [&](auto mm, int j) {
    constexpr int m = decltype(mm)::value;
    const size_t i = (size_t)ra * n1 + (j - 1);
    if ((mask[i] != 0) == want) z[i] = (double)reg[m].re;
    if (vb && (mask[i + n1] != 0) == want) z[i + n1] = (double)reg[m].im;
  });
}

}  // namespace rsfde
