// Internal declarations shared by the host driver and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fft_engine.hpp"

namespace rsfde {

constexpr int kMaxRestart = 64;       // largest GMRES restart length supported
constexpr int kRedThreads = 256;      // threads per block of the streaming reductions
constexpr int kMaxRedBlocks = 512;    // upper bound on blocks of a streaming reduction
constexpr int kMaxN = 4096;           // grid points per direction (FFT lengths <= 8192)

// Members of a batched launch (independent solves of one grid, rsfde_batch_*):
// slot k of the launch's member grid dimension works on member m[k], whose
// per-member arrays start m[k] * stride doubles after the pointers the launch
// is given.  A single plan launches one member with stride 0.
constexpr int kMaxBatch = 32;
struct Members {
  int32_t n;             // members in the launch (grid dimension z of the FFT
                         // kernels, y of the streaming Krylov kernels)
  int32_t m[kMaxBatch];  // their member indices
  size_t stride;         // doubles between consecutive members' arrays
  __host__ __device__ size_t off(int k) const { return (size_t)m[k] * stride; }
  static Members one() {
    Members b{};
    b.n = 1;
    return b;
  }
};

// Points per thread of the register-resident FFT of length L: all up to L = 8 (no
// rounded roots at all), 4 up to L = 256, 8 up to L = 1024, 16 above.  A pass
// over short lines is bound by one block's serial time (instruction fetch of the
// unrolled sweep, one radix butterfly after the other) on small grids and by the
// waves in flight on large ones; fewer points halve the code and the registers.  Measured, 16 points before:
// fused pass C 22.0 -> 11.2 us and pass A 10.5 -> 5.0 us at 63^2 (L = 128),
// chirp column pass 26.9 -> 15.0 us at 256^2 (L = 512), mv_rows 101 -> 89 us
// and z pass of the preconditioner 257 -> 213 us at 255^3 (L = 512).  8 points
// up to L = 256: fused pass 14.4, pass A 6.6 us.  From L = 2048 on the extra
// register stage costs more than the registers give: 8 points took mv_cols +
// mv_rows at 2047^2 (L = 4096) 59.6 -> 68.6 us, at 4095^2 (L = 8192) 322 -> 503.
constexpr int fft_pts(int L) { return L <= 8 ? L : (L <= 256 ? 4 : (L <= 1024 ? 8 : 16)); }

// Lengths whose exchanges may move both parts at once (lds_exchange, CX): at 4 and
// 8 points per thread twice the LDS still leaves 16 wavefronts per CU.  Used where
// registers or the grid hold a kernel to that anyway: pass B of 3-D plans (169 ->
// 148 us at 255^3) and their raw sine transforms (91 -> 88), the convolution of the
// fused pass, the chirp passes (200^2 22.5 -> 21.8 us), the product's column pass on
// small views and all of its passes up to L = 256.  The row passes of the
// preconditioner lose wavefronts by it at L = 512 (255^3: pass A 66 -> 77 us, pass
// C 101 -> 121).
constexpr bool fft_cx(int L) { return L <= 1024; }

// Transforms per block of the row passes: one wavefront's worth, or one
// transform where that takes more than a wavefront.  A transform inside one
// wavefront needs no block barrier, and small grids spread over more CUs: with
// 256-thread blocks 63^2 filled four of them (fused pass C 10.6 -> 7.7 us).
// Long views gain or lose little (255^3: pass A 67 -> 62 us, mv_rows 89 -> 92).
constexpr int row_ffts(int tpf) { return tpf >= 64 ? 1 : 64 / tpf; }

// Column pairs per block of the column passes, where tpf threads run one
// transform.  Large views: 512 threads (16 pairs at most), so that a block
// reads whole lines of each row.  Views whose large blocks would not give every
// CU one (kSmallGridBlocks): a wavefront's worth (at least 2 pairs).  At 63^2
// pass B 8.4 -> 4.9 us and mv_cols 6.7 -> 3.9, at 256^2 mv_cols 9.0 -> 6.5;
// beyond the line small blocks read part lines and lose (mv_cols at 255^3 +9 %).
constexpr int kSmallGridBlocks = 256;
constexpr int col_ffts_large(int tpf) {
  return 512 / tpf > 16 ? 16 : (512 / tpf > 0 ? 512 / tpf : 1);
}
constexpr int col_ffts_small(int tpf) { return tpf >= 64 ? 2 : 64 / tpf; }

// Values the device writes for the host after each Arnoldi step.  Lives in
// pinned, device-visible host memory; the host reads it after an event.
struct HostStatus {
  double est[kMaxRestart];  // |g_{j+1}|: residual-norm estimate after inner step j
  double beta;              // ||r|| of the last residual kernel
  double bnorm;             // ||b||
  int32_t flags;            // bit 0: non-finite value seen
  int32_t gram_seq;         // sequence number of the last Gram block written (s-step form)
};
constexpr int kFlagNonFinite = 1;

// Device-side Arnoldi / Givens state.
struct KrylovState {
  double H[(kMaxRestart + 1) * kMaxRestart];  // column-major, ld = kMaxRestart + 1
  double cs[kMaxRestart];
  double sn[kMaxRestart];
  double g[kMaxRestart + 1];
  double vscale[kMaxRestart + 1];             // V_i is stored unnormalised: v_i = vscale[i] * V_i
  double h2[kMaxRestart + 1];                 // second Gram-Schmidt pass (reorthogonalisation)
  int32_t gram_done;                          // blocks of a Gram finish done (0 between launches)
};
constexpr int kLdH = kMaxRestart + 1;

// Largest number of basis vectors one streaming launch handles; longer
// restarts are processed in chunks of this size.
constexpr int kChunk = 32;

// Reduction workspace: rows of per-block partial sums [value][block], written by a
// streaming kernel and read by the finishing kernel launched after it, or by the
// kernel that uses the sums.  The orthogonalisation needs two regions of kChunk
// rows, one per Gram-Schmidt pass, since one kernel reads the first pass's while
// it writes the second's; they start at rows 0 and kRedSecond.
constexpr int kRedSecond = kChunk + 1;
constexpr int kRedRows = kRedSecond + kChunk + 1;
struct RedWork {
  double* partial;     // [kRedRows][kMaxRedBlocks]
};

// ----------------------------- FFT kernels --------------------------------
// Row pass of the matrix-vector product:
//   out = coef * (C_x z) + diag * z - theta * sub,
//   diag = (mode==0) ? 1 + dpen (1 - mask) : 0 (sub = NULL: no shift term),
// where C_x is the Toeplitz matrix whose circulant embedding of length L has
// the symbol `sym` (already divided by L, stored in register-position order).
// tiled: out in the strip-tiled layout (tile_index; 8 ceil(n1/4) ceil(n2/2)
// values), as the column pass reads t on two-dimensional plans.
// Batched (mb.n > 1 or a nonzero stride): z, out and sub advance by the
// member offset; with mk given, coef = -mk[offset] (mk: the member's k).
hipError_t launch_mv_rows(int L, const double* z, const uint8_t* mask, double* out,
                          const double* sym, const void* tw, int n1, int n2,
                          double coef, double dpen, int mode, hipStream_t s,
                          const double* sub = nullptr, double theta = 0.0, bool tiled = false,
                          const Members& mb = Members::one(), const double* mk = nullptr);
// Column pass: out = coef * (C_y z) + (mode==0 ? t : 0) on `batch` [n2][n1]
// slices, slice b at offset b * bstride of z, t and out.  tiled (mode 0, one
// slice): t in the strip-tiled layout.
// z32 (mode 0, tiled, one slice): z is a float array (the preconditioned
// basis kept in FP32).
hipError_t launch_mv_cols(int L, const void* z, const double* t, double* out,
                          const double* sym, const void* tw, int n1, int n2,
                          double coef, int mode, hipStream_t s, int batch = 1,
                          size_t bstride = 0, bool tiled = false,
                          const Members& mb = Members::one(), const double* mk = nullptr,
                          bool z32 = false);

// Tables of the symmetric sine transform along one direction (sd_kernels.hpp;
// used by the tiled passes when L >= kSdMinL and twS is given): twS, the
// twiddles exp(-2 pi i j / (L/16)) in the pass's precision; msl (x only), the
// mirror slots of the upper halves of blocks 0 and 8 (2 L/16 entries, -1 at
// frequency L/2).  With the symmetric form the x slots follow Sd<L>::slot and
// pass B's y eigenvalues are indexed by block position (9 L/16 entries).
struct SdTabs {
  const void* twS = nullptr;
  const int32_t* msl = nullptr;
  bool many = false;  // L = kSdManyL with 16 points per thread (sd_many)
};

// Sine-transform preconditioner, three passes; T = float or double internally.
// tiled = false: Q, P1, P2 are [n2][n1+1] arrays.  tiled = true: Q is
// strip-tiled (tile_index; 8 ceil((n1+1)/4) ceil(n2/2) T values) and the
// interleaved P1/P2 pairs (array P1, P2 unused) are in row segments
// (pair_index; 2 W ceil((n1+1)/W) n2 T values, W = 64 / sizeof(T)).
// Pass A: Q[r][slot] = raw x-sine sums of (sig * v) rows.
// Batched: v, sig (when given), Q advance by the member offset (in doubles).
template <typename T>
hipError_t launch_pc_rows_fwd(int Lx, const double* v, const double* sig, T* Q,
                              const void* tw, int n1, int n2, bool tiled, hipStream_t s,
                              const Members& mb = Members::one(), const SdTabs& sd = SdTabs{});
// Pass B: column sine transforms of Q, the two eigenvalue scalings, two inverse
// column transforms -> P1, P2 (slot layout in x, natural rows in y).
// Batched: Q, P1, P2 advance by the member offset; with mk given, the
// member's (kx, ky) are mk[offset], mk[offset + 1].
template <typename T>
hipError_t launch_pc_cols(int Ly, const T* Q, T* P1, T* P2, const T* lamx_slot,
                          const T* lamy_pos, const void* tw, int n1, int n2,
                          double kx, double ky, double dpen, double Kfac, bool tiled,
                          hipStream_t s, const Members& mb = Members::one(),
                          const double* mk = nullptr, const SdTabs& sd = SdTabs{});
// Raw sine transform (DST-I without normalisation) along the columns of
// `batch` slices of [rows][ncol] values (slice b at offset b * bstride), ncol even:
//   out[k-1][c] = sum_{p=1..rows} in[p-1][c] sin(pi k p / (rows + 1)), k = 1..rows;
// inB / outB (both or neither): a second array in the same launch.  in and out
// must not overlap.  L = 2 (rows + 1).
template <typename T>
hipError_t launch_dst_cols(int L, const T* inA, T* outA, const T* inB, T* outB, const void* tw,
                           int ncol, int rows, int batch, size_t bstride, hipStream_t s);
// Pass C: inverse row transforms of P1, P2 and the mask combine -> z (FP64).
template <typename T>
hipError_t launch_pc_rows_inv(int Lx, const T* P1, const T* P2,
                              const uint8_t* mask, double* z, const void* tw,
                              int n1, int n2, bool tiled, hipStream_t s,
                              const Members& mb = Members::one(), const SdTabs& sd = SdTabs{});

// Pass C fused with the matrix-vector row pass (n1 + 1 a power of two, so
// L = 2(n1+1) is also the convolution length): z = pass C output (stored),
// t = (1 + dpen (1 - mask)) z + coef (C_x z) - theta sub (sub may be NULL);
// tiled: P1/P2 pairs in row segments, t strip-tiled over n1 columns.
// Batched: P1, P2, z, t, sub advance by the member offset; with mk given,
// coef = -mk[offset].  z32: z is stored in FP32 (a float array; tiled only),
// and the product uses the stored (rounded) values.
template <typename T>
hipError_t launch_pc_rows_inv_mv(int L, const T* P1, const T* P2,
                                 const uint8_t* mask, void* z, double* t, const void* twT,
                                 const void* tw64, const double* sym, double coef, double dpen,
                                 const double* sub, double theta, int n1, int n2, bool tiled,
                                 hipStream_t s, const Members& mb = Members::one(),
                                 const double* mk = nullptr, bool z32 = false,
                                 const SdTabs& sd = SdTabs{});

// Chirp (Bluestein) form of the same preconditioner for any n (n + 1 not a
// power of two), T internals.  Per direction: chn (n chirp values), khat (the
// convolution kernel's spectrum) and the twiddles of length L.  Plain form
// (twS = NULL): L >= 2n - 1, khat in register-position order (L entries).
// Symmetric form of long lines (cd_sd.hpp; tiled only): L >= 4n, twS the
// twiddles of length L / 16, khat by block position (9 L / 16 entries).
struct CdDir {
  int L;
  const void *chn, *khat, *tw, *twS;
};
// Length L of the symmetric form for an axis of n points and `lines` lines where it
// is used, 0 where the plain form is.
//
// Axes of at most 2048 points take the plain form.  In FP64 the symmetric one is the
// faster there by some per cent at L = 4096 (1000 x 700 82 -> 77 us when both were
// measured, the plain one 74 since) and not at the neighbouring lengths (2000^2, L =
// 8192, 305 -> 313; 300 x 200, L = 2048, 27 -> 32); in FP32 its error is the larger.
//
// Beyond, the plain transform is one 8192-point FFT per block and reads single
// columns: 4000^2 FP64 1859 -> 1122 us, FP32 1092 -> 738; 3000 x 1000 FP64 317 -> 247.
// But two lines in one transform halve the blocks and lengthen each, which pays
// only where the plain form's blocks outnumber what runs at once: one per CU in
// FP64 and three in FP32, two lines per row in the last row pass, one per column.
// Plain / symmetric: rows, FP64 4000 x 128 58.9 / 66.5 us, 4000 x 150 84.2 / 78.6;
// FP32 3000 x 300 77.9 / 82.1, 3000 x 400 86.9 / 84.3.  Columns, FP64 256 x 2049
// 73.2 / 85.1, 300 x 2049 137 / 99; in FP32 the symmetric column pass is level with
// the plain one at 16 columns (44.5 / 44.4) and ahead of it from there.
//
// Error of the symmetric form against FP64 products, plain form = 1: FP32 0.7 to 0.95
// over the whole result, on the penalty region alone (values dt/eta smaller) 1.05 to
// 1.6, as two lines share a transform; FP64 1.00 and 1.0 to 1.15.
constexpr int cd_sym_length(int n, int lines, bool rows, bool fp32) {
  const int least = rows ? (fp32 ? 385 : 129) : (fp32 ? 1 : 257);
  return n > 2048 && lines >= least ? 16384 : 0;
}
// W1, Y1, Y2: [n2][n1] arrays, or strip-tiled (tile_index).
template <typename T>
hipError_t launch_cd_rows_fwd(const CdDir& d, const double* v, const double* sig, T* W1, int n1,
                              int n2, bool tiled, hipStream_t s);
template <typename T>
hipError_t launch_cd_cols(const CdDir& d, const T* W1, T* Y1, T* Y2, const double* lamx,
                          const double* lamy, int n1, int n2, double kx, double ky, double dpen,
                          bool tiled, hipStream_t s);
template <typename T>
hipError_t launch_cd_rows_inv(const CdDir& d, const T* Y1, const T* Y2, const uint8_t* mask,
                              double* z, int n1, int n2, bool tiled, hipStream_t s);
// Three-dimensional plans: out = S in along the rows of `batch` slices of
// [rows][ncol] T values (slice b at offset b * bstride, the columns c < ncol);
// inB / outB (both or neither): a second array in the same launch.
template <typename T>
hipError_t launch_cd_dst_cols(int L, const T* inA, T* outA, const T* inB, T* outB, const void* chn,
                              const void* khat, const void* tw, int ncol, int rows, int batch,
                              size_t bstride, hipStream_t s);

// BF16 / MFMA form of the same preconditioner (dense sine-transform GEMMs,
// any n; dimensions padded to multiples of 128).  A1T holds 2 n1p n2p values
// (hi and lo parts of the split intermediate).
hipError_t launch_pc_gemm_bf16(const double* v, const double* sig, double* z, const uint8_t* mask,
                               const __bf16* Sx, const __bf16* Sy, const __bf16* Sx_lo,
                               const __bf16* Sy_lo, const float* lamx,
                               const float* lamy, __bf16* A1T, __bf16* R12T, __bf16* G,
                               int n1, int n2, int n1p, int n2p, double kx, double ky,
                               double dpen, hipStream_t s);

// ---------------------------- Krylov kernels ------------------------------
// b = u + dt * mask * (f(u) + src_scale * src)  (src may be NULL), x0 = 2u - u2
// (or u), ||b|| -> hs->bnorm.
// Batched (Krylov kernels): every per-member pointer (vectors, bases, the
// KrylovState, the reduction partials) advances by the member offset, and hs
// is an array indexed by member; u and u2 advance by ustride per member.
hipError_t launch_rhs(const double* u, const double* u2, const uint8_t* mask, double dt,
                      int f_kind, const double* src, double src_scale, double* b, double* x0,
                      size_t N, RedWork rw, HostStatus* hs, hipStream_t s,
                      const Members& mb = Members::one(), size_t ustride = 0);
// ||v|| -> hs->bnorm.
hipError_t launch_norm(const double* v, size_t N, RedWork rw, HostStatus* hs, hipStream_t s);
hipError_t launch_residual(const double* b, const double* w, double* r, size_t N,
                           RedWork rw, KrylovState* ks, HostStatus* hs, hipStream_t s,
                           const Members& mb = Members::one());
// h_i = <v_i, w>, i < nv.  finish: into column j of H (second = false) or into
// ks->h2 (second = true: the reorthogonalisation pass); otherwise (nv <= kChunk)
// the partials are left for the kernel that uses them.
hipError_t launch_multidot(const double* V, size_t ldv, int nv, const double* w, size_t N,
                           RedWork rw, KrylovState* ks, int j, bool second, bool finish,
                           hipStream_t s, const Members& mb = Members::one());
// The finishing kernel of one chunk's dots: dst[v0 + v] from nb partials each.
hipError_t launch_multidot_finish(int nb, int nv, RedWork rw, KrylovState* ks, double* dst, int v0,
                                  bool second, hipStream_t s, const Members& mb = Members::one());
// The orthogonalisation of one Arnoldi step, vout = w - sum_{i<nv} h_i v_i by
// one (reorth = false) or two passes of classical Gram-Schmidt: first the dots
// of the first pass, then everything else: the updates, the second pass's dots,
// ||vout||, the Givens step of column j and the residual estimate in hs.
hipError_t launch_orth_dots(const double* V, size_t ldv, int nv, const double* w, size_t N,
                            RedWork rw, KrylovState* ks, int j, hipStream_t s,
                            const Members& mb = Members::one());
hipError_t launch_orth_update(const double* V, size_t ldv, int nv, const double* w, double* vout,
                              size_t N, RedWork rw, KrylovState* ks, int j, bool reorth,
                              HostStatus* hs, hipStream_t s, const Members& mb = Members::one());
// x += sum_{i<jc} y_i Z_i with R y = g; scaled = true multiplies y_i by
// vscale[i] (Z = the unnormalised basis V: left preconditioning).
// Batched: member slot k uses jc[k] vectors (jcs given; jc = their maximum).
// z32: Z is a float array (vector i at Z + i * ldz floats).
hipError_t launch_update(const void* Z, size_t ldz, int jc, double* x, size_t N,
                         KrylovState* ks, bool scaled, hipStream_t s,
                         const Members& mb = Members::one(), const int32_t* jcs = nullptr,
                         bool z32 = false);
// x += sum_{i<jc} c_i Z_i with the coefficients c given (device array).
// As launch_update with the coefficients y given on the host (jc doubles,
// passed to the kernels as arguments).
hipError_t launch_update_coef(const void* Z, size_t ldz, int jc, double* x, size_t N,
                              const double* c_host, hipStream_t s, bool z32 = false);

// s-step blocks (krylov_block.hip).  G (pinned, device-visible, [nr][16]) =
// [V_0 .. V_{nr-1}]^T [V_{m1} .. V_{m1+s-1}]; gpart holds
// 16 * 16 * kGramMaxTiles * kGramBlocks partial sums.
constexpr int kGramBlocks = 1024;
constexpr int kGramMaxTiles = 5;  // up to 80 Gram rows
// After G is written and fenced, the finishing kernel stores seq to *seq_flag
// (pinned host memory), so that the host can wait for G by polling that word.
// done_count: a device word that is 0 between launches (the finishing
// kernel's blocks count themselves on it and the last one resets it).
hipError_t launch_bgram(const double* V, size_t ld, int nr, int m1, int s, size_t N,
                        double* gpart, double* G_host_dev, int32_t* seq_flag, int32_t seq,
                        int32_t* done_count, hipStream_t st);
// V_{m1..m1+s-1} <- (V_{m1..} - V_{0..nq-1} C) R^{-1}; coef = C [nq][s] then R^{-1} [s][s]
// (nq*s + s*s doubles).  Up to kCoefArgMax coefficients travel as kernel
// arguments (coef is then a host pointer); more are read from coef_dev, which
// the caller has filled on the stream.
constexpr int kCoefArgMax = 448;
struct CoefArgs {
  double v[kCoefArgMax];
};
hipError_t launch_bupd(double* V, size_t ld, int nq, int m1, int s, size_t N, const double* coef,
                       const double* coef_dev, hipStream_t st);
hipError_t launch_scale_copy(const double* v, const double* sig, double* z, size_t N,
                             hipStream_t s);
hipError_t launch_adj_lambda(const double* mu, const double* u_prev, const uint8_t* mask,
                             double dt, int f_kind, double* lam_prev, size_t N, hipStream_t s);
hipError_t launch_dot_accum(const double* a, const double* b, size_t N, RedWork rw,
                            int counter_slot, double* acc, hipStream_t s);

int red_blocks(size_t N);
// Grid of a streaming kernel without a cross-block reduction (grid-stride
// loops over double2 pairs): up to 4096 blocks, for memory-level parallelism.
int stream_blocks(size_t N);

}  // namespace rsfde
