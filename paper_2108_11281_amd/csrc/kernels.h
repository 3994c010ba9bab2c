// Launchers of the HIP kernels.  All vectors are RHS-major blocks: column k of
// length n starts at k*n.  `active` (nullable) is a per-column flag array on
// the device: kernels skip columns whose flag is 0 (converged solves).
#pragma once

#include <hip/hip_ext.h>

#include <type_traits>
#include <vector>

#include "common.h"

namespace mlmc {

constexpr int kThreads = 256;
constexpr int kMaxPartials = 1024;  // per-column partial sums of a reduction

// Measurement mode: when non-null, the next timed launch records, for each
// column k, its active flag at tlog[k] (written by the kernel itself).
int*& timing_log();

// Measurement mode: when non-null, launches made through MLMC_LAUNCH carry
// these events in the dispatch itself (hipExtLaunchKernel), so the events
// time the kernel's execution and not the gaps between launches.  The first
// such launch records `start`; every one records `stop` (the last one wins).
struct LaunchEvents {
  hipEvent_t start = nullptr, stop = nullptr;
  bool used = false;
};
LaunchEvents*& timing_events();

#define MLMC_LAUNCH(kern, grid, block, shmem, stream, ...)                                   \
  do {                                                                                       \
    ::mlmc::LaunchEvents* ev_ = ::mlmc::timing_events();                                     \
    if (ev_) {                                                                               \
      hipExtLaunchKernelGGL(kern, grid, block, shmem, stream, ev_->used ? nullptr : ev_->start, \
                            ev_->stop, 0, __VA_ARGS__);                                      \
      ev_->used = true;                                                                      \
    } else {                                                                                 \
      hipLaunchKernelGGL(kern, grid, block, shmem, stream, __VA_ARGS__);                     \
    }                                                                                        \
  } while (0)

// ----- blocks of vectors (deflation): FP64, RHS-major [m][n] -----------------
// row chunks of the Gram reduction over n for an ma x mb product
int gram_chunks(int64_t n, int ma, int mb);
// part[c][i][j] = sum over chunk c of A[i][r] B[j][r] (nchunks chunks of n)
void gram_partials(const double* A, int ma, const double* B, int mb, int64_t n, int nchunks,
                   double* part, hipStream_t s);
// C[i][j] = sum_c part[c][i][j] in chunk order (row-major ma x mb)
void gram_finish(const double* part, int nchunks, int ma, int mb, double* C, hipStream_t s);
// Out[j][r] = beta X[j][r] + alpha sum_{m < kk} U[m][r] C[m * ldc + j], j < nc;
// Out may equal X; X is not read when beta == 0
void block_combine(const double* U, int kk, const double* C, int ldc, const double* X,
                   double* Out, int nc, int64_t n, double alpha, double beta, hipStream_t s);

// streaming device copy of bytes (a multiple of 16, 16-byte aligned pointers)
void stream_copy(const void* src, void* dst, size_t bytes, hipStream_t s);

// ----- vectors ---------------------------------------------------------------
template <typename T>
void vec_zero(T* x, int64_t n, int nb, const int* active, hipStream_t s);
template <typename T>
void vec_copy(const T* x, T* y, int64_t n, int nb, const int* active, hipStream_t s);
template <typename To, typename From>
void vec_convert(const From* x, To* y, int64_t n, int nb, const int* active, hipStream_t s);

// number of partial sums per column for a reduction over n elements
int reduce_blocks(int64_t n);
// partials[k*nblk + b] (re, im) = sum over block b of conj(x) y, column k
template <typename T>
void vec_dot_partials(const T* x, const T* y, int64_t n, int nb, const int* active,
                      c64* partials, hipStream_t s);
// out[k] = fixed-order sum of column k's nblk partials
void finish_sums(const c64* partials, int nblk, int nb, c64* out, hipStream_t s);

// ----- Krylov scalars (one thread per column) --------------------------------
// finish_sums into pq, then cg_alpha from it, in one launch (same values);
// lastcorr (nullable): alpha rz of active columns (the CG step's share of b^H x)
void finish_alpha(const c64* partials, int nblk, int nb, c64* pq, const c64* rz,
                  const int* active, c64* alpha, hipStream_t s, c64* lastcorr = nullptr);
// finish_sums into rr of the active columns, then their convergence test
// (mark_converged's, without the count)
void finish_mark(const c64* partials, int nblk, int nb, c64* rr, const c64* ref, double tol2,
                 int* active, hipStream_t s);
// the scalars of a refinement of the refined CG, active columns: bd = sums of pbd
// (nullable: bd is given), rr_new = rr_upd = sums of prr, the stated error, rz = 0
// (so the next beta is 0) where rr_new exceeds factor x the recursion's own
// residual rr_rec, the convergence test and the count of columns left
void refine_finish(const c64* pbd, const c64* prr, int nblk, int nb, c64* bd, c64* rr_upd,
                   c64* rr_new, const c64* rr_rec, c64* rz, c64* err, const c64* bb, double tol2,
                   double factor, int* active, int* count, hipStream_t s);
// finish_sums into rz_new, then cg_beta from it, in one launch (same values)
void finish_beta(const c64* partials, int nblk, int nb, c64* rz_new, c64* rz, const int* active,
                 c64* beta, hipStream_t s);
// alpha = active ? rz/pq : 0   (Hermitian CG, real rz and pq)
void cg_alpha(const c64* rz, const c64* pq, const int* active, c64* alpha, int nb,
              hipStream_t s);
// beta = rz_new/rz ; rz = rz_new
void cg_beta(const c64* rz_new, c64* rz, const int* active, c64* beta, int nb,
             hipStream_t s);
// active[k] &= (rr[k] > tol2 * ref[k]); count = number still active
void mark_converged(const c64* rr, const c64* ref, double tol2, int* active, int nb,
                    int* count, hipStream_t s);
void count_active(const int* active, int nb, int* count, hipStream_t s);
void set_all_active(int* active, int nb, hipStream_t s);
void set_count(int* count, int value, hipStream_t s);
// count = number of active columns with rr <= delta2 * rr_upd or rr <= tol2 * bb
void refine_due(const c64* rr, const c64* rr_upd, const c64* bb, double delta2, double tol2,
                const int* active, int nb, int* count, hipStream_t s);
// err[k] = |bd[k]| * sqrt(rr_new[k]/rr_old[k]) for active columns
void ir_stated_error(const c64* bd, const c64* rr_old, const c64* rr_new, const int* active,
                     c64* err, int nb, hipStream_t s);
// dst[k] = active[k] ? src[k] : dst[k]
void select_active(c64* dst, const c64* src, const int* active, int nb, hipStream_t s);
// x += alpha p ; r -= alpha q ; partials of |r|^2.  x_zero: x is taken as zero
// and not read (the first update of a solve), x = alpha p
template <typename T>
void cg_update_xr(T* x, T* r, const T* p, const T* q, const c64* alpha, int64_t n,
                  int nb, const int* active, c64* partials, hipStream_t s,
                  bool x_zero = false);
// p = z + beta p
template <typename T>
void cg_update_p(T* p, const T* z, const c64* beta, int64_t n, int nb,
                 const int* active, hipStream_t s);
// refinement fold in one pass: y += d, partials of b^T d (reduce_blocks(n)
// blocks per column, as vec_dot_partials(b, d)), d = 0.  y_zero: y is taken as
// zero and not read (the first fold of a solve), y = 0 + d
void ir_fold(double* y, float* d, const double* b, int64_t n, int nb, const int* active,
             c64* partials, hipStream_t s, bool y_zero = false);
// r = b32 = b rounded to FP32 (nb columns of n); *inexact = 0 when every entry of
// b is an FP32 number (b32 then holds b exactly), else 1; partials of b^T b as
// vec_dot_partials(b, b) writes them (reduce_blocks(n) per column, same sums)
void rhs_fp32(const double* b, float* r, float* b32, int64_t n, int nb, int* inexact,
              c64* partials, hipStream_t s);
// y64 += convert(d)
template <typename T64, typename T32>
void ir_accumulate(T64* y, const T32* d, int64_t n, int nb, const int* active,
                   hipStream_t s);
// out = a - b
template <typename T>
void vec_sub(const T* a, const T* b, T* out, int64_t n, int nb, hipStream_t s);
// y += x (active columns)
template <typename T>
void vec_add_to(T* y, const T* x, int64_t n, int nb, const int* active, hipStream_t s);
// y += a[k] * x  (column scalars)
template <typename T>
void vec_axpy_cols(T* y, const T* x, const c64* a, int64_t n, int nb,
                   const int* active, hipStream_t s);

// ----- probes and quadratic forms -------------------------------------------
template <typename T>
void probes_write(T* out, int64_t n, int nb, uint64_t seed, uint64_t problem,
                  uint64_t first_sample, uint64_t level, uint64_t stream,
                  hipStream_t s);
// partials of x_k^H y_k with x_k regenerated from the RNG
template <typename T>
void probe_dot_partials(const T* y, int64_t n, int nb, uint64_t seed, uint64_t problem,
                        uint64_t first_sample, uint64_t level, uint64_t stream,
                        c64* partials, hipStream_t s);

// ----- dense coarsest level -------------------------------------------------
// inverse of the n x n matrix A held row-major with leading dimension lda in M
// (overwritten) by blocked Gauss-Jordan with partial pivoting; out receives
// A^{-1} row-major with leading dimension n.  Work: rowbuf kGjPanel + 1
// elements, colbuf n, tbuf kGjPanel * n, ipiv 2n + 1 ints; ipiv[2n] is set to
// 1 when a pivot is zero or not a number (A singular)
constexpr int kGjPanel = 64;
template <typename T>
void dense_inverse(T* M, int n, int64_t lda, T* out, T* rowbuf, T* colbuf, T* tbuf, int* ipiv,
                   hipStream_t s);
// trace partial: out = sum_i A[i][i] (single block)
template <typename T>
void dense_trace(const T* A, int n, c64* out, hipStream_t s);
// Z[k][i] = sum_j At[j][i] B[k][j], k < nb: the coarsest solve z_k = A^{-1} b_k
// with At the transposed inverse.  ld (0: n): leading dimension of At.  Real T
// with ld a multiple of 16 (dense_mfma_layout): the MFMA tile kernel, for any
// n, with At zero-padded to ld x ld and given in the layout of dense_pack4;
// otherwise (ld == n) a plain row-major At.
template <typename T>
void dense_apply(const T* At, const T* B, T* Z, int n, int nb, const int* active,
                 hipStream_t s, int ld = 0);
template <typename T>
constexpr bool dense_mfma_layout(int ld) {
  return (std::is_same<T, float>::value || std::is_same<T, double>::value) && ld % 16 == 0;
}
// the MFMA tile kernel's layout of an ld x ld row-major matrix At (ld a
// multiple of 4): out[((j / 4) ld + i) 4 + j % 4] = At[j][i], so the four
// consecutive rows j a lane reads for one column i are contiguous
template <typename T>
void dense_pack4(const T* At, T* out, int ld, hipStream_t s);
// the same for a complex matrix (n a multiple of 8) in an order of its own
// (dense_complex_elems reals), from the transposed matrix
int64_t dense_complex_elems(int n);
template <typename T>
void dense_complex_pack(const T* At, typename Traits<T>::real* M, int n, hipStream_t s);
template <typename T>
void dense_complex_apply(const typename Traits<T>::real* M, const T* b, T* z, int n, int nb,
                         const int* active, hipStream_t s);
// out[j][i] = in[i][j] (n x n)
template <typename T>
void dense_transpose(const T* in, T* out, int n, hipStream_t s);

// ----- 2D Poisson stencil: A = d I - c (grid neighbours), N x N Dirichlet -----
// ----- small 2D Poisson grids (one workgroup per right-hand side) -------------
constexpr int kSmallSide = 128;   // largest top side
constexpr int kSmallCoarse = 64;  // largest coarsest side
constexpr int kSmallPad = 4;      // row padding of the coarsest level's LDS planes
// levels from a top level (index 0) down to the coarsest (index nl - 1)
template <typename T>
struct SmallGrid {
  int nl, pre, post;
  int side[8], off[8];      // off: LDS elements of the levels 1 .. nl - 2 (b, then x)
  T d[8], c[8], dinv[8];
  T wh;                     // omega / 2
  int mp;                   // coarsest side rounded up to 16
  const T *basis, *ilam;    // its sine basis and reciprocal eigenvalues, mp x mp, zero padded
};
// bytes of LDS of a workgroup (refined: small_refined's)
template <typename T> size_t small_lds(const SmallGrid<T>& q, bool refined);
// lets the kernels use the device's whole LDS (once per device and context)
void small_setup();
// z = `cycles` V-cycles for b, from z0 (nullable: zero); partials (nullable): b^T z, one
// per column; nl == 1: the coarsest solve alone
template <typename T>
void small_vcycle(const T* b, T* z, const T* z0, const SmallGrid<T>& q, int cycles, int nb,
                  const int* active, c64* partials, hipStream_t s);
// whole solves: CG in precision T, and FP32 CG with FP64 refinement; rres: final
// |b - A x|^2 (re) and iterations (im), bb: |b|^2 (re) and refinements (im);
// pbuf, rbuf, xbuf: planes of nb columns
template <typename T>
void small_pcg(const T* b, T* x, T* pbuf, T* rbuf, const SmallGrid<T>& q, int child_cycles, double tol,
               int max_iter, int nb, c64* rres, c64* bb, c64* lastcorr, hipStream_t s);
void small_refined(const double* b, double* y, float* pbuf, float* xbuf,
                   const SmallGrid<float>& q, int child_cycles, double d, double c, double tol, double inner_tol, int max_it, int nb,
                   c64* rres, c64* bb, c64* err, hipStream_t s);

// partial-sum counts per column of the tiled kernels
int poisson_march_tiles(int N);   // apply / residual
// fused Gauss-Seidel pass of `sweeps` (1 or 2) sweeps, `rows` per segment
template <typename T>
int poisson_gs_tiles(int N, int rows, int sweeps);
// the three segment lengths the sweep is compiled for (ascending)
template <typename T>
void gs_rows_options(int out[3]);
template <typename T>
void poisson_dense_build(T* aug, int N, double d, double c, hipStream_t s);
// y = A x ; optional partials of conj(x)^T y (pass partials = nullptr to skip)
template <typename T>
void poisson_apply(const T* x, T* y, int N, double d, double c, int nb,
                   const int* active, c64* partials, hipStream_t s);
// p_new = z + beta p_old ; partials of conj(p_new)^T A p_new (even sides >= 64)
template <typename T>
void poisson_direction(const T* p_old, const T* z, const c64* beta, T* p_new, int N, double d,
                       double c, int nb, const int* active, c64* partials, hipStream_t s);
// x += alpha p ; r -= alpha A p ; partials of |r|^2 (even sides >= 64); x_zero: x
// holds no values yet and is taken as zero
template <typename T>
void poisson_xr(T* x, T* r, const T* p, const c64* alpha, int N, double d, double c, int nb,
                const int* active, c64* partials, hipStream_t s, bool x_zero);
// y_out = y_in + x32 (y_in nullptr: zero), r = b - A y_out in FP32, partials of
// b^T x32 and |r|^2 (poisson_fold_tiles per column); y_in and y_out are different
// planes, dst[k] = which for the active columns (even sides >= 64)
int poisson_fold_tiles(int N);
template <typename Tb>
void poisson_fold_residual(const Tb* b, const double* yin, const float* x, double* yout, float* r,
                           int N, double d, double c, int nb, const int* active, c64* pbd,
                           c64* prr, int* dst, int which, hipStream_t s);
// y[k] = alt[k] where dst[k] != 0
void poisson_collect(double* y, const double* alt, const int* dst, int64_t n, int nb,
                     hipStream_t s);
// r = b - A x (Tr may be lower precision) ; optional partials of |r|^2
template <typename Tb, typename Tx, typename Tr>
void poisson_residual(const Tb* b, const Tx* x, Tr* r, int N, double d, double c,
                      int nb, const int* active, c64* partials, hipStream_t s);
// one pass of `sweeps` (1 or 2; 2 needs N >= 64) red-black Gauss-Seidel sweeps,
// fused: xout = S^sweeps(xin + omega/2 P ec ; b), red first (reverse: black
// first) in every sweep; xin == nullptr means 0, ec == nullptr no correction;
// partials (nullable): shares of conj(b)^T xout, gs_tiles per column; rows:
// segment length (one of gs_rows_options; a tuning choice that does not change
// the swept values).  Two sweeps in one pass equal two one-sweep passes bit for
// bit.
template <typename T>
void poisson_rbgs_fused(const T* xin, const T* b, T* xout, const T* ec, double omega, int N,
                        double d, double c, int nb, const int* active, bool reverse,
                        c64* partials, int rows, int sweeps, hipStream_t s);
// last pre-smoothing pass: xout = S^2(xin ; b) (two fused sweeps, red first;
// xin == nullptr means 0) and rc = R (b - A xout) in the same pass; N even, >= 64
template <typename T>
void poisson_rbgs_restrict(const T* xin, const T* b, T* xout, T* rc, int N, double d, double c,
                           int nb, const int* active, int rows, hipStream_t s);
// rc = R (b - A x), R = P^T, P the orthonormal 2x2 aggregation (entries 1/2)
template <typename T>
void poisson_residual_restrict(const T* b, const T* x, T* rc, int N, double d,
                               double c, int nb, const int* active, hipStream_t s);
// xc = R x
template <typename T>
void agg2d_restrict(const T* x, T* xc, int N, int nb, const int* active, hipStream_t s);
// x = beta*x + omega * P ec
template <typename T>
void agg2d_prolong(const T* ec, T* x, int N, double omega, double beta, int nb,
                   const int* active, hipStream_t s);

// ----- 3D 7-point variable-coefficient operator, N^3 cells, Dirichlet faces -----
// Face coefficients of one level: k[3][N][N][N+1] (x-faces [z][y][f], y-faces
// [z][x][f], z-faces [y][x][f]); the stencil kernels read the cell-major
// couplings kl[3][N^3 + N^2] (face below cell i in x, y, z; zero on the
// boundary; padded) and diag dg[i] = shift + the six faces of cell i.  `cols`
// (1, 2, 4 or 8): right-hand sides per thread, a tuning choice that does not
// change results.
int varcoef_blocks(int N);  // partial sums per column of residual / update_apply
// r = b - A x ; b == nullptr: r = A x (partials then of conj(x)^T r)
template <typename Tb, typename T, typename Tr>
void varcoef_residual(const Tb* b, const T* x, Tr* r, const typename Traits<T>::real* kl,
                      const typename Traits<T>::real* dg, int N, int nb, int cols,
                      const int* active, c64* partials, hipStream_t s);
// one in-place red-black Gauss-Seidel sweep (reverse: black first); zero_init:
// x = 0 on entry (not read); ec (nullable): x + omega P ec is swept instead of
// x (the coarse-grid correction folded into the sweep; the result is written
// to x)
template <typename T>
void varcoef_rbgs(const T* b, T* x, const typename Traits<T>::real* kl,
                  const typename Traits<T>::real* dg, int N, int nb, int cols, const int* active,
                  bool zero_init, bool reverse, const T* ec, double omega, hipStream_t s);
// one red-black sweep fused into one out-of-place pass (both colours; reverse:
// black first): xout = S(xin + omega/sqrt(8) P ec ; b); xin == nullptr means 0,
// ec nullable; `cols` in {1, 2, 4}: right-hand sides per lane.  For even sides
// up to 128 (varcoef_march_ok).
bool varcoef_march_ok(int N);
template <typename T>
void varcoef_rbgs_march(const T* xin, const T* b, T* xout, const T* ec, double omega,
                        const typename Traits<T>::real* kl, const typename Traits<T>::real* dg,
                        int N, int nb, int cols, const int* active, bool reverse,
                        hipStream_t s);
// xc = R (b - A x) when residual, else xc = R x; R the orthonormal 2x2x2
// aggregation (entries 1/sqrt(8)).  swept: x has just left a forward sweep (its
// second colour's residual is zero and not formed)
template <typename T>
void varcoef_restrict(const T* b, const T* x, T* xc, const typename Traits<T>::real* kl,
                      const typename Traits<T>::real* dg, int N, bool residual, bool swept, int nb,
                      int cols, const int* active, hipStream_t s);
// x = beta x + omega P ec
template <typename T>
void varcoef_prolong(const T* ec, T* x, int N, double omega, double beta, int nb,
                     const int* active, hipStream_t s);
// p_new = z + beta p_old ; q = A p_new ; partials of conj(p_new)^T q
template <typename T>
void varcoef_update_apply(const T* p_old, const T* z, const c64* beta, T* p_new, T* q,
                          const typename Traits<T>::real* kl,
                          const typename Traits<T>::real* dg, int N, int nb, int cols,
                          const int* active, c64* partials, hipStream_t s);
// Galerkin faces of the next level: kc = 1/8 (sum of the 4 fine faces covered)
void varcoef_coarsen(const double* kf, double* kc, int N, hipStream_t s);
// diagonal, followed by its reciprocals, and cell-major couplings (FP64 and FP32) of
// one level
void varcoef_diag(const double* k, double shift, int N, double* d64, float* d32, double* kl64,
                  float* kl32, hipStream_t s);
// left half of aug (n x 2n row-major, n = N^3) = the dense operator
void varcoef_dense(const double* k, const double* diag, int N, double* aug, hipStream_t s);

// ----- learned smoother (2-spin lattice; N a multiple of 16) --------------------
// weights: 4032 FP32 values, W1 [16][8][3][3], W2 [16][16][3][3], W3 [4][16][3][3]
int nn_num_weights();
int nn_frag_count();          // packed BF16 B fragments (16 bytes each)
int nn_crop_in_elems();       // BF16 per training-crop input (22 * 22 * 8)
int nn_crop_out_elems();      // FP32 per training-crop target (16 * 16 * 4)
int nn_crop_side();           // 22
// link features (cos, sin of theta_mu) in BF16 [site][4]; theta [2][N][N] FP64
void nn_links(const double* theta, void* links, int N, hipStream_t s);
// BF16 B fragments of the three layers from the FP32 master weights
void nn_pack(const float* w, void* frag, hipStream_t s);
// x += s * net(r / s), s^2 = rr[k].re * inv_n per column (skipped when 0)
void nn_apply(const c32* r, c32* x, const c64* rr, double inv_n, const void* links,
              const void* frag, int N, int nb, const int* active, hipStream_t s);
// forward + backward of ncrops crops (crop order[i], or i when order is null):
// (inputs BF16, or FP32 that are rounded) per-crop gradients, then grad = their fixed-order sum and *loss = the mean
// squared error
void nn_train_step(const void* in, bool in_fp32, const float* tgt, const int* order, int ncrops,
                   const void* frag, const float* w, float* gpart, double* lpart, float* grad,
                   double* loss, hipStream_t s);
// Adam step t (from 1) on the FP32 master weights, and their fragments as nn_pack's
void nn_adam(float* w, float* m, float* v, const float* g, void* frag, double lr, double b1,
             double b2, double eps, int t, hipStream_t s);
// training crops from FP64 residual / error fields (origin: column, y0, x0 per crop)
void nn_crops(const c64* r, const c64* e, const c64* rr, double inv_n, const void* links,
              const int* origin, int ncrops, int N, void* in, float* tgt, hipStream_t s);

// ----- complex lattice operators (Wilson 2-spin, block stencils, transfers) ---
int wilson_residual_blocks(int N);
int bsr_residual_blocks(int Nc, int dof);
// r = b - D x ; b == nullptr: r = D x (partials then of conj(x)^T r)
template <typename Tb, typename T, typename Tr>
void wilson_residual(const Tb* b, const T* x, Tr* r, const T* U, int N, double diag, int nb,
                     const int* active, c64* partials, hipStream_t s);
template <typename T>
void wilson_rbgs(const T* b, T* x, const T* U, int N, double diag, int nb, const int* active,
                 bool zero_init, bool reverse, hipStream_t s);
// one red-black sweep with both colours in one launch, out of place: xout =
// S(xin) (xin unread when zero_init, else it must differ from xout); needs
// wilson_rbgs_fused_ok(N) (side divisible by 16)
bool wilson_rbgs_fused_ok(int N);
template <typename T>
void wilson_rbgs_fused(const T* b, const T* xin, T* xout, const T* U, int N, double diag, int nb,
                       const int* active, bool zero_init, bool reverse, hipStream_t s);
// block stencils: form 0 = a thread per (site, column), 1 = a wave per site
// and 64 columns with the site's blocks read wave-uniformly (a tuning choice;
// results agree up to rounding); partial sums always come from form 0
template <typename Tb, typename T, typename Tr>
void bsr_residual(const Tb* b, const T* x, Tr* r, const T* B, int Nc, int dof, int nb,
                  const int* active, c64* partials, int form, hipStream_t s);
template <typename T>
void bsr_rbgs(const T* b, T* x, const T* B, const T* Dinv, int Nc, int dof, int nb,
              const int* active, bool zero_init, bool reverse, int form, hipStream_t s);
// the same with four or eight unknowns per (coarse) site, on the matrix cores; the
// restriction needs rows of blk dofF fine unknowns that are a multiple of eight
inline bool bsr8_ok(int dof) { return dof == 4 || dof == 8; }
int bsr8_residual_blocks(int Nc);
template <typename T>
void bsr8_rbgs(const T* b, T* x, const T* B, const T* Dinv, int Nc, int dof, int nb,
               const int* active, bool zero_init, bool reverse, hipStream_t s);
// a sweep of x + omega P xc (Q: the aggregates' bases, dof columns), the sum not stored
template <typename T>
void bsr8_prolong_rbgs(const T* xc, const T* Q, int blk, double omega, const T* b, T* x,
                       const T* B, const T* Dinv, int Nc, int dof, int nb, const int* active,
                       bool reverse, hipStream_t s);
template <typename T, typename Tr>
void bsr8_residual(const T* b, const T* x, Tr* r, const T* B, int Nc, int dof, int nb,
                   const int* active, c64* partials, hipStream_t s);
// xc = P^H (b - A x) of an x that a sweep (reverse as there) has just left
template <typename T>
void bsr8_residual_restrict(const T* b, const T* x, T* xc, const T* B, const T* Q, int Nc, int dof,
                            int blk, int nb, const int* active, bool reverse, hipStream_t s);
// the same from the two-spin lattice, blk even
template <typename T>
void wilson_residual_restrict(const T* b, const T* x, T* xc, const T* U, const T* Q, int N,
                              double diag, int blk, int dofC, int nb, const int* active,
                              bool reverse, hipStream_t s);
template <typename T>
void agg8_restrict(const T* x, T* xc, const T* q, int Nf, int dofF, int blk, int dofC, int nb,
                   const int* active, hipStream_t s);
template <typename T>
void agg_restrict(const T* x, T* xc, const T* q, int Nf, int dofF, int blk, int dofC, int nb,
                  const int* active, hipStream_t s);
template <typename T>
void agg_prolong(const T* xc, T* x, const T* q, int Nf, int dofF, int blk, int dofC,
                 double omega, double beta, int nb, const int* active, hipStream_t s);
void wilson_links(const double* theta, c64* U64, c32* U32, int N, hipStream_t s);
// gauge Laplacian (4 + m) I - linked neighbours as 1 x 1 blocks B[site][5]
void gauge_blocks(const c64* U, int N, double diag, c64* B, hipStream_t s);
void agg_orthonormalise(const c64* V, c64* q, int Nf, int dofF, int blk, int nv, bool split,
                        hipStream_t s);
void galerkin_blocks(const c64* Bf, const c64* U, double wdiag, const c64* q, int Nf, int dofF,
                     int blk, int nv, c64* Bc, hipStream_t s);
void dense_from_stencil(const c64* Bf, const c64* U, double wdiag, int Nf, int dof, c64* aug,
                        hipStream_t s);
void block_diag_inverse(const c64* B, c64* Dinv64, c32* Dinv32, int ns, int dof, hipStream_t s);
// the 5 dof-blocks of every row of a block stencil (or the Wilson operator) as
// column indices and values, 5 * dof entries per row, direction-major
void stencil_entries(const c64* Bf, const c64* U, double wdiag, int Nf, int dof, int* cols,
                     c64* vals, hipStream_t s);

// ----- batched flexible GMRES helpers ------------------------------------------
// one step of classical Gram-Schmidt: h = V^H w, w -= V h, wn2 = |w|^2, w /= |w|
template <typename T>
void krylov_orthonormalise(const T* V, int64_t vstride, int nv, T* w, int64_t n, int nb,
                           const int* active, c64* h, c64* wn2, c64* partials, hipStream_t s);
// dst = src / |src| and nrm2 = |src|^2
template <typename T>
void krylov_normalise(T* dst, const T* src, int64_t n, int nb, const int* active, c64* nrm2,
                      c64* partials, hipStream_t s);
template <typename T>
void krylov_combine(const T* Z, int64_t vstride, const c64* y, int ldy, const int* dims, T* d,
                    int64_t n, int nb, const int* start, hipStream_t s);
void givens_init(c64* H, c64* cs, c64* sn, c64* g, int* dims, const c64* beta2,
                 const int* active, int m, int nb, hipStream_t s);
void givens_step(c64* H, c64* cs, c64* sn, c64* g, int* dims, const c64* h, const c64* wn2,
                 const c64* beta2, double tol, int j, int m, int* active, int nb, int* count,
                 hipStream_t s);
void givens_solve(c64* H, c64* cs, c64* sn, c64* g, int* dims, c64* y, const int* start, int m,
                  int nb, hipStream_t s);

// ----- general sparse (CSR) operators -----------------------------------------
// The kernels read sliced ELLPACK copies (SELL-64): slice s holds 64
// consecutive rows (or colour-class positions) and w_s = (sptr[s+1] -
// sptr[s]) / 64 entries per row, entry e of lane l at sptr[s] + 64 e + l, so
// the column indices and values of a wave's rows load coalesced and every lane
// runs the same trip count.  Entries keep the row's column order; rows shorter
// than w_s are padded with value 0 and their own row as column.
//
// A by rows, diagonal included (device arrays; values in precision T); rp/ci/v
// are the plain CSR arrays (dense build of the coarsest level)
template <typename T>
struct CsrMat {
  int n = 0;                  // rows
  int ncol = 0;               // columns (the length of the vectors it multiplies)
  const int* rp = nullptr;    // n + 1 row offsets
  const int* ci = nullptr;    // column of each entry
  const T* v = nullptr;       // value of each entry
  const int* sptr = nullptr;  // SELL-64 slice offsets (ceil(n/64) + 1), FP64 only
  const int* sci = nullptr;
  const T* sv = nullptr;
};
// the off-diagonal part with rows grouped by colour class (ascending within a
// class): class c owns positions off[c]..off[c+1]-1 (host offsets); position k is
// the row rows[k].x with entries rows[k].y .. rows[k].z - 1 and di[k] = 1 / a_ii
template <typename T>
struct CsrSweep {
  const int4* rows = nullptr;
  const int* ci = nullptr;
  const T *v = nullptr, *di = nullptr;
  std::vector<int> off;
};
// aggregation to the next level: agg[i] = aggregate of unknown i; the members
// of J are arows[aptr[J]..aptr[J+1]-1] (ascending); fs[i] = cs[agg[i]] = 1/sqrt|J|
template <typename T>
struct CsrAgg {
  int nc = 0;
  const int *agg = nullptr, *aptr = nullptr, *arows = nullptr;
  const T *fs = nullptr, *cs = nullptr;
};
// FP64 building blocks on RHS-major blocks (from the SELL-64 copies)
int csr_blocks(int n);  // partial sums per column of csr_residual
// r = b - A x (r = A x when b is null); partials as the stencil residuals
void csr_residual(const double* b, const double* x, double* r, const CsrMat<double>& A, int nb,
                  const int* active, c64* partials, hipStream_t s);
// xc = R x, R = P^T
void csr_restrict(const double* x, double* xc, const CsrAgg<double>& G, int n, int nb,
                  const int* active, hipStream_t s);
// x = beta x + omega P ec
void csr_prolong(const double* ec, double* x, const CsrAgg<double>& G, int n, double omega,
                 double beta, int nb, const int* active, hipStream_t s);
// y = beta y + w M x for a rectangular M (M.n x M.ncol; y has M.n, x M.ncol
// entries per column; beta = 0: y is not read): the general prolongation
// (M = P) and restriction (M = R = P^T) between CSR levels
void csr_spmm(const double* x, double* y, const CsrMat<double>& M, double w, double beta, int nb,
              const int* active, hipStream_t s);
// left half of the n x 2n augmented matrix [A | .] (rows of width 2n)
void csr_dense(const CsrMat<double>& A, double* aug, hipStream_t s);

// ----- the solver's kernels on interleaved blocks of W vectors ----------------
// (element i of vector c at [i W + c]; from the plain CSR copies)
int rows_per_block(int n);
int rows_blocks(int n);  // partial sums per column of the reductions below
// RHS-major FP64 block -> interleaved FP64 (dst, nullable) and To (dst2, nullable)
template <typename To>
void rows_in(const double* src, double* dst, To* dst2, int64_t n, int W, hipStream_t s);
// interleaved block -> RHS-major FP64 block
template <typename Ts>
void rows_out(const Ts* src, double* dst, int64_t n, int W, hipStream_t s);
// One Gauss-Seidel sweep in place over the colour classes (reverse: last class
// first).  Each class is one launch, except the trailing run of classes of at
// most tail_rows rows each (csr_tail_start; 0: none), which shares launches of up
// to kMaxTailClasses classes: one workgroup of kTailWaves waves per vector, a
// barrier between classes.  The rows of a class are independent, so both
// schedules give the same result.
constexpr int kTailWaves = 16;
constexpr int kMaxTailClasses = 64;
struct CsrTail {
  int count, reverse;
  int off[kMaxTailClasses + 1];
};
inline int csr_tail_start(const std::vector<int>& off, int tail_rows) {
  int c = (int)off.size() - 1;
  if (tail_rows <= 0) return c;
  while (c > 0 && off[c] - off[c - 1] <= tail_rows) --c;
  return c;
}
template <typename T>
void rows_gs_sweep(const T* b, T* x, const CsrSweep<T>& S, int W, int tail_rows, const int* active,
                   bool reverse, hipStream_t s);
// r = b - A x ; partials (nullable) of |r|^2
template <typename T, typename Tr>
void rows_residual(const T* b, const T* x, Tr* r, const CsrMat<T>& A, int W, const int* active,
                   c64* partials, hipStream_t s);
// p_new = z + beta p_old, q = A p_new, partials of p_new^T q
template <typename T>
void rows_update_apply(const T* p_old, const T* z, const c64* beta, T* p_new, T* q,
                       const CsrMat<T>& A, int W, const int* active, c64* partials, hipStream_t s);
// x += alpha p ; r -= alpha q ; partials of |r|^2 (x_zero: x taken as zero)
template <typename T>
void rows_xr(T* x, T* r, const T* p, const T* q, const c64* alpha, int n, int W, const int* active,
             c64* partials, bool x_zero, hipStream_t s);
// partials of x^T y
template <typename T>
void rows_dot(const T* x, const T* y, int n, int W, const int* active, c64* partials,
              hipStream_t s);
// y += d, partials of b^T d, d = 0 (y_zero: y taken as zero)
void rows_fold(double* y, float* d, const double* b, int n, int W, const int* active,
               c64* partials, bool y_zero, hipStream_t s);
// y = beta y + w M x (M rectangular; beta = 0: y is not read)
template <typename T>
void rows_spmm(const T* x, T* y, const CsrMat<T>& M, double w, double beta, int W,
               const int* active, hipStream_t s);
// rc = R r ; x = beta x + omega P ec, aggregation
template <typename T>
void rows_agg_sum(const T* r, T* rc, const CsrAgg<T>& A, int W, const int* active, hipStream_t s);
template <typename T>
void rows_prolong(const T* ec, T* x, const CsrAgg<T>& A, int n, double omega, double beta, int W,
                  const int* active, hipStream_t s);
// Z = A^-1 B from the packed transposed inverse (dense_pack4)
template <typename T>
void rows_dense(const T* Pk, const T* B, T* Z, int n, int ld, int W, const int* active,
                hipStream_t s);

// ----- small levels of a matrix-given hierarchy, one vector per workgroup -----
constexpr int kSmallCsrLds = 160 * 1024;  // a compute unit's LDS: the iterate fits
constexpr int kSmallCsrDense = 256;       // largest coarsest level solved in the kernel
// SELL-64 rows (slice s: ptr[s] .. ptr[s + 1] - 1, entry-major), 16-bit columns
template <typename T>
struct SellView {
  const int* ptr = nullptr;
  const unsigned short* ci = nullptr;
  const T* v = nullptr;
};
// a smoothed level; unknowns numbered by position in the sweep's order, classes
// padded to whole slices (np positions in all)
template <typename T>
struct SmallCsrLevel {
  int np = 0, ncls = 0;
  const int* cls = nullptr;          // first slice of each class (ncls + 1)
  const int* row = nullptr;          // natural index of a position (-1: padding)
  SellView<T> off;                   // off-diagonal part
  const T *di = nullptr, *dd = nullptr;  // 1 / a_ii and a_ii (padding: 0)
  const int* dp = nullptr;               // off-diagonal entries before a_ii in its row
  // transfers to the next level (its positions; natural order on the coarsest):
  // aggregation (members of J in mem[mptr[J]..], scales) or, with mptr null, R and P
  const int *mptr = nullptr, *mem = nullptr, *agg = nullptr;
  const T *cs = nullptr, *fs = nullptr;
  SellView<T> R, P;
  T *b = nullptr, *x = nullptr, *r = nullptr;  // blocks [vector][position]
};
template <typename T>
struct SmallCsrCoarse {
  int n = 0, ld = 0;
  const T* inv = nullptr;            // packed transposed inverse (dense_pack4)
  T *b = nullptr, *x = nullptr;      // blocks [vector][unknown]
};
enum { kSmallCsrAll = 0, kSmallCsrDown = 1, kSmallCsrUp = 2 };
void small_csr_setup();
// one V-cycle x = M b of the nl levels lev (device array), b and x interleaved
// blocks of W vectors of the first one: all of it (coarsest solve included, n <=
// kSmallCsrDense), or the parts before and after the coarsest solve
template <typename T>
void small_csr(const SmallCsrLevel<T>* lev, int nl, int np_max, const SmallCsrCoarse<T>& cs,
               const T* b, T* x, int W, int pre, int post, double omega, int mode,
               const int* active, hipStream_t s);
// `sweeps` sweeps of level *lev (np positions) alone from xin (nullptr: zero; may be x);
// element i of vector c at [i row_stride + c col_stride]
template <typename T, typename U>
void small_csr_sweeps(const SmallCsrLevel<T>* lev, int np, const U* b, const U* xin, U* x, int W,
                      int64_t row_stride, int64_t col_stride, int sweeps, bool reverse,
                      const int* active, hipStream_t s);

}  // namespace mlmc
