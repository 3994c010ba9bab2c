// General sparse operators given in compressed sparse row form: the FP64 building
// blocks on RHS-major blocks (residual and product, the transfers of Sec. 4.1);
// the solver's kernels work on interleaved blocks (kernels_rows.hip).  The matrix
// is read from sliced ELLPACK copies (SELL-64, described with CsrMat): a wave
// takes the 64 rows of one slice, so each load of column indices and values is
// one coalesced 256-byte access and all lanes run the same trip count.  A
// thread takes one row (or one aggregate) and COLS right-hand sides, so each
// index and value is loaded once for COLS columns; the gathers from x stay
// close in memory when neighbouring unknowns carry nearby indices.  Row sums
// run in the stored column order.  Indices are 32-bit (n, nnz < 2^31); column
// offsets 64-bit.
#include "kernels.h"

namespace mlmc {
namespace {

__device__ __forceinline__ bool col_on(const int* active, int col, int nb) {
  return col < nb && (!active || active[col]);
}

// U entries of a SELL-64 row: indices and values first, then the gathers of
// every column, so U gathers per column are in flight; sums in entry order
template <typename T, int COLS, int U>
__device__ __forceinline__ void sell_chunk(const int* __restrict__ sci, const T* __restrict__ sv,
                                           int at, const T* __restrict__ x, int64_t n, int col0,
                                           const bool* on, T* acc) {
  int j[U];
  T a[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    j[u] = sci[at + u * 64];
    a[u] = sv[at + u * 64];
  }
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    if (!on[q]) continue;
    const T* xq = x + (int64_t)(col0 + q) * n;
    T g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) g[u] = xq[j[u]];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[q] += a[u] * g[u];
  }
}

// Row sum over one SELL-64 slice: acc[q] += sum_e v_e x_q[j_e] for the w
// entries of this lane's row, in stored order, in chunks of 8, 4 and 1
template <typename T, int COLS>
__device__ __forceinline__ void sell_row_sum(const int* __restrict__ sci,
                                             const T* __restrict__ sv, int base, int w,
                                             const T* __restrict__ x, int64_t n, int col0,
                                             const bool* on, T* acc) {
  int e = 0;
  for (; e + 8 <= w; e += 8) sell_chunk<T, COLS, 8>(sci, sv, base + e * 64, x, n, col0, on, acc);
  if (e + 4 <= w) {
    sell_chunk<T, COLS, 4>(sci, sv, base + e * 64, x, n, col0, on, acc);
    e += 4;
  }
  for (; e < w; ++e) sell_chunk<T, COLS, 1>(sci, sv, base + e * 64, x, n, col0, on, acc);
}

// r = b - A x (or r = A x when b is null); partials (nullable): per column and
// block of |r|^2 (or x^T A x).  Block = 4 slices = 256 consecutive rows.
template <typename T, int COLS>
__global__ __launch_bounds__(kThreads) void k_csr_residual(
    const T* __restrict__ b, const T* __restrict__ x, T* __restrict__ r,
    const int* __restrict__ sptr, const int* __restrict__ sci, const T* __restrict__ sv, int n,
    int nb, const int* active, c64* partials, int* tlog) {
  __shared__ double red[16];
  const int col0 = blockIdx.y * COLS;
  if (tlog && blockIdx.x == 0 && threadIdx.x < COLS && col0 + (int)threadIdx.x < nb)
    tlog[col0 + threadIdx.x] = active ? active[col0 + threadIdx.x] : 1;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  const bool in = i < n;
  bool on[COLS];
  T acc[COLS];
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    on[q] = col_on(active, col0 + q, nb);  // uniform over the block
    acc[q] = T(0);
  }
  if (in) {
    const int sl = i >> 6;
    const int base = sptr[sl] + (i & 63);
    sell_row_sum<T, COLS>(sci, sv, base, (sptr[sl + 1] - sptr[sl]) >> 6, x, n, col0, on, acc);
  }
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    if (!on[q]) continue;
    const int64_t off = (int64_t)(col0 + q) * n;
    double dre = 0.0, dim = 0.0;
    if (in) {
      T val = acc[q];
      if (b) {
        val = b[off + i] - val;
        cdot_acc(dre, dim, val, val);
      } else {
        cdot_acc(dre, dim, x[off + i], val);
      }
      r[off + i] = val;
    }
    if (partials) {
      block_sum2<kThreads>(dre, dim, red);
      if (threadIdx.x == 0) partials[(int64_t)(col0 + q) * gridDim.x + blockIdx.x] = {dre, dim};
    }
  }
}

// y = beta y + w M x, M rectangular (m rows, x of length nx per column)
template <typename T, int COLS>
__global__ __launch_bounds__(kThreads) void k_csr_spmm(
    const T* __restrict__ x, T* __restrict__ y, const int* __restrict__ sptr,
    const int* __restrict__ sci, const T* __restrict__ sv, int m, int nx, T w, T beta, int nb,
    const int* active, int* tlog) {
  const int col0 = blockIdx.y * COLS;
  if (tlog && blockIdx.x == 0 && threadIdx.x < COLS && col0 + (int)threadIdx.x < nb)
    tlog[col0 + threadIdx.x] = active ? active[col0 + threadIdx.x] : 1;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= m) return;
  bool on[COLS];
  T acc[COLS];
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    on[q] = col_on(active, col0 + q, nb);
    acc[q] = T(0);
  }
  const int sl = i >> 6;
  sell_row_sum<T, COLS>(sci, sv, sptr[sl] + (i & 63), (sptr[sl + 1] - sptr[sl]) >> 6, x, nx,
                        col0, on, acc);
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    if (!on[q]) continue;
    T* yq = y + (int64_t)(col0 + q) * m + i;
    *yq = (beta == T(0)) ? w * acc[q] : beta * *yq + w * acc[q];
  }
}

// rc_J = s_J sum_{i in J} r_i, a thread per aggregate J and vector, members in
// ascending order
template <typename T>
__global__ __launch_bounds__(kThreads) void k_csr_agg_sum(
    const T* __restrict__ r, T* __restrict__ rc, const int* __restrict__ aptr,
    const int* __restrict__ arows, const T* __restrict__ cs, int n, int nc, const int* active,
    int* tlog) {
  const int col = blockIdx.y;
  if (tlog && blockIdx.x == 0 && threadIdx.x == 0) tlog[col] = active ? active[col] : 1;
  if (active && !active[col]) return;
  const int J = blockIdx.x * kThreads + threadIdx.x;
  if (J >= nc) return;
  const T* rk = r + (int64_t)col * n;
  T acc = T(0);
  const int m1 = aptr[J + 1];
  for (int m = aptr[J]; m < m1; ++m) acc += rk[arows[m]];
  rc[(int64_t)col * nc + J] = cs[J] * acc;
}

// x_i = beta x_i + w s_{J(i)} ec_{J(i)}  (x_i = w s ec when beta = 0)
template <typename T>
__global__ __launch_bounds__(kThreads) void k_csr_prolong(
    const T* __restrict__ ec, T* __restrict__ x, const int* __restrict__ agg,
    const T* __restrict__ fs, int n, int nc, T w, T beta, const int* active, int* tlog) {
  const int col = blockIdx.y;
  if (tlog && blockIdx.x == 0 && threadIdx.x == 0) tlog[col] = active ? active[col] : 1;
  if (active && !active[col]) return;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const T e = w * fs[i] * ec[(int64_t)col * nc + agg[i]];
  T* xk = x + (int64_t)col * n;
  xk[i] = (beta == T(0)) ? e : beta * xk[i] + e;
}

// row i of the left half of the n x 2n augmented matrix: A's row
__global__ __launch_bounds__(kThreads) void k_csr_dense(const int* __restrict__ rp,
                                                        const int* __restrict__ ci,
                                                        const double* __restrict__ v, int n,
                                                        double* __restrict__ aug) {
  const int i = blockIdx.x;
  double* row = aug + (int64_t)i * 2 * n;
  for (int c = threadIdx.x; c < n; c += kThreads) row[c] = 0.0;
  __syncthreads();
  for (int e = rp[i] + threadIdx.x; e < rp[i + 1]; e += kThreads) row[ci[e]] = v[e];
}

}  // namespace

int csr_blocks(int n) { return (n + kThreads - 1) / kThreads; }

static dim3 csr_grid(int rows, int nb, int cols) {
  return dim3((unsigned)((rows + kThreads - 1) / kThreads), (unsigned)((nb + cols - 1) / cols));
}

// Vectors per thread of the products: four share a row's indices and values where that
// leaves enough threads, from 2^19 rows x vectors on; below, one.  Measured with 1 / 2 /
// 4 / 8, 64 vectors: 230 / 151 / 127 / 122 us for 120,000 rows of a geometric graph, 67 /
// 57 / 53 / 51 for 255^2 rows, 32 / 29 / 29 / 30 for 127^2; 16 vectors of 3,000 rows: 21.8
// / 22.3 / 24.2 / 27.8.  The aggregate sums share nothing between vectors and take one
// (120,000 rows, 64 vectors: 78 / 106 / 114 / 125).
template <typename F>
static void csr_cols(int rows, int nb, F&& f) {
  if ((int64_t)rows * nb >= 1 << 19)
    f(std::integral_constant<int, 4>());
  else
    f(std::integral_constant<int, 1>());
}

void csr_residual(const double* b, const double* x, double* r, const CsrMat<double>& A, int nb,
                  const int* active, c64* partials, hipStream_t s) {
  if (A.n == 0) return;
  csr_cols(A.n, nb, [&](auto c) {
    constexpr int C = decltype(c)::value;
    MLMC_LAUNCH((k_csr_residual<double, C>), csr_grid(A.n, nb, C), dim3(kThreads), 0, s, b, x, r,
                A.sptr, A.sci, A.sv, A.n, nb, active, partials, timing_log());
  });
}

void csr_restrict(const double* x, double* xc, const CsrAgg<double>& G, int n, int nb,
                  const int* active, hipStream_t s) {
  if (G.nc == 0) return;
  MLMC_LAUNCH(k_csr_agg_sum<double>, csr_grid(G.nc, nb, 1), dim3(kThreads), 0, s, x, xc, G.aptr,
              G.arows, G.cs, n, G.nc, active, timing_log());
}

void csr_prolong(const double* ec, double* x, const CsrAgg<double>& G, int n, double omega,
                 double beta, int nb, const int* active, hipStream_t s) {
  if (n == 0) return;
  MLMC_LAUNCH(k_csr_prolong<double>, dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)nb),
              dim3(kThreads), 0, s, ec, x, G.agg, G.fs, n, G.nc, omega, beta, active,
              timing_log());
}

void csr_spmm(const double* x, double* y, const CsrMat<double>& M, double w, double beta, int nb,
              const int* active, hipStream_t s) {
  if (M.n == 0) return;
  csr_cols(M.n, nb, [&](auto c) {
    constexpr int C = decltype(c)::value;
    MLMC_LAUNCH((k_csr_spmm<double, C>), csr_grid(M.n, nb, C), dim3(kThreads), 0, s, x, y, M.sptr,
                M.sci, M.sv, M.n, M.ncol, w, beta, nb, active, timing_log());
  });
}

void csr_dense(const CsrMat<double>& A, double* aug, hipStream_t s) {
  if (A.n == 0) return;
  MLMC_LAUNCH(k_csr_dense, dim3((unsigned)A.n), dim3(kThreads), 0, s, A.rp, A.ci, A.v, A.n, aug);
}

}  // namespace mlmc
