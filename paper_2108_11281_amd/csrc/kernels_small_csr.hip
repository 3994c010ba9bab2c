// Small levels of a matrix-given hierarchy: the whole V-cycle below a level, one
// vector per workgroup.
//
// A multicolour sweep is a chain of dependent colour classes.  On levels of some
// ten thousand rows and fewer every class is a launch of 3-5 us whatever it holds
// (a random geometric graph has about 16 classes, so four sweeps are some 64
// launches per level and V-cycle).  A workgroup keeps one vector's iterate in LDS
// and runs the classes with its own barrier between them, the gathers going to LDS.
// Bound by what one compute unit loads and gathers, about 0.2 us per 1000 entries
// (fetching each slice's entries one slice ahead changed nothing on scattered graphs
// and cost 25% on regular ones: 45 -> 60 ms for the trace of a 511^2 bilinear
// hierarchy); on the smallest levels by the chain of a class (about 0.5 us).
//
// The unknowns of these levels are numbered by position in the sweep's order
// (classes padded to whole slices of 64), so that right-hand side, diagonal and
// matrix (SELL-64, 16-bit columns) are all read in order; padding positions hold
// zeros throughout.  The first level's right-hand side and result are the solver's
// interleaved blocks in natural order.
#include "kernels.h"
#include "vec_body.h"

namespace mlmc {
namespace {

constexpr int kWaves = 16, kNT = kWaves * 64;

// wave-uniform reads of arrays that no kernel writes: scalar loads
__device__ __forceinline__ int uniform_at(const int* p, int i) {
  typedef const __attribute__((address_space(4))) int* constant_ptr;
  return ((constant_ptr)(uintptr_t)p)[i];
}

template <typename T, int U>
__device__ __forceinline__ void sell_step(const unsigned short* __restrict__ ci,
                                          const T* __restrict__ v, int at, const T* xs, T& acc) {
  int j[U];
  T a[U], g[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    j[u] = ci[at + u * 64];
    a[u] = v[at + u * 64];
  }
#pragma unroll
  for (int u = 0; u < U; ++u) g[u] = xs[j[u]];
#pragma unroll
  for (int u = 0; u < U; ++u) acc += a[u] * g[u];
}

// sum of a SELL-64 row against xs (LDS or global), in entry order
template <typename T>
__device__ __forceinline__ T sell_sum(const SellView<T>& M, int sl, int lane, const T* xs) {
  const int p0 = uniform_at(M.ptr, sl), w = (uniform_at(M.ptr, sl + 1) - p0) >> 6;
  int at = p0 + lane, e = 0;
  T acc = T(0);
  for (; e + 8 <= w; e += 8, at += 512) sell_step<T, 8>(M.ci, M.v, at, xs, acc);
  if (e + 4 <= w) {
    sell_step<T, 4>(M.ci, M.v, at, xs, acc);
    e += 4;
    at += 256;
  }
  if (e + 2 <= w) {
    sell_step<T, 2>(M.ci, M.v, at, xs, acc);
    e += 2;
    at += 128;
  }
  if (e < w) sell_step<T, 1>(M.ci, M.v, at, xs, acc);
  return acc;
}

// a rounded product, not contracted with a sum
template <typename T>
__device__ __forceinline__ T product(T a, T b) {
#pragma clang fp contract(off)
  return a * b;
}
__device__ __forceinline__ float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

// the same with the diagonal d xk in its place before entry dp: the order of the full
// row, so that the sum is that of the residual on levels with a launch per operation
template <typename T>
__device__ __forceinline__ T sell_sum_diag(const SellView<T>& M, int sl, int lane, const T* xs,
                                           int dp, T d, T xk) {
  const int p0 = uniform_at(M.ptr, sl), w = (uniform_at(M.ptr, sl + 1) - p0) >> 6;
  int at = p0 + lane;
  T acc = T(0);
  for (int e = 0; e < w; e += 4, at += 256) {
    int j[4];
    T a[4], g[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      j[u] = e + u < w ? M.ci[at + u * 64] : 0;
      a[u] = e + u < w ? M.v[at + u * 64] : T(0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = xs[j[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (e + u == dp) acc = fused(d, xk, acc);  // a product added under a condition is
                                                 // not contracted
      if (e + u < w) acc += a[u] * g[u];
    }
  }
  if (dp >= ((w + 3) & ~3)) acc = fused(d, xk, acc);  // not met in the loop
  return acc;
}

template <typename T>
__device__ __forceinline__ void sweep(const SmallCsrLevel<T>& L, T* xs, const T* b, bool reverse,
                                      int wave, int lane) {
  for (int q = 0; q < L.ncls; ++q) {
    const int c = reverse ? L.ncls - 1 - q : q;
    const int s1 = uniform_at(L.cls, c + 1);
    for (int sl = uniform_at(L.cls, c) + wave; sl < s1; sl += kWaves) {
      const int k = sl * 64 + lane;
      const T bk = b[k], d = L.di[k];
      const T sum = sell_sum(L.off, sl, lane, xs);
      xs[k] = (bk - sum) * d;
    }
    __syncthreads();
  }
}

template <typename T>
__global__ __launch_bounds__(kNT) void k_small_csr(const SmallCsrLevel<T>* __restrict__ lev,
                                                   int nl, SmallCsrCoarse<T> cs, const T* bin,
                                                   T* xout, int W, int pre, int post, T omega,
                                                   int mode, const int* active, int* tlog) {
  extern __shared__ __align__(16) char small_csr_lds[];
  T* xs = reinterpret_cast<T*>(small_csr_lds);
  const int col = blockIdx.x;
  if (tlog && threadIdx.x == 0) tlog[col] = active ? active[col] : 1;
  if (active && !active[col]) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (mode != kSmallCsrUp) {
    for (int l = 0; l < nl; ++l) {
      const SmallCsrLevel<T> L = lev[l];
      T* b = L.b + (int64_t)col * L.np;
      T* r = L.r + (int64_t)col * L.np;
      for (int k = tid; k < L.np; k += kNT) {
        if (l == 0) {  // gather the interleaved right-hand side
          const int row = L.row[k];
          b[k] = row >= 0 ? bin[(int64_t)row * W + col] : T(0);
        }
        xs[k] = T(0);
      }
      __syncthreads();
      for (int s = 0; s < pre; ++s) sweep(L, xs, b, false, wave, lane);
      // r = b - A x, kept for the restriction; x kept for the way up
      T* x = L.x + (int64_t)col * L.np;
      for (int sl = wave; sl < (L.np >> 6); sl += kWaves) {
        const int k = sl * 64 + lane;
        const T xk = xs[k];
        r[k] = b[k] - sell_sum_diag(L.off, sl, lane, xs, L.dp[k], L.dd[k], xk);
        x[k] = xk;
      }
      __syncthreads();
      const bool last = l + 1 == nl;
      const int nc = last ? cs.n : lev[l + 1].np;
      T* bc = last ? cs.b + (int64_t)col * cs.n : lev[l + 1].b + (int64_t)col * nc;
      if (L.mptr) {
        for (int J = tid; J < nc; J += kNT) {
          T acc = T(0);
          const int m1 = L.mptr[J + 1];
          for (int m = L.mptr[J]; m < m1; ++m) acc += r[L.mem[m]];
          bc[J] = L.cs[J] * acc;
        }
      } else {
        for (int sl = wave; sl < (nc + 63) >> 6; sl += kWaves) {
          const T acc = sell_sum(L.R, sl, lane, (const T*)r);
          if (sl * 64 + lane < nc) bc[sl * 64 + lane] = acc;
        }
      }
      __syncthreads();
    }
  }
  if (mode == kSmallCsrAll) {  // coarsest solve, the sums of the solver's own product
    for (int bx = 0; bx < (cs.ld >> 4); ++bx) {
      body::dense_apply_mfma<T, kWaves>(cs.inv, cs.b + (int64_t)col * cs.n,
                                        cs.x + (int64_t)col * cs.n, cs.n, cs.ld, 1, nullptr, bx, 0,
                                        true, xs, tid);
      __syncthreads();
    }
  }
  if (mode != kSmallCsrDown) {
    for (int l = nl - 1; l >= 0; --l) {
      const SmallCsrLevel<T> L = lev[l];
      const T* b = L.b + (int64_t)col * L.np;
      T* x = L.x + (int64_t)col * L.np;
      const bool last = l + 1 == nl;
      const T* ec = last ? cs.x + (int64_t)col * cs.n
                         : lev[l + 1].x + (int64_t)col * lev[l + 1].np;
      if (L.mptr) {
        for (int k = tid; k < L.np; k += kNT)
          xs[k] = x[k] + product(omega * L.fs[k], ec[L.agg[k]]);
      } else {
        for (int sl = wave; sl < (L.np >> 6); sl += kWaves) {
          const int k = sl * 64 + lane;
          xs[k] = x[k] + omega * sell_sum(L.P, sl, lane, ec);
        }
      }
      __syncthreads();
      for (int s = 0; s < post; ++s) sweep(L, xs, b, true, wave, lane);
      for (int k = tid; k < L.np; k += kNT) {
        if (l == 0) {
          const int row = L.row[k];
          if (row >= 0) xout[(int64_t)row * W + col] = xs[k];
        } else {
          x[k] = xs[k];
        }
      }
      __syncthreads();
    }
  }
}

// `sweeps` sweeps of one level (xin nullptr: from zero), for the visits to a small level
// that need its iterate in between (two coarse-grid cycles below it, sweeps asked for by
// themselves), in place of a launch per class: 3000 rows of a geometric graph, 64 FP32
// vectors, a call of four sweeps 200 -> 73 us, a solve with two cycles 7.2 -> 4.3 ms.
template <typename T, typename U>
__global__ __launch_bounds__(kNT) void k_small_csr_sweeps(const SmallCsrLevel<T>* __restrict__ lev,
                                                          const U* bin, const U* xin, U* xout,
                                                          int64_t row_stride, int64_t col_stride,
                                                          int sweeps, int reverse,
                                                          const int* active, int* tlog) {
  extern __shared__ __align__(16) char small_csr_lds[];
  T* xs = reinterpret_cast<T*>(small_csr_lds);
  const int col = blockIdx.x;
  if (tlog && threadIdx.x == 0) tlog[col] = active ? active[col] : 1;
  if (active && !active[col]) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const SmallCsrLevel<T> L = *lev;
  T* b = L.b + (int64_t)col * L.np;
  for (int k = tid; k < L.np; k += kNT) {
    const int row = L.row[k];
    const int64_t at = row * row_stride + col * col_stride;
    b[k] = row >= 0 ? (T)bin[at] : T(0);
    xs[k] = row >= 0 && xin ? (T)xin[at] : T(0);
  }
  __syncthreads();
  for (int s = 0; s < sweeps; ++s) sweep(L, xs, b, reverse != 0, wave, lane);
  for (int k = tid; k < L.np; k += kNT) {
    const int row = L.row[k];
    if (row >= 0) xout[row * row_stride + col * col_stride] = (U)xs[k];
  }
}

}  // namespace

template <typename T>
size_t small_csr_lds(int np_max, bool dense) {
  const int parts = body::kDenseParts * 4 * 64;
  return sizeof(T) * (size_t)(dense && np_max < parts ? parts : np_max);
}

void small_csr_setup() {
  MLMC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_csr<float>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSmallCsrLds));
  MLMC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_csr<double>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSmallCsrLds));
  MLMC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_csr_sweeps<float, float>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSmallCsrLds));
  MLMC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_csr_sweeps<float, double>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSmallCsrLds));
  MLMC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(k_small_csr_sweeps<double, double>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSmallCsrLds));
}

template <typename T, typename U>
void small_csr_sweeps(const SmallCsrLevel<T>* lev, int np, const U* b, const U* xin, U* x, int W,
                      int64_t row_stride, int64_t col_stride, int sweeps, bool reverse,
                      const int* active, hipStream_t s) {
  MLMC_LAUNCH((k_small_csr_sweeps<T, U>), dim3(W), dim3(kNT), small_csr_lds<T>(np, false), s, lev,
              b, xin, x, row_stride, col_stride, sweeps, reverse ? 1 : 0, active, timing_log());
}

template <typename T>
void small_csr(const SmallCsrLevel<T>* lev, int nl, int np_max, const SmallCsrCoarse<T>& cs,
               const T* b, T* x, int W, int pre, int post, double omega, int mode,
               const int* active, hipStream_t s) {
  MLMC_LAUNCH(k_small_csr<T>, dim3(W), dim3(kNT),
              small_csr_lds<T>(np_max, mode == kSmallCsrAll), s, lev, nl, cs, b, x, W,
              pre, post, (T)omega, mode, active, timing_log());
}

#define SMALL_SWEEPS_INST(T, U)                                                                 \
  template void small_csr_sweeps<T, U>(const SmallCsrLevel<T>*, int, const U*, const U*, U*, int, \
                                       int64_t, int64_t, int, bool, const int*, hipStream_t);
SMALL_SWEEPS_INST(float, float)
SMALL_SWEEPS_INST(float, double)
SMALL_SWEEPS_INST(double, double)
template void small_csr<float>(const SmallCsrLevel<float>*, int, int, const SmallCsrCoarse<float>&,
                               const float*, float*, int, int, int, double, int, const int*,
                               hipStream_t);
template void small_csr<double>(const SmallCsrLevel<double>*, int, int,
                                const SmallCsrCoarse<double>&, const double*, double*, int, int,
                                int, double, int, const int*, hipStream_t);

}  // namespace mlmc
