// Sparse operators given as a matrix: the kernels of the solver (Gauss-Seidel
// sweeps, residual, CG updates, transfers, coarsest solve) on interleaved blocks
// of W vectors, element i of vector c at [i W + c].
//
// On RHS-major blocks a wave gathers 64 scattered 4-byte entries of one vector per
// matrix entry: one cache line each, and the address unit, not the memory, sets the
// rate.  Interleaved, the W values that a matrix entry multiplies lie next to each
// other, so a gather is one contiguous read of 4 W bytes and the row's index and
// value are the same for the lanes that share the row.  G lanes (the power of two
// from 8 to 64 that holds W; two vectors per lane above 64) take a row; with G = 64
// the row is wave-uniform and its indices and values are scalar loads.  A solve
// converts its right-hand sides once and its solutions back once.  Trace of a
// 262,144-vertex geometric graph, a launch per class everywhere: 264 -> 179 ms; a
// class now costs 3.5-5 us for narrow batches, most of it launch and load latency.
//
// Row sums run in the stored column order.  Indices are 32-bit (n, nnz < 2^31).
#include <algorithm>

#include "kernels.h"
#include "vec_body.h"

namespace mlmc {
namespace {

template <typename T, int V>
struct alignas(V * sizeof(T)) Pack {
  T v[V];
};

// the vectors of a lane: c .. c + V - 1 of row i at x[i W + c]; lanes beyond W read
// vector 0 and write nothing
template <int G, int V>
struct Lane {
  int c;
  bool on[V], live;  // live: some vector of the wave is active
  __device__ Lane(int W, const int* active) {
    const int c0 = ((int)blockIdx.y * G + ((int)threadIdx.x & (G - 1))) * V;
    c = c0 < W ? c0 : 0;
    bool any = false;
#pragma unroll
    for (int v = 0; v < V; ++v) {
      on[v] = c0 < W && (!active || active[c0 + v]);
      any = any || on[v];
    }
    live = __any(any);
  }
  template <typename T>
  __device__ void store(T* p, int64_t at, const T (&val)[V]) const {
    if (V == 2 && on[0] && on[V - 1]) {
      Pack<T, V> o;
#pragma unroll
      for (int v = 0; v < V; ++v) o.v[v] = val[v];
      *reinterpret_cast<Pack<T, V>*>(p + at) = o;
      return;
    }
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (on[v]) p[at + v] = val[v];
  }
};

template <typename T, int V>
__device__ __forceinline__ Pack<T, V> ldv(const T* p, int64_t at) {
  return *reinterpret_cast<const Pack<T, V>*>(p + at);
}

template <int G>
__device__ __forceinline__ int group_of(int tid) {
  return G == 64 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid / G;
}

// U entries: indices and values first, then the gathers, then the sums in order
template <typename T, int V, int U, typename F>
__device__ __forceinline__ void entries(const int* __restrict__ ci, const T* __restrict__ a, int e,
                                        T (&acc)[V], F&& gather) {
  int j[U];
  T w[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    j[u] = ci[e + u];
    w[u] = a[e + u];
  }
  Pack<T, V> g[U];
#pragma unroll
  for (int u = 0; u < U; ++u) g[u] = gather(j[u]);
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] += w[u] * g[u].v[v];
}
template <typename T, int V, typename F>
__device__ __forceinline__ void row_sum(const int* __restrict__ ci, const T* __restrict__ a,
                                        int beg, int end, T (&acc)[V], F&& gather) {
  int e = beg;
  for (; e + 8 <= end; e += 8) entries<T, V, 8>(ci, a, e, acc, gather);
  if (e + 4 <= end) {
    entries<T, V, 4>(ci, a, e, acc, gather);
    e += 4;
  }
  if (e + 2 <= end) {
    entries<T, V, 2>(ci, a, e, acc, gather);
    e += 2;
  }
  if (e < end) entries<T, V, 1>(ci, a, e, acc, gather);
}

// partials[(c + v) nblk + blk] = the block's sum of acc over its row groups
template <int G, int V>
__device__ __forceinline__ void block_columns(double (&acc)[V], int W, const Lane<G, V>& ln,
                                              c64* partials) {
  __shared__ double lds[kThreads / 64][64 * V];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int v = 0; v < V; ++v) {
#pragma unroll
    for (int off = G; off < 64; off <<= 1) acc[v] += __shfl_xor(acc[v], off, 64);
    lds[wave][lane * V + v] = acc[v];
  }
  __syncthreads();
  if ((int)threadIdx.x < G) {
#pragma unroll
    for (int v = 0; v < V; ++v) {
      double s = lds[0][lane * V + v];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) s += lds[w][lane * V + v];
      if (ln.on[v]) partials[(int64_t)(ln.c + v) * gridDim.x + blockIdx.x] = {s, 0.0};
    }
  }
}

template <int G, int V>
__device__ __forceinline__ void log_columns(int* tlog, const Lane<G, V>& ln, int W) {
  if (tlog && blockIdx.x == 0 && (int)threadIdx.x < G) {
    const int c0 = ((int)blockIdx.y * G + (int)threadIdx.x) * V;
#pragma unroll
    for (int v = 0; v < V; ++v)
      if (c0 < W) tlog[c0 + v] = ln.on[v] ? 1 : 0;
  }
}

// x_i = (b_i - sum_{j != i} a_ij x_j) / a_ii of the row at position k
template <typename T, int G, int V>
__device__ __forceinline__ void gs_row(const T* b, T* x, const int4* __restrict__ rows,
                                       const int* __restrict__ ci, const T* __restrict__ a,
                                       const T* __restrict__ di, int k, int W,
                                       const Lane<G, V>& ln) {
  const int4 r = rows[k];
  const T d = di[k];
  const int64_t at = (int64_t)r.x * W + ln.c;
  const Pack<T, V> bv = ldv<T, V>(b, at);
  T sum[V], out[V];
#pragma unroll
  for (int v = 0; v < V; ++v) sum[v] = T(0);
  row_sum<T, V>(ci, a, r.y, r.z, sum, [&](int j) { return ldv<T, V>(x, (int64_t)j * W + ln.c); });
#pragma unroll
  for (int v = 0; v < V; ++v) out[v] = (bv.v[v] - sum[v]) * d;
  ln.store(x, at, out);
}

// one colour class (positions k0 .. k1 - 1) of a sweep, in place
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_gs(const T* b, T* x,
                                                      const int4* __restrict__ rows,
                                                      const int* __restrict__ ci,
                                                      const T* __restrict__ a,
                                                      const T* __restrict__ di, int k0, int k1,
                                                      int W, const int* active, int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const int k = k0 + blockIdx.x * (kThreads / G) + group_of<G>(threadIdx.x);
  if (k >= k1 || !ln.live) return;
  gs_row<T, G, V>(b, x, rows, ci, a, di, k, W, ln);
}

// Several consecutive colour classes of a sweep in one launch (the small classes
// that a greedy colouring leaves at its end): a workgroup per vector runs the
// classes one after another, a row per lane; the rows of a class are independent, so
// only the class boundaries need its barrier (which also orders its waves' stores
// before the next class's loads).  Bound by the chain of rounds, so rows in flight
// count for more than wide gathers: the sweep of 20,000 rows of a geometric graph with
// 5 of its 13 classes here, 8 / 16 / 64 FP32 vectors, takes 49 / 50 / 48 us (53 / 54 /
// 48 with a launch per class); with the rows' lanes of the other launches it took 51 /
// 55 / 61.
template <typename T>
__global__ __launch_bounds__(kTailWaves * 64) void k_rows_gs_tail(
    const T* b, T* x, const int4* __restrict__ rows, const int* __restrict__ ci,
    const T* __restrict__ a, const T* __restrict__ di, CsrTail t, int W, const int* active,
    int* tlog) {
  const Lane<1, 1> ln(W, active);
  log_columns(tlog, ln, W);
  if (!ln.live) return;  // the whole workgroup: one vector
  for (int q = 0; q < t.count; ++q) {
    const int cc = t.reverse ? t.count - 1 - q : q;
    for (int k = t.off[cc] + (int)threadIdx.x; k < t.off[cc + 1]; k += kTailWaves * 64)
      gs_row<T, 1, 1>(b, x, rows, ci, a, di, k, W, ln);
    __syncthreads();
  }
}

// the rows of a block: [beg, end) of n, strided by the block's row groups
struct Rows {
  int beg, end;
  __device__ Rows(int n, int rpb, bool live) {
    beg = blockIdx.x * rpb;
    end = beg + rpb < n ? beg + rpb : n;
    if (!live) end = beg;
  }
};

// r = b - A x ; partials (nullable) of |r|^2
template <typename T, typename Tr, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_residual(
    const T* __restrict__ b, const T* __restrict__ x, Tr* __restrict__ r,
    const int* __restrict__ rp, const int* __restrict__ ci, const T* __restrict__ a, int n, int rpb,
    int W, const int* active, c64* partials, int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const Rows rows(n, rpb, ln.live);
  double acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0.0;
  for (int i = rows.beg + group_of<G>(threadIdx.x); i < rows.end; i += kThreads / G) {
    const int64_t at = (int64_t)i * W + ln.c;
    const Pack<T, V> bv = ldv<T, V>(b, at);
    T sum[V];
    Tr out[V];
#pragma unroll
    for (int v = 0; v < V; ++v) sum[v] = T(0);
    row_sum<T, V>(ci, a, rp[i], rp[i + 1], sum,
                  [&](int j) { return ldv<T, V>(x, (int64_t)j * W + ln.c); });
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const T val = bv.v[v] - sum[v];
      out[v] = convert<Tr, T>(val);
      acc[v] += (double)val * val;
    }
    ln.store(r, at, out);
  }
  if (partials) block_columns<G, V>(acc, W, ln, partials);
}

// p_new = z + beta p_old ; q = A p_new ; partials of p_new^T q.  The neighbours'
// p_new values are formed again from z and p_old, so one pass serves both.
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_update_apply(
    const T* __restrict__ p_old, const T* __restrict__ z, const c64* __restrict__ beta,
    T* __restrict__ p_new, T* __restrict__ q, const int* __restrict__ rp,
    const int* __restrict__ ci, const T* __restrict__ a, int n, int rpb, int W, const int* active,
    c64* partials, int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const Rows rows(n, rpb, ln.live);
  double acc[V];
  T bt[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    acc[v] = 0.0;
    bt[v] = (T)beta[ln.c + v].re;
  }
  auto dir = [&](int64_t at) {
    const Pack<T, V> zz = ldv<T, V>(z, at), pp = ldv<T, V>(p_old, at);
    Pack<T, V> o;
#pragma unroll
    for (int v = 0; v < V; ++v) o.v[v] = zz.v[v] + bt[v] * pp.v[v];
    return o;
  };
  for (int i = rows.beg + group_of<G>(threadIdx.x); i < rows.end; i += kThreads / G) {
    const int64_t at = (int64_t)i * W + ln.c;
    T sum[V], pi[V];
#pragma unroll
    for (int v = 0; v < V; ++v) sum[v] = T(0);
    row_sum<T, V>(ci, a, rp[i], rp[i + 1], sum,
                  [&](int j) { return dir((int64_t)j * W + ln.c); });
    const Pack<T, V> own = dir(at);
#pragma unroll
    for (int v = 0; v < V; ++v) {
      pi[v] = own.v[v];
      acc[v] += (double)pi[v] * sum[v];
    }
    ln.store(p_new, at, pi);
    ln.store(q, at, sum);
  }
  block_columns<G, V>(acc, W, ln, partials);
}

// y = beta y + w M x, M rectangular (m rows)
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_spmm(const T* __restrict__ x, T* __restrict__ y,
                                                        const int* __restrict__ rp,
                                                        const int* __restrict__ ci,
                                                        const T* __restrict__ a, int m, T w,
                                                        T beta, int W, const int* active,
                                                        int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const int i = blockIdx.x * (kThreads / G) + group_of<G>(threadIdx.x);
  if (i >= m || !ln.live) return;
  const int64_t at = (int64_t)i * W + ln.c;
  T sum[V], out[V];
#pragma unroll
  for (int v = 0; v < V; ++v) sum[v] = T(0);
  row_sum<T, V>(ci, a, rp[i], rp[i + 1], sum,
                [&](int j) { return ldv<T, V>(x, (int64_t)j * W + ln.c); });
  Pack<T, V> old = {};
  if (beta != T(0)) old = ldv<T, V>(y, at);
#pragma unroll
  for (int v = 0; v < V; ++v)
    out[v] = beta == T(0) ? w * sum[v] : beta * old.v[v] + w * sum[v];
  ln.store(y, at, out);
}

// rc_J = s_J sum_{i in J} r_i, members in ascending order
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_agg_sum(const T* __restrict__ r,
                                                           T* __restrict__ rc,
                                                           const int* __restrict__ aptr,
                                                           const int* __restrict__ arows,
                                                           const T* __restrict__ cs, int nc, int W,
                                                           const int* active, int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const int J = blockIdx.x * (kThreads / G) + group_of<G>(threadIdx.x);
  if (J >= nc || !ln.live) return;
  T acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = T(0);
  const int end = aptr[J + 1];
  int m = aptr[J];
  for (; m + 4 <= end; m += 4) {
    Pack<T, V> g[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) g[u] = ldv<T, V>(r, (int64_t)arows[m + u] * W + ln.c);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int v = 0; v < V; ++v) acc[v] += g[u].v[v];
  }
  for (; m < end; ++m) {
    const Pack<T, V> g = ldv<T, V>(r, (int64_t)arows[m] * W + ln.c);
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] += g.v[v];
  }
  const T sj = cs[J];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = sj * acc[v];
  ln.store(rc, (int64_t)J * W + ln.c, acc);
}

// a rounded product, not contracted with a sum: the prolongation of every form rounds
// the correction before adding it
template <typename T>
__device__ __forceinline__ T product(T a, T b) {
#pragma clang fp contract(off)
  return a * b;
}

// x_i = beta x_i + w s_{J(i)} ec_{J(i)}  (x_i = w s ec when beta = 0)
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_prolong(const T* __restrict__ ec,
                                                           T* __restrict__ x,
                                                           const int* __restrict__ agg,
                                                           const T* __restrict__ fs, int n, T w,
                                                           T beta, int W, const int* active,
                                                           int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const int i = blockIdx.x * (kThreads / G) + group_of<G>(threadIdx.x);
  if (i >= n || !ln.live) return;
  const int64_t at = (int64_t)i * W + ln.c;
  const Pack<T, V> e = ldv<T, V>(ec, (int64_t)agg[i] * W + ln.c);
  const T s = w * fs[i];
  Pack<T, V> old = {};
  if (beta != T(0)) old = ldv<T, V>(x, at);
  T out[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const T c = product(s, e.v[v]);
    out[v] = beta == T(0) ? c : beta * old.v[v] + c;
  }
  ln.store(x, at, out);
}

// partials of x^T y
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_dot(const T* __restrict__ x,
                                                       const T* __restrict__ y, int n, int rpb,
                                                       int W, const int* active, c64* partials) {
  const Lane<G, V> ln(W, active);
  const Rows rows(n, rpb, ln.live);
  double acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = 0.0;
#pragma unroll 4
  for (int i = rows.beg + group_of<G>(threadIdx.x); i < rows.end; i += kThreads / G) {
    const int64_t at = (int64_t)i * W + ln.c;
    const Pack<T, V> a = ldv<T, V>(x, at), b = ldv<T, V>(y, at);
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] += (double)a.v[v] * b.v[v];
  }
  block_columns<G, V>(acc, W, ln, partials);
}

// x += alpha p ; r -= alpha q ; partials of |r|^2 (x_zero: x taken as zero, not read)
template <typename T, int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_xr(T* __restrict__ x, T* __restrict__ r,
                                                      const T* __restrict__ p,
                                                      const T* __restrict__ q, const c64* alpha,
                                                      int n, int rpb, int W, const int* active,
                                                      c64* partials, int x_zero, int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const Rows rows(n, rpb, ln.live);
  double acc[V];
  T al[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    acc[v] = 0.0;
    al[v] = (T)alpha[ln.c + v].re;
  }
#pragma unroll 2
  for (int i = rows.beg + group_of<G>(threadIdx.x); i < rows.end; i += kThreads / G) {
    const int64_t at = (int64_t)i * W + ln.c;
    Pack<T, V> xv = {};
    if (!x_zero) xv = ldv<T, V>(x, at);
    const Pack<T, V> rv = ldv<T, V>(r, at), pv = ldv<T, V>(p, at), qv = ldv<T, V>(q, at);
    T xo[V], ro[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      xo[v] = xv.v[v] + al[v] * pv.v[v];
      ro[v] = rv.v[v] - al[v] * qv.v[v];
      acc[v] += (double)ro[v] * ro[v];
    }
    ln.store(x, at, xo);
    ln.store(r, at, ro);
  }
  block_columns<G, V>(acc, W, ln, partials);
}

// the FP64 refinement's fold: y += d, partials of b^T d, d = 0 (y_zero: y taken as
// zero, not read)
template <int G, int V>
__global__ __launch_bounds__(kThreads) void k_rows_fold(double* __restrict__ y,
                                                        float* __restrict__ d,
                                                        const double* __restrict__ b, int n,
                                                        int rpb, int W, const int* active,
                                                        c64* partials, int y_zero, int* tlog) {
  const Lane<G, V> ln(W, active);
  log_columns(tlog, ln, W);
  const Rows rows(n, rpb, ln.live);
  double acc[V];
  float zero[V];
#pragma unroll
  for (int v = 0; v < V; ++v) {
    acc[v] = 0.0;
    zero[v] = 0.f;
  }
#pragma unroll 2
  for (int i = rows.beg + group_of<G>(threadIdx.x); i < rows.end; i += kThreads / G) {
    const int64_t at = (int64_t)i * W + ln.c;
    Pack<double, V> yv = {};
    if (!y_zero) yv = ldv<double, V>(y, at);
    const Pack<float, V> dv = ldv<float, V>(d, at);
    const Pack<double, V> bv = ldv<double, V>(b, at);
    double yo[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      yo[v] = yv.v[v] + (double)dv.v[v];
      acc[v] += bv.v[v] * (double)dv.v[v];
    }
    ln.store(y, at, yo);
    ln.store(d, at, zero);
  }
  block_columns<G, V>(acc, W, ln, partials);
}

// Z = A^-1 B on interleaved blocks: the tile kernel of dense_apply with the
// right-hand sides of a reduction index next to each other (one 64-byte read per
// index and 16 columns); same ranges and sums.
template <typename T>
__global__ __launch_bounds__(body::kDenseParts * 64) void k_rows_dense(
    const T* __restrict__ Pk, const T* __restrict__ B, T* __restrict__ Z, int n, int ld, int W,
    const int* active) {
  using V4 = typename body::Vec4<T>::type;
  constexpr int P = body::kDenseParts;
  __shared__ T part[P * 4 * 64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  const int g = lane >> 4, c = lane & 15;
  const bool row_ok = m0 + c < W;
  const T* col = B + (row_ok ? m0 + c : 0);
  const int chunks = ld / 16;
  const int cbeg = wave * chunks / P, cend = (wave + 1) * chunks / P;
  typename body::Mfma<T>::acc_t acc = {0, 0, 0, 0};
  auto load = [&](int ch, T* av, T* bv) {
    const int j = ch * 16 + 4 * g;
    const V4 p = *reinterpret_cast<const V4*>(Pk + ((int64_t)(ch * 4 + g) * ld + i0 + c) * 4);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool ok = row_ok && j + s < n;
      const T q = col[ok ? (int64_t)(j + s) * W : 0];
      av[s] = ok ? q : (T)0;
      bv[s] = p[s];
    }
  };
  int ch = cbeg;
  for (; ch + 2 <= cend; ch += 2) {
    T av[2][4], bv[2][4];
#pragma unroll
    for (int u = 0; u < 2; ++u) load(ch + u, av[u], bv[u]);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s) acc = body::Mfma<T>::step(av[u][s], bv[u][s], acc);
  }
  for (; ch < cend; ++ch) {
    T av[4], bv[4];
    load(ch, av, bv);
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = body::Mfma<T>::step(av[s], bv[s], acc);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) part[(wave * 4 + r) * 64 + lane] = acc[r];
  __syncthreads();
  if (wave < 4) {
    const int r = wave;
    T v = part[r * 64 + lane];
#pragma unroll
    for (int p = 1; p < P; ++p) v = v + part[(p * 4 + r) * 64 + lane];
    const int k = m0 + body::Mfma<T>::row(g, r);
    if (k < W && (!active || active[k]) && i0 + c < n) Z[(int64_t)(i0 + c) * W + k] = v;
  }
}

// RHS-major block -> interleaved blocks in FP64 (dst, nullable) and in To (dst2,
// nullable), 64 rows x 32 vectors through LDS
template <typename To>
__global__ __launch_bounds__(kThreads) void k_rows_in(const double* __restrict__ src,
                                                      double* __restrict__ dst,
                                                      To* __restrict__ dst2, int64_t n, int W) {
  __shared__ double tile[32][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int c0 = blockIdx.y * 32;
  for (int t = threadIdx.x; t < 32 * 64; t += kThreads) {
    const int c = t >> 6, i = t & 63;
    if (c0 + c < W && i0 + i < n) tile[c][i] = src[(int64_t)(c0 + c) * n + i0 + i];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 32 * 64; t += kThreads) {
    const int c = t & 31, i = t >> 5;
    if (c0 + c < W && i0 + i < n) {
      const int64_t at = (i0 + i) * W + c0 + c;
      if (dst) dst[at] = tile[c][i];
      if (dst2) dst2[at] = (To)tile[c][i];
    }
  }
}

// interleaved block -> RHS-major FP64 block
template <typename Ts>
__global__ __launch_bounds__(kThreads) void k_rows_out(const Ts* __restrict__ src,
                                                       double* __restrict__ dst, int64_t n, int W) {
  __shared__ Ts tile[32][65];
  const int64_t i0 = (int64_t)blockIdx.x * 64;
  const int c0 = blockIdx.y * 32;
  for (int t = threadIdx.x; t < 32 * 64; t += kThreads) {
    const int c = t & 31, i = t >> 5;
    if (c0 + c < W && i0 + i < n) tile[c][i] = src[(i0 + i) * W + c0 + c];
  }
  __syncthreads();
  for (int t = threadIdx.x; t < 32 * 64; t += kThreads) {
    const int c = t >> 6, i = t & 63;
    if (c0 + c < W && i0 + i < n) dst[(int64_t)(c0 + c) * n + i0 + i] = (double)tile[c][i];
  }
}

// lanes per row and vectors per lane for blocks of W vectors
template <typename F>
void with_lanes(int W, F&& f) {
  using std::integral_constant;
  if (W <= 8)
    f(integral_constant<int, 8>(), integral_constant<int, 1>());
  else if (W <= 16)
    f(integral_constant<int, 16>(), integral_constant<int, 1>());
  else if (W <= 32)
    f(integral_constant<int, 32>(), integral_constant<int, 1>());
  else if (W <= 64 || (W & 1))  // an odd row stride leaves pairs of vectors unaligned
    f(integral_constant<int, 64>(), integral_constant<int, 1>());
  else
    f(integral_constant<int, 64>(), integral_constant<int, 2>());
}

template <int G, int V>
dim3 row_grid(int rows, int W) {
  return dim3((unsigned)((rows + kThreads / G - 1) / (kThreads / G)),
              (unsigned)((W + G * V - 1) / (G * V)));
}
template <int G, int V>
dim3 block_grid(int n, int W) {
  return dim3((unsigned)rows_blocks(n), (unsigned)((W + G * V - 1) / (G * V)));
}

}  // namespace

// at most 1024 partial sums per column, at least 32 rows per block
int rows_per_block(int n) { return std::max(32, ((n + 1023) / 1024 + 31) / 32 * 32); }
int rows_blocks(int n) { return (n + rows_per_block(n) - 1) / rows_per_block(n); }

#define ROWS_LAUNCH(...)                       \
  with_lanes(W, [&](auto g_, auto v_) {        \
    constexpr int G = decltype(g_)::value;     \
    constexpr int V = decltype(v_)::value;     \
    __VA_ARGS__;                               \
  })

template <typename T>
void rows_gs_sweep(const T* b, T* x, const CsrSweep<T>& S, int W, int tail_rows, const int* active,
                   bool reverse, hipStream_t s) {
  const int classes = (int)S.off.size() - 1;
  const int tail = csr_tail_start(S.off, tail_rows);
  auto one_class = [&](int c) {
    const int k0 = S.off[c], k1 = S.off[c + 1];
    if (k1 == k0) return;
    ROWS_LAUNCH(MLMC_LAUNCH((k_rows_gs<T, G, V>), (row_grid<G, V>(k1 - k0, W)), dim3(kThreads), 0,
                            s, b, x, S.rows, S.ci, S.v, S.di, k0, k1, W, active, timing_log()));
  };
  auto fused = [&](int c0, int c1) {  // classes [c0, c1), at most kMaxTailClasses
    CsrTail t;
    t.count = c1 - c0;
    t.reverse = reverse ? 1 : 0;
    for (int c = c0; c <= c1; ++c) t.off[c - c0] = S.off[c];
    MLMC_LAUNCH(k_rows_gs_tail<T>, dim3(1u, (unsigned)W), dim3(kTailWaves * 64), 0, s, b, x,
                S.rows, S.ci, S.v, S.di, t, W, active, timing_log());
  };
  if (!reverse) {
    for (int c = 0; c < tail; ++c) one_class(c);
    for (int c0 = tail; c0 < classes; c0 += kMaxTailClasses)
      fused(c0, std::min(classes, c0 + kMaxTailClasses));
  } else {
    for (int c1 = classes; c1 > tail; c1 -= kMaxTailClasses)
      fused(std::max(tail, c1 - kMaxTailClasses), c1);
    for (int c = tail - 1; c >= 0; --c) one_class(c);
  }
}

template <typename T, typename Tr>
void rows_residual(const T* b, const T* x, Tr* r, const CsrMat<T>& A, int W, const int* active,
                   c64* partials, hipStream_t s) {
  if (A.n == 0) return;
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_residual<T, Tr, G, V>), (block_grid<G, V>(A.n, W)),
                          dim3(kThreads), 0, s, b, x, r, A.rp, A.ci, A.v, A.n,
                          rows_per_block(A.n), W, active, partials, timing_log()));
}

template <typename T>
void rows_update_apply(const T* p_old, const T* z, const c64* beta, T* p_new, T* q,
                       const CsrMat<T>& A, int W, const int* active, c64* partials,
                       hipStream_t s) {
  if (A.n == 0) return;
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_update_apply<T, G, V>), (block_grid<G, V>(A.n, W)),
                          dim3(kThreads), 0, s, p_old, z, beta, p_new, q, A.rp, A.ci, A.v, A.n,
                          rows_per_block(A.n), W, active, partials, timing_log()));
}

template <typename T>
void rows_xr(T* x, T* r, const T* p, const T* q, const c64* alpha, int n, int W, const int* active,
             c64* partials, bool x_zero, hipStream_t s) {
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_xr<T, G, V>), (block_grid<G, V>(n, W)), dim3(kThreads), 0, s, x,
                          r, p, q, alpha, n, rows_per_block(n), W, active, partials,
                          x_zero ? 1 : 0, timing_log()));
}

template <typename T>
void rows_dot(const T* x, const T* y, int n, int W, const int* active, c64* partials,
              hipStream_t s) {
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_dot<T, G, V>), (block_grid<G, V>(n, W)), dim3(kThreads), 0, s, x,
                          y, n, rows_per_block(n), W, active, partials));
}

void rows_fold(double* y, float* d, const double* b, int n, int W, const int* active,
               c64* partials, bool y_zero, hipStream_t s) {
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_fold<G, V>), (block_grid<G, V>(n, W)), dim3(kThreads), 0, s, y,
                          d, b, n, rows_per_block(n), W, active, partials, y_zero ? 1 : 0,
                          timing_log()));
}

template <typename T>
void rows_spmm(const T* x, T* y, const CsrMat<T>& M, double w, double beta, int W,
               const int* active, hipStream_t s) {
  if (M.n == 0) return;
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_spmm<T, G, V>), (row_grid<G, V>(M.n, W)), dim3(kThreads), 0, s,
                          x, y, M.rp, M.ci, M.v, M.n, (T)w, (T)beta, W, active, timing_log()));
}

template <typename T>
void rows_agg_sum(const T* r, T* rc, const CsrAgg<T>& A, int W, const int* active, hipStream_t s) {
  if (A.nc == 0) return;
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_agg_sum<T, G, V>), (row_grid<G, V>(A.nc, W)), dim3(kThreads), 0,
                          s, r, rc, A.aptr, A.arows, A.cs, A.nc, W, active, timing_log()));
}

template <typename T>
void rows_prolong(const T* ec, T* x, const CsrAgg<T>& A, int n, double omega, double beta, int W,
                  const int* active, hipStream_t s) {
  if (n == 0) return;
  ROWS_LAUNCH(MLMC_LAUNCH((k_rows_prolong<T, G, V>), (row_grid<G, V>(n, W)), dim3(kThreads), 0, s,
                          ec, x, A.agg, A.fs, n, (T)omega, (T)beta, W, active, timing_log()));
}

template <typename T>
void rows_dense(const T* Pk, const T* B, T* Z, int n, int ld, int W, const int* active,
                hipStream_t s) {
  MLMC_LAUNCH(k_rows_dense<T>, dim3((unsigned)(ld / 16), (unsigned)((W + 15) / 16)),
              dim3(body::kDenseParts * 64), 0, s, Pk, B, Z, n, ld, W, active);
}

static dim3 convert_grid(int64_t n, int W) {
  return dim3((unsigned)((n + 63) / 64), (unsigned)((W + 31) / 32));
}
// one vector is the same in both layouts
template <typename To, typename Ts>
static void copy_one(const Ts* src, To* dst, int64_t n, hipStream_t s) {
  if constexpr (std::is_same<To, Ts>::value)
    vec_copy<To>(src, dst, n, 1, nullptr, s);
  else
    vec_convert<To, Ts>(src, dst, n, 1, nullptr, s);
}
template <typename To>
void rows_in(const double* src, double* dst, To* dst2, int64_t n, int W, hipStream_t s) {
  if (W == 1) {
    if (dst) copy_one<double, double>(src, dst, n, s);
    if (dst2) copy_one<To, double>(src, dst2, n, s);
    return;
  }
  MLMC_LAUNCH(k_rows_in<To>, convert_grid(n, W), dim3(kThreads), 0, s, src, dst, dst2, n, W);
}
template <typename Ts>
void rows_out(const Ts* src, double* dst, int64_t n, int W, hipStream_t s) {
  if (W == 1) return copy_one<double, Ts>(src, dst, n, s);
  MLMC_LAUNCH(k_rows_out<Ts>, convert_grid(n, W), dim3(kThreads), 0, s, src, dst, n, W);
}

#define ROWS_INST(T)                                                                            \
  template void rows_gs_sweep<T>(const T*, T*, const CsrSweep<T>&, int, int, const int*, bool,   \
                                 hipStream_t);                                                  \
  template void rows_residual<T, T>(const T*, const T*, T*, const CsrMat<T>&, int, const int*,   \
                                    c64*, hipStream_t);                                         \
  template void rows_update_apply<T>(const T*, const T*, const c64*, T*, T*, const CsrMat<T>&,   \
                                     int, const int*, c64*, hipStream_t);                       \
  template void rows_xr<T>(T*, T*, const T*, const T*, const c64*, int, int, const int*, c64*,   \
                           bool, hipStream_t);                                                  \
  template void rows_dot<T>(const T*, const T*, int, int, const int*, c64*, hipStream_t);       \
  template void rows_spmm<T>(const T*, T*, const CsrMat<T>&, double, double, int, const int*,    \
                             hipStream_t);                                                      \
  template void rows_agg_sum<T>(const T*, T*, const CsrAgg<T>&, int, const int*, hipStream_t);  \
  template void rows_prolong<T>(const T*, T*, const CsrAgg<T>&, int, double, double, int,        \
                                const int*, hipStream_t);                                       \
  template void rows_dense<T>(const T*, const T*, T*, int, int, int, const int*, hipStream_t);  \
  template void rows_in<T>(const double*, double*, T*, int64_t, int, hipStream_t);              \
  template void rows_out<T>(const T*, double*, int64_t, int, hipStream_t);
ROWS_INST(float)
ROWS_INST(double)
template void rows_residual<double, float>(const double*, const double*, float*,
                                           const CsrMat<double>&, int, const int*, c64*,
                                           hipStream_t);

}  // namespace mlmc
