// Batched flexible GMRES building blocks: columns iterate in lockstep, each
// with its own Hessenberg matrix, Givens rotations and residual estimate
// (FP64 scalars on the device; vectors in the working precision).
// Krylov vectors of one basis are stored consecutively: vector i of column k
// at base + i*vstride + k*n.
#include "kernels.h"
#include "vec_body.h"

namespace mlmc {
namespace {

constexpr int kMaxBasis = 33;  // restart length + 1

// the sums over a block of N values per thread, in the order of block_sum2; thread
// t < N receives value t
template <int N>
__device__ __forceinline__ double block_sums(double (&v)[N], double* lds) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double t = wave_sum(v[i]);
    if (lane == 0) lds[wave * N + i] = t;
  }
  __syncthreads();
  double sum = 0.0;
  if ((int)threadIdx.x < N) {
    for (int w = 0; w < kThreads / 64; ++w) sum += lds[w * N + threadIdx.x];
  }
  return sum;
}

// partials[((k*nv + i) * nblk) + b] = sum over block b of conj(V_i) w  (column k);
// blockIdx.z is a group of four vectors (register accumulators): w is re-read per
// group from cache.  The groups ran one after the other in a block before, each
// ending in four block sums: 8.8 us instead of 5.1 for 5 columns of 8192 unknowns.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_mdot(const T* __restrict__ V, int64_t vstride,
                                                   int nv, const T* __restrict__ w, int64_t n,
                                                   const int* active, c64* partials) {
  __shared__ double red[kThreads / 64 * 8];
  const int k = blockIdx.y, nblk = gridDim.x, i0 = 4 * blockIdx.z;
  if (active && !active[k]) return;
  const int64_t chunk = (n + nblk - 1) / nblk;
  const int64_t lo = (int64_t)blockIdx.x * chunk;
  const int64_t hi = lo + chunk < n ? lo + chunk : n;
  const T* wk = w + (int64_t)k * n;
  double sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  const int gcount = nv - i0 < 4 ? nv - i0 : 4;
  // two elements per step, their ten loads issued before the products, which
  // accumulate in element order as in a plain strided loop
  for (int64_t e0 = lo + threadIdx.x; e0 < hi; e0 += 2 * kThreads) {
    T we[2], ve[2][4];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int64_t e = e0 + (int64_t)q * kThreads;
      const int64_t ec = e < hi ? e : lo;
      we[q] = wk[ec];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        ve[q][u] = V[(i0 + (u < gcount ? u : 0)) * vstride + (int64_t)k * n + ec];
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (e0 + (int64_t)q * kThreads < hi) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if (u < gcount) cdot_acc(sum[2 * u], sum[2 * u + 1], ve[q][u], we[q]);
      }
    }
  }
  const double v = block_sums<8>(sum, red);
  const int t = threadIdx.x;
  if (t < 2 * gcount) {
    double* out = reinterpret_cast<double*>(partials + ((int64_t)k * nv + i0 + (t >> 1)) * nblk +
                                            blockIdx.x);
    out[t & 1] = v;
  }
}

// w -= sum_i h[k*nv + i] V_i, and partials of |w|^2 per block of kThreads EPT elements.
// hparts != nullptr: h is formed here from the nhp partials of each entry (eight lanes
// per entry), and block 0 stores it.  w may not be shared with the partials' readers:
// wparts is another region than hparts.
template <typename T, int EPT>
__global__ __launch_bounds__(kThreads) void k_maxpy(const T* __restrict__ V, int64_t vstride,
                                                    int nv, c64* h, const c64* hparts, int nhp,
                                                    T* __restrict__ w, int64_t n,
                                                    const int* active, c64* wparts) {
  __shared__ double hs[2 * kMaxBasis], red[kThreads / 64];
  const int k = blockIdx.y, t = threadIdx.x;
  if (active && !active[k]) return;
  const int64_t e0 = (int64_t)blockIdx.x * (kThreads * EPT) + t;
  T acc[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int64_t e = e0 + (int64_t)u * kThreads;
    acc[u] = e < n ? w[(int64_t)k * n + e] : zero_of(T());
  }
  if (hparts) {
    for (int i = t >> 3; i < nv; i += kThreads / 8) {
      const c64* p = hparts + ((int64_t)k * nv + i) * nhp;
      double re = 0.0, im = 0.0;
      for (int b = t & 7; b < nhp; b += 8) {
        re += p[b].re;
        im += p[b].im;
      }
#pragma unroll
      for (int m = 1; m < 8; m *= 2) {
        re += __shfl_xor(re, m, 64);
        im += __shfl_xor(im, m, 64);
      }
      if ((t & 7) == 0) {
        hs[2 * i] = re;
        hs[2 * i + 1] = im;
        if (blockIdx.x == 0) h[(int64_t)k * nv + i] = {re, im};
      }
    }
  } else if (t < nv) {
    const c64 c = h[(int64_t)k * nv + t];
    hs[2 * t] = c.re;
    hs[2 * t + 1] = c.im;
  }
  __syncthreads();
#pragma unroll 4
  for (int i = 0; i < nv; ++i) {
    const T* vk = V + i * vstride + (int64_t)k * n;
    T ve[EPT];
#pragma unroll
    for (int u = 0; u < EPT; ++u) {
      const int64_t e = e0 + (int64_t)u * kThreads;
      ve[u] = vk[e < n ? e : 0];
    }
#pragma unroll
    for (int u = 0; u < EPT; ++u) acc[u] -= scale_by(hs[2 * i], hs[2 * i + 1], ve[u]);
  }
  double sum[1] = {0.0}, unused = 0.0;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int64_t e = e0 + (int64_t)u * kThreads;
    if (e < n) {
      w[(int64_t)k * n + e] = acc[u];
      cdot_acc(sum[0], unused, acc[u], acc[u]);
    }
  }
  const double v = block_sums<1>(sum, red);
  if (t == 0) wparts[(int64_t)k * gridDim.x + blockIdx.x] = {v, 0.0};
}

// d = sum_{i < dims[k]} y[k*ldy + i] Z_i for columns with start[k]
template <typename T>
__global__ __launch_bounds__(kThreads) void k_combine(const T* __restrict__ Z, int64_t vstride,
                                                      const c64* __restrict__ y, int ldy,
                                                      const int* __restrict__ dims,
                                                      T* __restrict__ d, int64_t n,
                                                      const int* start) {
  const int k = blockIdx.y;
  if (!start[k]) return;
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= n) return;
  T acc = zero_of(T());
  const int m = dims[k];
#pragma unroll 4
  for (int i = 0; i < m; ++i) {
    const c64 c = y[(int64_t)k * ldy + i];
    acc += scale_by(c.re, c.im, Z[i * vstride + (int64_t)k * n + e]);
  }
  d[(int64_t)k * n + e] = acc;
}

// dst = src / |src|, |src|^2 the sum of column k's np partials, which every block forms
// and block 0 stores in nrm2 (dst may be src)
template <typename T, int EPT>
__global__ __launch_bounds__(kThreads) void k_scale_inv_norm(T* dst, const T* src,
                                                             const c64* parts, int np, c64* nrm2,
                                                             int64_t n, const int* active) {
  __shared__ double lds[16], total;
  const int k = blockIdx.y;
  if (active && !active[k]) return;
  const int64_t e0 = (int64_t)blockIdx.x * (kThreads * EPT) + threadIdx.x;
  T v[EPT];
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int64_t e = e0 + (int64_t)u * kThreads;
    v[u] = src[(int64_t)k * n + (e < n ? e : 0)];
  }
  const c64 f = body::finish(parts, np, k, lds);
  if (threadIdx.x == 0) {
    total = f.re;
    if (blockIdx.x == 0) nrm2[k] = f;
  }
  __syncthreads();
  const double s = total > 0.0 ? 1.0 / sqrt(total) : 0.0;
#pragma unroll
  for (int u = 0; u < EPT; ++u) {
    const int64_t e = e0 + (int64_t)u * kThreads;
    if (e < n) dst[(int64_t)k * n + e] = scale_by(s, 0.0, v[u]);
  }
}

struct GState {
  c64* H;     // [nb][m+1][m]  Hessenberg (rotated in place: upper triangle R)
  c64* cs;    // [nb][m]       rotation cosines (real part used)
  c64* sn;    // [nb][m]       rotation sines
  c64* g;     // [nb][m+1]     rotated right-hand side
  int* dims;  // [nb]          basis size used by the column
};

__global__ void k_givens_init(GState st, const c64* beta2, const int* active, int m, int nb) {
  const int k = blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nb) return;
  st.dims[k] = 0;
  for (int i = 0; i <= m; ++i) st.g[(int64_t)k * (m + 1) + i] = {0.0, 0.0};
  if (active[k]) st.g[(int64_t)k * (m + 1)] = {sqrt(beta2[k].re), 0.0};
}

// Column j of the Hessenberg matrix: h[k*(j+1) + i] (i <= j) and |w|^2 (h_{j+1,j}^2).
// Applies the previous rotations, forms the new one, updates g; columns whose
// residual estimate |g_{j+1}| <= tol * beta stop (active = 0, dims = j+1).
__global__ void k_givens_step(GState st, const c64* h, const c64* wn2, const c64* beta2,
                              double tol, int j, int m, int* active, int nb, int* count) {
  __shared__ int cnt;
  if (threadIdx.x == 0) cnt = 0;
  __syncthreads();
  for (int k = threadIdx.x; k < nb; k += blockDim.x) {
    if (!active[k]) continue;
    c64* __restrict__ Hk = st.H + (int64_t)k * (m + 1) * m;
    const c64* __restrict__ hk = h + (int64_t)k * (j + 1);
    const c64* __restrict__ csk = st.cs + (int64_t)k * m;
    const c64* __restrict__ snk = st.sn + (int64_t)k * m;
    // rotation i acts on entries i (already rotated by rotation i - 1) and i + 1
    // (still as formed): the column streams through `a`, and entry i is final
    // after rotation i (no indexed local array, which would live in scratch)
    c64 a = hk[0];
    // four rotations' loads at a time ahead of their chain
    for (int i0 = 0; i0 < j; i0 += 4) {
      double c[4];
      c64 s[4], b[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u < j ? i0 + u : i0;
        c[u] = csk[i].re;
        s[u] = snk[i];
        b[u] = hk[i + 1];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (i0 + u >= j) break;
        // [a; b] <- [c a + s b; -conj(s) a + c b]
        Hk[(int64_t)(i0 + u) * m + j] = c[u] * a + s[u] * b[u];
        const c64 sc = {s[u].re, -s[u].im};
        a = c[u] * b[u] - sc * a;
      }
    }
    const c64 b = {sqrt(wn2[k].re), 0.0};
    const double na = sqrt(a.re * a.re + a.im * a.im), nbv = sqrt(b.re * b.re + b.im * b.im);
    const double r = sqrt(na * na + nbv * nbv);
    double c;
    c64 s;
    if (r == 0.0) {
      c = 1.0;
      s = {0.0, 0.0};
    } else if (na == 0.0) {
      c = 0.0;
      s = {b.re / nbv, -b.im / nbv};  // conj(b)/|b|
    } else {
      c = na / r;
      const c64 ph = {a.re / na, a.im / na};
      const c64 bc = {b.re / r, -b.im / r};  // conj(b)/r
      s = ph * bc;
    }
    st.cs[(int64_t)k * m + j] = {c, 0.0};
    st.sn[(int64_t)k * m + j] = s;
    Hk[(int64_t)j * m + j] = c * a + s * b;
    c64* gk = st.g + (int64_t)k * (m + 1);
    const c64 gj = gk[j];
    const c64 sc = {s.re, -s.im};
    gk[j] = c * gj;
    gk[j + 1] = -1.0 * (sc * gj);
    const double res = sqrt(gk[j + 1].re * gk[j + 1].re + gk[j + 1].im * gk[j + 1].im);
    st.dims[k] = j + 1;
    const double bn = sqrt(beta2[k].re);
    if (res <= tol * bn || !(res == res) || j + 1 == m)
      active[k] = 0;
    else
      atomicAdd(&cnt, 1);
  }
  __syncthreads();
  if (threadIdx.x == 0) *count = cnt;
}

// y = R^{-1} g (back substitution on the rotated Hessenberg): a wave per column, lane i
// keeps row i's right-hand side, R in LDS (one thread per column and loads in the chain:
// 15 us for 16 vectors)
__global__ __launch_bounds__(64) void k_givens_solve(GState st, c64* y, const int* start, int m) {
  __shared__ c64 R[(kMaxBasis - 1) * (kMaxBasis - 1)];
  const int k = blockIdx.x, lane = threadIdx.x;
  if (!start[k]) return;
  const c64* Hk = st.H + (int64_t)k * (m + 1) * m;
  const int d = st.dims[k];
  for (int i = lane; i < d * d; i += 64) R[i] = Hk[(int64_t)(i / d) * m + i % d];
  c64 acc = lane < d ? st.g[(int64_t)k * (m + 1) + lane] : c64{0.0, 0.0};
  __syncthreads();
  for (int i = d - 1; i >= 0; --i) {
    const c64 rii = R[i * d + i];
    const double dd = rii.re * rii.re + rii.im * rii.im;
    const c64 inv = dd > 0.0 ? c64{rii.re / dd, -rii.im / dd} : c64{0.0, 0.0};
    const c64 yi = inv * c64{__shfl(acc.re, i, 64), __shfl(acc.im, i, 64)};
    if (lane == i) y[(int64_t)k * m + i] = yi;
    if (lane < i) acc -= R[lane * d + i] * yi;
  }
}

inline dim3 grid_n(int64_t n, int nb) {
  return dim3((unsigned)((n + kThreads - 1) / kThreads), (unsigned)nb);
}

// elements per thread of the passes over one vector: one while that keeps the launch
// below four blocks per CU, else four (fewer partials to sum in each block)
inline int elems_per_thread(int64_t n, int nb) {
  return (n + kThreads - 1) / kThreads * nb < 1024 ? 1 : 4;
}
inline int pass_blocks(int64_t n, int ept) {
  return (int)((n + kThreads * ept - 1) / (kThreads * ept));
}
// partials per dot product up to which every block of the update sums them itself
// instead of a launch between: 64 partials of 17 vectors are 17 KB per block, half of
// what the block reads of the vectors, against 3 us for the launch
constexpr int kInlineSums = 64;

}  // namespace

// one step of classical Gram-Schmidt for the basis V_0 .. V_{nv-1}: h = V^H w,
// w -= V h, wn2 = |w|^2, w /= |w|
template <typename T>
void krylov_orthonormalise(const T* V, int64_t vstride, int nv, T* w, int64_t n, int nb,
                           const int* active, c64* h, c64* wn2, c64* partials, hipStream_t s) {
  MLMC_REQUIRE(nv <= kMaxBasis, MLMC_EUNSUPPORTED, "Krylov basis too large");
  // enough parallelism but few partials: nv*nb*nblk entries
  int nblk = reduce_blocks(n);
  if (nblk > 256) nblk = 256;
  hipLaunchKernelGGL(k_mdot<T>, dim3(nblk, nb, (nv + 3) / 4), dim3(kThreads), 0, s, V, vstride,
                     nv, w, n, active, partials);
  const bool fused = nblk <= kInlineSums;
  if (!fused) finish_sums(partials, nblk, nb * nv, h, s);
  c64* wparts = fused ? partials + (int64_t)nblk * nb * nv : partials;
  const c64* hparts = fused ? partials : nullptr;
  const int ept = elems_per_thread(n, nb), np = pass_blocks(n, ept);
  const dim3 g((unsigned)np, (unsigned)nb);
  if (ept == 1) {
    hipLaunchKernelGGL((k_maxpy<T, 1>), g, dim3(kThreads), 0, s, V, vstride, nv, h, hparts, nblk,
                       w, n, active, wparts);
    hipLaunchKernelGGL((k_scale_inv_norm<T, 1>), g, dim3(kThreads), 0, s, w, w, wparts, np, wn2,
                       n, active);
  } else {
    hipLaunchKernelGGL((k_maxpy<T, 4>), g, dim3(kThreads), 0, s, V, vstride, nv, h, hparts, nblk,
                       w, n, active, wparts);
    hipLaunchKernelGGL((k_scale_inv_norm<T, 4>), g, dim3(kThreads), 0, s, w, w, wparts, np, wn2,
                       n, active);
  }
}

// dst = src / |src| and nrm2 = |src|^2
template <typename T>
void krylov_normalise(T* dst, const T* src, int64_t n, int nb, const int* active, c64* nrm2,
                      c64* partials, hipStream_t s) {
  vec_dot_partials<T>(src, src, n, nb, active, partials, s);
  const int ept = elems_per_thread(n, nb);
  const dim3 g((unsigned)pass_blocks(n, ept), (unsigned)nb);
  if (ept == 1)
    hipLaunchKernelGGL((k_scale_inv_norm<T, 1>), g, dim3(kThreads), 0, s, dst, src, partials,
                       reduce_blocks(n), nrm2, n, active);
  else
    hipLaunchKernelGGL((k_scale_inv_norm<T, 4>), g, dim3(kThreads), 0, s, dst, src, partials,
                       reduce_blocks(n), nrm2, n, active);
}

template <typename T>
void krylov_combine(const T* Z, int64_t vstride, const c64* y, int ldy, const int* dims, T* d,
                    int64_t n, int nb, const int* start, hipStream_t s) {
  hipLaunchKernelGGL(k_combine<T>, grid_n(n, nb), dim3(kThreads), 0, s, Z, vstride, y, ldy,
                     dims, d, n, start);
}

void givens_init(c64* H, c64* cs, c64* sn, c64* g, int* dims, const c64* beta2,
                 const int* active, int m, int nb, hipStream_t s) {
  GState st{H, cs, sn, g, dims};
  hipLaunchKernelGGL(k_givens_init, dim3((nb + 255) / 256), dim3(256), 0, s, st, beta2, active,
                     m, nb);
}

void givens_step(c64* H, c64* cs, c64* sn, c64* g, int* dims, const c64* h, const c64* wn2,
                 const c64* beta2, double tol, int j, int m, int* active, int nb, int* count,
                 hipStream_t s) {
  GState st{H, cs, sn, g, dims};
  hipLaunchKernelGGL(k_givens_step, dim3(1), dim3(256), 0, s, st, h, wn2, beta2, tol, j, m,
                     active, nb, count);
}

void givens_solve(c64* H, c64* cs, c64* sn, c64* g, int* dims, c64* y, const int* start, int m,
                  int nb, hipStream_t s) {
  GState st{H, cs, sn, g, dims};
  MLMC_REQUIRE(m < kMaxBasis, MLMC_EUNSUPPORTED, "Krylov basis too large");
  hipLaunchKernelGGL(k_givens_solve, dim3(nb), dim3(64), 0, s, st, y, start, m);
}

#define MLMC_INST_K(T)                                                                        \
  template void krylov_orthonormalise<T>(const T*, int64_t, int, T*, int64_t, int, const int*, \
                                         c64*, c64*, c64*, hipStream_t);                      \
  template void krylov_normalise<T>(T*, const T*, int64_t, int, const int*, c64*, c64*,       \
                                    hipStream_t);                                             \
  template void krylov_combine<T>(const T*, int64_t, const c64*, int, const int*, T*,         \
                                  int64_t, int, const int*, hipStream_t);

MLMC_INST_K(c32)
MLMC_INST_K(c64)

}  // namespace mlmc
