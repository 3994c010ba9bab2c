// Small 2D Poisson grids (sides up to 128): a whole V-cycle, and a whole Krylov
// solve, of one right-hand side per workgroup.
//
// The lockstep launches of these levels are bound by latency: each stage of a
// V-cycle on 128^2 and below takes 4-10 us whatever the batch width, mostly
// launch, load and drain, and one CG iteration on a 128^2 hierarchy is about 20
// such launches.  A column's solve touches nothing of the other columns, so a
// workgroup of 16 waves runs it alone: a level's iterate and right-hand side
// stay in registers, the levels below in LDS, and the reductions of the
// recursion never leave the workgroup.
//
// Layout of a level of side S (even): a lane holds a column pair and R rows, so
// every row has exactly one cell of each colour per lane, as in k_rbgs2_march.
// Strips of R rows go to waves (R = 8, 64 column pairs, sides 66..128) or to
// half waves (R = 2, 32 column pairs, sides up to 64: two rows per lane instead
// of four with half the lanes idle).  A colour stage needs one lane shift per
// row, and for the strip's first and last row one value of the neighbouring
// strip, exchanged through LDS: a stage of colour C writes its own edge cells to
// the buffers of colour C and reads those of the other colour, which gives one
// barrier per stage.
//
// The coarsest level (side m <= 64, constant coefficients) is solved in the sine
// basis, X = S ((S B S) / lambda) S, as four m x m x m products on
// v_mfma_{f32,f64}_16x16x4: 8 m^3 operations from LDS instead of the 2 m^4 (and
// the m^4 matrix entries read through L2) of the explicit inverse.
#include "kernels.h"
#include "lanes.h"
#include "vec_body.h"

namespace mlmc {
namespace {

constexpr int kSmT = 1024;              // threads: 16 waves
constexpr int kSmallLds = 160 * 1024;   // LDS of a compute unit

// planes that fill half of the 128 registers of a thread
template <typename T, int R>
constexpr bool kWide = sizeof(T) == 8 && R == 8;

template <typename T>
struct alignas(2 * sizeof(T)) Pair2 {
  T e0, e1;
};

// LDS pieces of a workgroup (offsets from the dynamic base; see small_lds)
template <typename T>
struct SmLds {
  double* red;  // 2 x 16 wave sums
  T* ed;        // [colour][first, last row of the strip][thread]
  T* bas;       // sine basis, mp x ld
  T *t0, *t1;   // coarsest right-hand side / solution and the products' scratch
  T* lev;       // b and x of the smoothed levels below the top
  double* yed;  // FP64 edges of the refinement residual (over lev and below)
  int slot;     // reduction slot in use
};

// the thread's index behind a barrier for the optimiser: a level's addresses and
// masks are then formed where the level is visited instead of being hoisted out
// of every loop around it, which spills the registers that hold the planes
__device__ __forceinline__ int fresh_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// where a strip lies on a level of side S
struct Geo {
  int S, W, sub, strip, y0, tid;
  bool col;
};

template <int R>
__device__ __forceinline__ Geo geo_of(int S) {
  Geo g;
  g.tid = fresh_tid();
  const int lane = g.tid & 63, w = g.tid >> 6;
  g.S = S;
  if (R == 2 && S > 32) {
    g.W = 32;
    g.sub = lane & 31;
    g.strip = 2 * w + (lane >> 5);
  } else {
    g.W = 64;
    g.sub = lane;
    g.strip = w;
  }
  g.y0 = g.strip * R;
  g.col = 2 * g.sub < S;
  return g;
}

template <typename T>
__device__ __forceinline__ T from_left(T v, const Geo& g) {
  const T s = wave_shr1(v);
  return g.sub == 0 ? (T)0 : s;
}
template <typename T>
__device__ __forceinline__ T from_right(T v, const Geo& g) {
  const T s = wave_shl1(v);
  return g.sub == g.W - 1 ? (T)0 : s;
}

// edge values of the strips above and below in the buffers of colour C
template <typename U>
__device__ __forceinline__ U edge_above(const U* ed, int C, const Geo& g) {
  return g.strip > 0 ? ed[(2 * C + 1) * kSmT + g.tid - g.W] : (U)0;
}
template <typename U>
__device__ __forceinline__ U edge_below(const U* ed, int C, const Geo& g) {
  return g.tid + g.W < kSmT ? ed[(2 * C) * kSmT + g.tid + g.W] : (U)0;
}

// this strip's edge cells of colour C (row 0 is an even row, row R - 1 an odd one)
template <int R, int C, typename U>
__device__ __forceinline__ void publish(U* ed, const U (&X0)[R], const U (&X1)[R],
                                        const Geo& g) {
  ed[(2 * C) * kSmT + g.tid] = C == 0 ? X0[0] : X1[0];
  ed[(2 * C + 1) * kSmT + g.tid] = C == 1 ? X0[R - 1] : X1[R - 1];
}

// one colour stage of the Gauss-Seidel sweep; Z: the iterate is zero so far
template <int R, int C, bool Z, typename T>
__device__ __forceinline__ void stage(T (&X0)[R], T (&X1)[R], const T (&B0)[R], const T (&B1)[R],
                                      T dinv, T c, const Geo& g, T* ed) {
  T up = 0, dn = 0;
  if (!Z) {
    up = edge_above(ed, 1 - C, g);
    dn = edge_below(ed, 1 - C, g);
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (R > 2 && r % 2 == 0) __builtin_amdgcn_sched_barrier(0);  // rows in order: few temporaries
    const bool in = g.col && g.y0 + r < g.S;
    if (((C + r) & 1) == 0) {
      T v = dinv * B0[r];
      if (!Z) {
        const T a = r > 0 ? X0[r > 0 ? r - 1 : 0] : up, b = r < R - 1 ? X0[r < R - 1 ? r + 1 : r] : dn;
        v = dinv * (B0[r] + c * (from_left(X1[r], g) + X1[r] + a + b));
      }
      X0[r] = in ? v : (T)0;
    } else {
      T v = dinv * B1[r];
      if (!Z) {
        const T a = r > 0 ? X1[r > 0 ? r - 1 : 0] : up, b = r < R - 1 ? X1[r < R - 1 ? r + 1 : r] : dn;
        v = dinv * (B1[r] + c * (X0[r] + from_right(X0[r], g) + a + b));
      }
      X1[r] = in ? v : (T)0;
    }
  }
  publish<R, C>(ed, X0, X1, g);
  __syncthreads();
}

// neighbour sums of the strip's cells (both colours of the edges published):
// f(r, sum of column 2 sub, sum of column 2 sub + 1)
template <int R, typename U, typename F>
__device__ __forceinline__ void neighbour_sums(const U (&X0)[R], const U (&X1)[R], const Geo& g,
                                               const U* ed, F&& f) {
  const U up0 = edge_above(ed, 1, g), up1 = edge_above(ed, 0, g);
  const U dn0 = edge_below(ed, 0, g), dn1 = edge_below(ed, 1, g);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (R > 2) __builtin_amdgcn_sched_barrier(0);
    const U a0 = r > 0 ? X0[r > 0 ? r - 1 : 0] : up0, a1 = r > 0 ? X1[r > 0 ? r - 1 : 0] : up1;
    const U b0 = r < R - 1 ? X0[r < R - 1 ? r + 1 : r] : dn0;
    const U b1 = r < R - 1 ? X1[r < R - 1 ? r + 1 : r] : dn1;
    f(r, from_left(X1[r], g) + X1[r] + a0 + b0, X0[r] + from_right(X0[r], g) + a1 + b1);
  }
}

// sweeps of the pre-smoother (first colour first); `zero`: from a zero iterate,
// else both colours of the edges are published
template <int R, typename T>
__device__ __forceinline__ void pre_smooth(T (&X0)[R], T (&X1)[R], const T (&B0)[R],
                                           const T (&B1)[R], T dinv, T c, const Geo& g, T* ed,
                                           int sweeps, bool zero) {
  if (sweeps == 0 && zero) {  // the residual below reads the edges
    publish<R, 0>(ed, X0, X1, g);
    publish<R, 1>(ed, X0, X1, g);
    __syncthreads();
  }
  for (int s = 0; s < sweeps; ++s) {
    if (s == 0 && zero)
      stage<R, 0, true>(X0, X1, B0, B1, dinv, c, g, ed);
    else
      stage<R, 0, false>(X0, X1, B0, B1, dinv, c, g, ed);
    stage<R, 1, false>(X0, X1, B0, B1, dinv, c, g, ed);
  }
}

template <int R, typename T>
__device__ __forceinline__ void post_smooth(T (&X0)[R], T (&X1)[R], const T (&B0)[R],
                                            const T (&B1)[R], T dinv, T c, const Geo& g, T* ed,
                                            int sweeps) {
  // both colours of the edges: the first stage reads colour 0, the stencils
  // that follow a V-cycle without post-smoothing both
  publish<R, 0>(ed, X0, X1, g);
  publish<R, 1>(ed, X0, X1, g);
  __syncthreads();
  for (int s = 0; s < sweeps; ++s) {
    stage<R, 1, false>(X0, X1, B0, B1, dinv, c, g, ed);
    stage<R, 0, false>(X0, X1, B0, B1, dinv, c, g, ed);
  }
}

// rc = R (b - A x) over the 2 x 2 aggregates into an LDS plane of row stride st
template <int R, typename T>
__device__ __forceinline__ void restrict_residual(const T (&X0)[R], const T (&X1)[R],
                                                  const T (&B0)[R], const T (&B1)[R], T d, T c,
                                                  const Geo& g, const T* ed, T* rc, int st) {
  T acc = 0;
  neighbour_sums<R>(X0, X1, g, ed, [&](int r, T s0, T s1) {
    acc += B0[r] - (d * X0[r] - c * s0);
    acc += B1[r] - (d * X1[r] - c * s1);
    if (r & 1) {
      if (g.col && g.y0 + r < g.S) rc[((g.y0 + r) >> 1) * st + g.sub] = (T)0.5 * acc;
      acc = 0;
    }
  });
}

// X += wh * (coarse correction of the cell's aggregate)
template <int R, typename T>
__device__ __forceinline__ void correct(T (&X0)[R], T (&X1)[R], T wh, const Geo& g, const T* ec,
                                        int st) {
#pragma unroll
  for (int r = 0; r < R; r += 2) {
    if (g.col && g.y0 + r < g.S) {
      const T e = wh * ec[((g.y0 + r) >> 1) * st + g.sub];
      X0[r] += e;
      X1[r] += e;
      X0[r + 1] += e;
      X1[r + 1] += e;
    }
  }
}

// rows of a plane of side S (registers of out-of-grid cells: zero)
template <int R, typename T, typename U>
__device__ __forceinline__ void load_plane(T (&X0)[R], T (&X1)[R], const U* p, const Geo& g) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool in = g.col && g.y0 + r < g.S;
    const Pair2<U> v =
        reinterpret_cast<const Pair2<U>*>(p)[in ? (g.y0 + r) * (g.S >> 1) + g.sub : 0];
    X0[r] = in ? (T)v.e0 : (T)0;
    X1[r] = in ? (T)v.e1 : (T)0;
  }
}
template <int R, typename T>
__device__ __forceinline__ void store_plane(const T (&X0)[R], const T (&X1)[R], T* p,
                                            const Geo& g) {
#pragma unroll
  for (int r = 0; r < R; ++r)
    if (g.col && g.y0 + r < g.S)
      reinterpret_cast<Pair2<T>*>(p)[(g.y0 + r) * (g.S >> 1) + g.sub] = Pair2<T>{X0[r], X1[r]};
}

// out = scale o (L Rm) of mp x mp LDS planes (row stride ld), a 16 x 16 tile per
// wave; scale (global, mp x mp; nullptr: 1)
template <typename T>
__device__ __forceinline__ void sine_product(const T* L, const T* Rm, T* out, int mp, int ld,
                                             const T* scale) {
  const int tid = fresh_tid(), tiles = mp >> 4, wave = tid >> 6, lane = tid & 63;
  if (wave < tiles * tiles) {
    const int ti = wave / tiles, tj = wave - ti * tiles;
    const int g = lane >> 4, cc = lane & 15;
    const T* a = L + (16 * ti + cc) * ld + g;
    const T* b = Rm + g * ld + 16 * tj + cc;
    typename body::Mfma<T>::acc_t acc = {0, 0, 0, 0};
    for (int k = 0; k < mp; k += 16) {
#pragma unroll
      for (int u = 0; u < 16; u += 4)
        acc = body::Mfma<T>::step(a[k + u], b[(k + u) * ld], acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * ti + body::Mfma<T>::row(g, r), j = 16 * tj + cc;
      out[i * ld + j] = scale ? acc[r] * scale[i * mp + j] : acc[r];
    }
  }
  __syncthreads();
}

// coarsest solve: t0 = A^-1 t0
template <typename T>
__device__ __forceinline__ void coarsest(const SmallGrid<T>& q, const SmLds<T>& sm) {
  const int ld = q.mp + kSmallPad;
  sine_product<T>(sm.bas, sm.t0, sm.t1, q.mp, ld, nullptr);
  sine_product<T>(sm.t1, sm.bas, sm.t0, q.mp, ld, q.ilam);
  sine_product<T>(sm.bas, sm.t0, sm.t1, q.mp, ld, nullptr);
  sine_product<T>(sm.t1, sm.bas, sm.t0, q.mp, ld, nullptr);
}

// where level j's right-hand side and iterate lie in LDS, and their row stride
template <typename T>
__device__ __forceinline__ T* lev_b(const SmallGrid<T>& q, const SmLds<T>& sm, int j) {
  return j == q.nl - 1 ? sm.t0 : sm.lev + q.off[j];
}
template <typename T>
__device__ __forceinline__ T* lev_x(const SmallGrid<T>& q, const SmLds<T>& sm, int j) {
  return j == q.nl - 1 ? sm.t0 : sm.lev + q.off[j] + q.side[j] * q.side[j];
}
template <typename T>
__device__ __forceinline__ int lev_st(const SmallGrid<T>& q, int j) {
  return j == q.nl - 1 ? q.mp + kSmallPad : q.side[j];
}

// `cycles` V-cycles on level j0 (below the top) for its right-hand side in LDS,
// the second one started from the first one's result; the result in lev_x
template <typename T>
__device__ void coarse_levels(const SmallGrid<T>& q, const SmLds<T>& sm, int j0, int cycles) {
  const int J = q.nl - 1;
  if (j0 == J) {
    coarsest(q, sm);
    return;
  }
  for (int cyc = 0; cyc < cycles; ++cyc) {
    for (int j = j0; j < J; ++j) {
      const Geo g = geo_of<2>(q.side[j]);
      T X0[2], X1[2], B0[2], B1[2];
      load_plane<2>(B0, B1, lev_b(q, sm, j), g);
      const bool zero = j > j0 || cyc == 0;
      if (zero) {
#pragma unroll
        for (int r = 0; r < 2; ++r) X0[r] = X1[r] = 0;
      } else {
        load_plane<2>(X0, X1, lev_x(q, sm, j), g);
        publish<2, 0>(sm.ed, X0, X1, g);
        publish<2, 1>(sm.ed, X0, X1, g);
        __syncthreads();
      }
      pre_smooth<2>(X0, X1, B0, B1, q.dinv[j], q.c[j], g, sm.ed, q.pre, zero);
      restrict_residual<2>(X0, X1, B0, B1, q.d[j], q.c[j], g, sm.ed, lev_b(q, sm, j + 1),
                           lev_st(q, j + 1));
      store_plane<2>(X0, X1, lev_x(q, sm, j), g);
      __syncthreads();
    }
    coarsest(q, sm);
    for (int j = J - 1; j >= j0; --j) {
      const Geo g = geo_of<2>(q.side[j]);
      T X0[2], X1[2], B0[2], B1[2];
      load_plane<2>(B0, B1, lev_b(q, sm, j), g);
      load_plane<2>(X0, X1, lev_x(q, sm, j), g);
      correct<2>(X0, X1, q.wh, g, lev_x(q, sm, j + 1), lev_st(q, j + 1));
      post_smooth<2>(X0, X1, B0, B1, q.dinv[j], q.c[j], g, sm.ed, q.post);
      store_plane<2>(X0, X1, lev_x(q, sm, j), g);
      __syncthreads();
    }
  }
}

// one V-cycle on the top level (index 0, smoothed), X <- X + V(B - A X); `zero`:
// X is zero on entry, else both colours of its edges are published.  On return
// both are published.  bmem: B in global memory, read again after the coarse
// levels where X and B are half of the registers (FP64, R = 8).
template <int R, typename T>
__device__ __forceinline__ void top_cycle(const SmallGrid<T>& q, const SmLds<T>& sm, const Geo& g,
                                          T (&X0)[R], T (&X1)[R], T (&B0)[R], T (&B1)[R],
                                          bool zero, int child_cycles, const T* bmem) {
  if (zero) {
#pragma unroll
    for (int r = 0; r < R; ++r) X0[r] = X1[r] = 0;
  }
  pre_smooth<R>(X0, X1, B0, B1, q.dinv[0], q.c[0], g, sm.ed, q.pre, zero);
  restrict_residual<R>(X0, X1, B0, B1, q.d[0], q.c[0], g, sm.ed, lev_b(q, sm, 1), lev_st(q, 1));
  __syncthreads();
  coarse_levels<T>(q, sm, 1, child_cycles);
  if constexpr (kWide<T, R>) load_plane<R>(B0, B1, bmem, g);
  correct<R>(X0, X1, q.wh, g, lev_x(q, sm, 1), lev_st(q, 1));
  post_smooth<R>(X0, X1, B0, B1, q.dinv[0], q.c[0], g, sm.ed, q.post);
}

// sum of v over the workgroup (waves in order), the same on every thread
template <typename T>
__device__ __forceinline__ double wg_sum(SmLds<T>& sm, double v) {
  v = wave_sum(v);
  double* red = sm.red + 16 * sm.slot;
  sm.slot ^= 1;
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = red[0];
#pragma unroll
  for (int w = 1; w < 16; ++w) s += red[w];
  return s;
}

template <int R, typename T>
__device__ __forceinline__ double dot_local(const T (&A0)[R], const T (&A1)[R], const T (&C0)[R],
                                            const T (&C1)[R]) {
  double s = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    s += (double)A0[r] * C0[r];
    s += (double)A1[r] * C1[r];
  }
  return s;
}

template <typename T>
__device__ __forceinline__ SmLds<T> lds_of(const SmallGrid<T>& q, char* base) {
  SmLds<T> sm;
  sm.red = reinterpret_cast<double*>(base);
  sm.ed = reinterpret_cast<T*>(base + 2 * 16 * sizeof(double));
  sm.bas = sm.ed + 4 * kSmT;
  const int plane = q.mp * (q.mp + kSmallPad);
  sm.t0 = sm.bas + plane;
  sm.t1 = sm.t0 + plane;
  sm.lev = sm.t1 + plane;
  sm.yed = reinterpret_cast<double*>(sm.lev);
  sm.slot = 0;
  return sm;
}

// sine basis into LDS; t0's padding has to be finite (the basis is zero there)
template <typename T>
__device__ __forceinline__ void lds_init(const SmallGrid<T>& q, const SmLds<T>& sm) {
  const int ld = q.mp + kSmallPad;
  for (int i = threadIdx.x; i < q.mp * ld; i += kSmT) {
    const int row = i / ld, col = i - row * ld;
    sm.bas[i] = col < q.mp ? q.basis[row * q.mp + col] : (T)0;
    sm.t0[i] = 0;
  }
  __syncthreads();
}

// Z = `cycles` V-cycles for B from Z0 (nullptr: zero), the second one started
// from the first; with partials also the column's conj(b)^T z.  nl == 1: the
// coarsest solve alone.
// Bound by the chain of stages (barrier, LDS edge, update), not by bandwidth: the
// two cycles below a 256^2 level (128^2, 64^2, 32^2; 128 columns, FP32, 2 + 2
// sweeps) take 21 us against about 82 us as lockstep launches.
template <typename T, int R>
__global__ __launch_bounds__(kSmT) void k_small_vcycle(const T* b, T* z, const T* z0,
                                                       SmallGrid<T> q, int cycles,
                                                       const int* active, c64* partials,
                                                       int* tlog) {
  extern __shared__ __align__(16) char small_lds_base[];
  const int k = blockIdx.x;
  if (tlog && threadIdx.x == 0) tlog[k] = active ? active[k] : 1;
  if (active && !active[k]) return;
  SmLds<T> sm = lds_of(q, small_lds_base);
  const int S = q.side[0];
  const int64_t off = (int64_t)k * S * S;
  lds_init(q, sm);
  if (q.nl == 1) {
    const int ld = q.mp + kSmallPad;
    for (int i = threadIdx.x; i < S * S; i += kSmT) sm.t0[(i / S) * ld + i % S] = b[off + i];
    __syncthreads();
    coarsest(q, sm);
    double s = 0.0;
    for (int i = threadIdx.x; i < S * S; i += kSmT) {
      const T v = sm.t0[(i / S) * ld + i % S];
      if (partials) s += (double)b[off + i] * v;
      z[off + i] = v;
    }
    if (partials) {
      s = wg_sum(sm, s);
      if (threadIdx.x == 0) partials[k] = {s, 0.0};
    }
    return;
  }
  const Geo g = geo_of<R>(S);
  T X0[R], X1[R], B0[R], B1[R];
  load_plane<R>(B0, B1, b + off, g);
  if (z0) {
    load_plane<R>(X0, X1, z0 + off, g);
    publish<R, 0>(sm.ed, X0, X1, g);
    publish<R, 1>(sm.ed, X0, X1, g);
    __syncthreads();
  }
  for (int cyc = 0; cyc < cycles; ++cyc)
    top_cycle<R>(q, sm, g, X0, X1, B0, B1, !z0 && cyc == 0, 1, b + off);
  store_plane<R>(X0, X1, z + off, g);
  if (partials) {
    const double s = wg_sum(sm, dot_local<R>(B0, B1, X0, X1));
    if (threadIdx.x == 0) partials[k] = {s, 0.0};
  }
}

// p <- z + beta p, kept in P for the stencils that follow (edges published);
// R = 8: the direction lives in global memory between the iterations
template <int R, typename T>
__device__ __forceinline__ void next_direction(const T (&Z0)[R], const T (&Z1)[R], T (&P0)[R],
                                               T (&P1)[R], T beta, bool first, T* pbuf, int S,
                                               T* ed) {
  const Geo g = geo_of<R>(S);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    Pair2<T> p = {P0[r], P1[r]};
    if constexpr (R == 8) {
      const bool in = g.col && g.y0 + r < g.S;
      Pair2<T>* at = reinterpret_cast<Pair2<T>*>(pbuf) + (in ? (g.y0 + r) * (g.S >> 1) + g.sub : 0);
      p = {0, 0};
      if (!first && in) p = *at;
      p = {Z0[r] + beta * p.e0, Z1[r] + beta * p.e1};
      if (in) *at = p;
    } else {
      p = {Z0[r] + beta * p.e0, Z1[r] + beta * p.e1};
    }
    P0[r] = p.e0;
    P1[r] = p.e1;
  }
  publish<R, 0>(ed, P0, P1, g);
  publish<R, 1>(ed, P0, P1, g);
  __syncthreads();
}

// p^T A p of the strip
template <int R, typename T>
__device__ __forceinline__ double curvature(const T (&P0)[R], const T (&P1)[R], T d, T c,
                                            const Geo& g, const T* ed) {
  double pq = 0.0;
  neighbour_sums<R>(P0, P1, g, ed, [&](int r, T s0, T s1) {
    pq += (double)P0[r] * (d * P0[r] - c * s0);
    pq += (double)P1[r] * (d * P1[r] - c * s1);
  });
  return pq;
}

// x += a p ; r -= a A p (A p formed again from P) ; |r|^2 of the strip.  R = 8: x
// in global memory (x_zero: not read); FP64: r also written there (rbuf)
template <int R, typename T>
__device__ __forceinline__ double step_xr(T (&x0)[R], T (&x1)[R], T (&r0)[R], T (&r1)[R],
                                          const T (&P0)[R], const T (&P1)[R], T a, T d, T c,
                                          bool x_zero, T* xbuf, T* rbuf, int S,
                                          const T* ed) {
  const Geo g = geo_of<R>(S);
  double rr = 0.0;
  neighbour_sums<R>(P0, P1, g, ed, [&](int r, T s0, T s1) {
    const bool in = g.col && g.y0 + r < g.S;
    const int at = in ? (g.y0 + r) * (g.S >> 1) + g.sub : 0;
    if constexpr (R == 8) {
      Pair2<T>* xm = reinterpret_cast<Pair2<T>*>(xbuf) + at;
      Pair2<T> v = {0, 0};
      if (!x_zero && in) v = *xm;
      if (in) *xm = Pair2<T>{v.e0 + a * P0[r], v.e1 + a * P1[r]};
    } else {
      x0[r] = (x_zero ? (T)0 : x0[r]) + a * P0[r];
      x1[r] = (x_zero ? (T)0 : x1[r]) + a * P1[r];
    }
    const T v0 = r0[r] - a * (d * P0[r] - c * s0), v1 = r1[r] - a * (d * P1[r] - c * s1);
    r0[r] = in ? v0 : (T)0;
    r1[r] = in ? v1 : (T)0;
    if constexpr (kWide<T, R>) {
      if (in) reinterpret_cast<Pair2<T>*>(rbuf)[at] = Pair2<T>{v0, v1};
    }
    rr += (double)r0[r] * r0[r];
    rr += (double)r1[r] * r1[r];
  });
  return rr;
}

// Preconditioned CG in precision T from x = 0 to |r| <= tol |b|, a column per
// workgroup: the arithmetic and the per-column decisions of the lockstep pcg, A p
// formed twice instead of stored.  rres: final
// |b - A x|^2 and the iterations taken (im); bb: |b|^2; lastcorr: alpha r^T z of
// the last step.  pbuf, rbuf: a plane per column (sides above 64 only).  64^2 in
// FP64 (three levels, 1 + 1 sweeps): 9.4 us per iteration whatever the batch, 55 us
// as lockstep launches; the 1e-2 trace of that grid 10.6 -> 2.15 ms.
template <typename T, int R>
__global__ __launch_bounds__(kSmT) void k_small_pcg(const T* b, T* x, T* pbuf, T* rbuf,
                                                    SmallGrid<T> q, int child_cycles, double tol2,
                                                    int max_iter, c64* rres, c64* bb,
                                                    c64* lastcorr, int* tlog) {
  extern __shared__ __align__(16) char small_lds_base[];
  const int k = blockIdx.x;
  if (tlog && threadIdx.x == 0) tlog[k] = 1;
  SmLds<T> sm = lds_of(q, small_lds_base);
  const int S = q.side[0];
  const int64_t off = (int64_t)k * S * S;
  const Geo g = geo_of<R>(S);
  const T d = q.d[0], c = q.c[0];
  lds_init(q, sm);
  T r0[R], r1[R], Z0[R], Z1[R], P0[R], P1[R], x0[R], x1[R];
  load_plane<R>(r0, r1, b + off, g);
#pragma unroll
  for (int r = 0; r < R; ++r) x0[r] = x1[r] = P0[r] = P1[r] = 0;
  const double rr0 = wg_sum(sm, dot_local<R>(r0, r1, r0, r1));
  double rz = 0.0, lc = 0.0, rr = 0.0;
  int it = 0;
  for (int tries = 0;; ++tries) {
    for (;;) {
      const Geo g = geo_of<R>(S);
      top_cycle<R>(q, sm, g, Z0, Z1, r0, r1, true, child_cycles, it == 0 ? b + off : rbuf + off);
      const double rzn = wg_sum(sm, dot_local<R>(r0, r1, Z0, Z1));
      const double beta = it > 0 && rz != 0.0 ? rzn / rz : 0.0;
      rz = rzn;
      ++it;
      next_direction<R>(Z0, Z1, P0, P1, (T)beta, it == 1, pbuf + off, S, sm.ed);
      const double pq = wg_sum(sm, curvature<R>(P0, P1, d, c, g, sm.ed));
      const double alpha = pq != 0.0 && isfinite(pq) ? rz / pq : 0.0;
      lc = alpha * rz;
      rr = wg_sum(sm, step_xr<R>(x0, x1, r0, r1, P0, P1, (T)alpha, d, c, it == 1, x + off,
                                 rbuf + off, S, sm.ed));
      if (rr <= tol2 * rr0 || !isfinite(rr) || it >= max_iter) break;
    }
    const bool passed = rr <= tol2 * rr0;
    // the true residual of the result, in place of the recursion's
    if constexpr (R == 8) load_plane<R>(x0, x1, x + off, g);
    publish<R, 0>(sm.ed, x0, x1, g);
    publish<R, 1>(sm.ed, x0, x1, g);
    __syncthreads();
    rr = 0.0;
    neighbour_sums<R>(x0, x1, g, sm.ed, [&](int r, T s0, T s1) {
      const bool in = g.col && g.y0 + r < g.S;
      const int at = in ? (g.y0 + r) * (g.S >> 1) + g.sub : 0;
      const Pair2<T> bv = reinterpret_cast<const Pair2<T>*>(b + off)[at];
      const T v0 = bv.e0 - (d * x0[r] - c * s0), v1 = bv.e1 - (d * x1[r] - c * s1);
      r0[r] = in ? v0 : (T)0;
      r1[r] = in ? v1 : (T)0;
      if constexpr (kWide<T, R>) {
        if (in) reinterpret_cast<Pair2<T>*>(rbuf + off)[at] = Pair2<T>{v0, v1};
      }
      rr += (double)r0[r] * r0[r];
      rr += (double)r1[r] * r1[r];
    });
    rr = wg_sum(sm, rr);
    // Rounding separates the two residuals by some 1e-15 of |b|, so the recursion may
    // pass a column whose true residual misses the tolerance: that column goes on from
    // its true residual with a new direction
    if (!passed || rr <= tol2 * rr0 || !isfinite(rr) || it >= max_iter || tries == 2) break;
    rz = 0.0;
  }
  if constexpr (R != 8) store_plane<R>(x0, x1, x + off, g);
  if (threadIdx.x == 0) {
    rres[k] = {rr, (double)it};
    bb[k] = {rr0, 0.0};
    lastcorr[k] = {lc, 0.0};
  }
}

// FP32 preconditioned CG with FP64 refinement (the rules of pcg_refined), a
// column per workgroup, so that a column is refined when its own recursion asks
// for it.  rres: final |b - A y|^2 and the iterations (im); bb: |b|^2 and the
// refinements (im); err: stated error of the last correction.  pbuf, xbuf: a
// plane per column (sides above 64 only).  A 128-column solve to 1e-10 takes 311 us
// on 128^2 and 97 us on 64^2 (about 0.9 and 0.5 ms as lockstep launches).
template <int R>
__global__ __launch_bounds__(kSmT) void k_small_refined(const double* b, double* y, float* pbuf,
                                                        float* xbuf, SmallGrid<float> q,
                                                        int child_cycles, double d64, double cc64,
                                                        double tol2, double delta2, int max_it,
                                                        c64* rres, c64* bb_out, c64* err,
                                                        int* tlog) {
  extern __shared__ __align__(16) char small_lds_base[];
  const int k = blockIdx.x;
  if (tlog && threadIdx.x == 0) tlog[k] = 1;
  SmLds<float> sm = lds_of(q, small_lds_base);
  const int S = q.side[0];
  const int64_t off = (int64_t)k * S * S;
  const Geo g = geo_of<R>(S);
  const float d = q.d[0], c = q.c[0];
  lds_init(q, sm);
  float r0[R], r1[R], Z0[R], Z1[R], P0[R], P1[R], x0[R], x1[R];
  double bb = 0.0;
  {
    double b0[R], b1[R];
    load_plane<R>(b0, b1, b + off, g);
    bb = wg_sum(sm, dot_local<R>(b0, b1, b0, b1));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      r0[r] = (float)b0[r];
      r1[r] = (float)b1[r];
      x0[r] = x1[r] = P0[r] = P1[r] = 0.f;
    }
  }
  double rr_upd = bb, rz = 0.0, stated = 0.0;
  int it = 0, refs = 0;
  bool x_zero = true;
  for (;;) {
    const Geo g = geo_of<R>(S);
    top_cycle<R>(q, sm, g, Z0, Z1, r0, r1, true, child_cycles, (const float*)nullptr);
    const double rzn = wg_sum(sm, dot_local<R>(r0, r1, Z0, Z1));
    const double beta = it > 0 && rz != 0.0 ? rzn / rz : 0.0;
    rz = rzn;
    ++it;
    next_direction<R>(Z0, Z1, P0, P1, (float)beta, it == 1, pbuf + off, S, sm.ed);
    const double pq = wg_sum(sm, curvature<R>(P0, P1, d, c, g, sm.ed));
    const double alpha = pq != 0.0 && isfinite(pq) ? rz / pq : 0.0;
    const double rr = wg_sum(sm, step_xr<R>(x0, x1, r0, r1, P0, P1, (float)alpha, d, c, x_zero,
                                            xbuf + off, (float*)nullptr, S, sm.ed));
    x_zero = false;
    const bool last = it >= max_it;
    if (!last && (it & 1)) continue;  // tested after every second iteration
    const bool due = rr <= delta2 * rr_upd || rr <= tol2 * bb || !isfinite(rr);
    if (!due && !last) continue;
    // y += x32 and the FP64 residual
    double y0[R], y1[R], bd = 0.0, rn = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const bool in = g.col && g.y0 + r < g.S;
      const int at = in ? (g.y0 + r) * (g.S >> 1) + g.sub : 0;
      const Pair2<double> bv = reinterpret_cast<const Pair2<double>*>(b + off)[at];
      Pair2<double>* ym = reinterpret_cast<Pair2<double>*>(y + off) + at;
      Pair2<float> xv = {x0[r], x1[r]};
      if constexpr (R == 8) xv = reinterpret_cast<const Pair2<float>*>(xbuf + off)[at];
      Pair2<double> yv = {0.0, 0.0};
      if (in) {
        if (refs > 0) yv = *ym;
        yv = {yv.e0 + (double)xv.e0, yv.e1 + (double)xv.e1};
        *ym = yv;
        bd += bv.e0 * (double)xv.e0;
        bd += bv.e1 * (double)xv.e1;
      }
      y0[r] = yv.e0;
      y1[r] = yv.e1;
    }
    publish<R, 0>(sm.yed, y0, y1, g);
    publish<R, 1>(sm.yed, y0, y1, g);
    __syncthreads();
    neighbour_sums<R>(y0, y1, g, sm.yed, [&](int r, double s0, double s1) {
      const bool in = g.col && g.y0 + r < g.S;
      const Pair2<double> bv = reinterpret_cast<const Pair2<double>*>(
          b + off)[in ? (g.y0 + r) * (g.S >> 1) + g.sub : 0];
      const double v0 = in ? bv.e0 - (d64 * y0[r] - cc64 * s0) : 0.0;
      const double v1 = in ? bv.e1 - (d64 * y1[r] - cc64 * s1) : 0.0;
      rn += v0 * v0;
      rn += v1 * v1;
      r0[r] = (float)v0;
      r1[r] = (float)v1;
    });
    x_zero = true;
    bd = wg_sum(sm, bd);
    rn = wg_sum(sm, rn);
    ++refs;
    stated = fabs(bd) * (rr_upd > 0.0 ? sqrt(rn / rr_upd) : 1.0);
    // the kept direction stays only while the recursion's residual describes
    // the true one
    if (!(rn <= 100.0 * rr)) rz = 0.0;
    rr_upd = rn;
    if (rn <= tol2 * bb || !isfinite(rn) || last) break;
  }
  if (threadIdx.x == 0) {
    rres[k] = {rr_upd, (double)it};
    bb_out[k] = {bb, (double)refs};
    err[k] = {stated, 0.0};
  }
}

template <typename K>
void allow_lds(K kern) {
  MLMC_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                               hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLds));
}

}  // namespace

// bytes of LDS: reductions, edges, the coarsest level's three planes, the levels
// between (b and x each); at least the FP64 edges of the refinement over the last
template <typename T>
size_t small_lds(const SmallGrid<T>& q, bool refined) {
  const size_t plane = (size_t)q.mp * (q.mp + kSmallPad);
  size_t lev = 0;
  for (int j = 1; j < q.nl - 1; ++j) lev += 2 * (size_t)q.side[j] * q.side[j];
  size_t tail = lev * sizeof(T);
  if (refined && tail < 4 * (size_t)kSmT * sizeof(double)) tail = 4 * (size_t)kSmT * sizeof(double);
  return 2 * 16 * sizeof(double) + (4 * (size_t)kSmT + 3 * plane) * sizeof(T) + tail;
}

template <typename T>
void small_vcycle(const T* b, T* z, const T* z0, const SmallGrid<T>& q, int cycles, int nb,
                  const int* active, c64* partials, hipStream_t s) {
  const size_t lds = small_lds(q, false);
  if (q.side[0] > 64) {
    MLMC_LAUNCH((k_small_vcycle<T, 8>), dim3(nb), dim3(kSmT), lds, s, b, z, z0, q, cycles, active,
                partials, timing_log());
  } else {
    MLMC_LAUNCH((k_small_vcycle<T, 2>), dim3(nb), dim3(kSmT), lds, s, b, z, z0, q, cycles, active,
                partials, timing_log());
  }
}

template <typename T>
void small_pcg(const T* b, T* x, T* pbuf, T* rbuf, const SmallGrid<T>& q, int child_cycles, double tol,
               int max_iter, int nb, c64* rres, c64* bb, c64* lastcorr, hipStream_t s) {
  const size_t lds = small_lds(q, false);
  if (q.side[0] > 64) {
    MLMC_LAUNCH((k_small_pcg<T, 8>), dim3(nb), dim3(kSmT), lds, s, b, x, pbuf, rbuf, q, child_cycles,
                tol * tol, max_iter, rres, bb, lastcorr, timing_log());
  } else {
    MLMC_LAUNCH((k_small_pcg<T, 2>), dim3(nb), dim3(kSmT), lds, s, b, x, pbuf, rbuf, q, child_cycles,
                tol * tol, max_iter, rres, bb, lastcorr, timing_log());
  }
}

void small_refined(const double* b, double* y, float* pbuf, float* xbuf,
                   const SmallGrid<float>& q, int child_cycles, double d, double c, double tol, double inner_tol, int max_it, int nb,
                   c64* rres, c64* bb, c64* err, hipStream_t s) {
  const size_t lds = small_lds(q, true);
  if (q.side[0] > 64) {
    MLMC_LAUNCH((k_small_refined<8>), dim3(nb), dim3(kSmT), lds, s, b, y, pbuf, xbuf, q, child_cycles, d, c,
                tol * tol, inner_tol * inner_tol, max_it, rres, bb, err, timing_log());
  } else {
    MLMC_LAUNCH((k_small_refined<2>), dim3(nb), dim3(kSmT), lds, s, b, y, pbuf, xbuf, q, child_cycles, d, c,
                tol * tol, inner_tol * inner_tol, max_it, rres, bb, err, timing_log());
  }
}

void small_setup() {
  allow_lds(k_small_vcycle<float, 2>);
  allow_lds(k_small_vcycle<float, 8>);
  allow_lds(k_small_vcycle<double, 2>);
  allow_lds(k_small_vcycle<double, 8>);
  allow_lds(k_small_pcg<double, 2>);
  allow_lds(k_small_pcg<double, 8>);
  allow_lds(k_small_refined<2>);
  allow_lds(k_small_refined<8>);
}

template size_t small_lds<float>(const SmallGrid<float>&, bool);
template size_t small_lds<double>(const SmallGrid<double>&, bool);
template void small_vcycle<float>(const float*, float*, const float*, const SmallGrid<float>&, int,
                                  int, const int*, c64*, hipStream_t);
template void small_vcycle<double>(const double*, double*, const double*,
                                   const SmallGrid<double>&, int, int, const int*, c64*,
                                   hipStream_t);
template void small_pcg<double>(const double*, double*, double*, double*, const SmallGrid<double>&, int,
                                double, int, int, c64*, c64*, c64*, hipStream_t);

}  // namespace mlmc
