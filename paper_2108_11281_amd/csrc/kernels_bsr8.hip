// Block stencils and aggregation with 4 or 8 complex unknowns per lattice site on the
// matrix cores (v_mfma_{f32,f64}_16x16x4).
//
// A block row is a DOF x DOF complex block per neighbour.  Its real and imaginary parts
// are stacked as the 16 rows of the A operand (with 4 unknowns half of the rows repeat
// others and are not used) and eight right-hand sides, real and imaginary parts next to
// each other, are the 16 columns of the B operand: one product gives A_re x_re,
// A_re x_im, A_im x_re and A_im x_im without the doubled matrix of a real
// representation, and the complex result is a sum of two accumulators of neighbouring
// lanes.  The rows are ordered so that a lane's accumulators are the real and imaginary
// rows of its one or two unknowns:
//   f32 (accumulator r of lane group g is row 4 g + r): row 2 i + p (8), 4 i + p (4),
//   f64 (row 4 r + g):                                   row i + 8 p,
// p = 0 real, 1 imaginary, so after the sum lane group g holds the unknowns 2 g, 2 g + 1
// (8 in f32), g, g + 4 (8 in f64) or g (4), which is the B operand of the next product
// (the inverted diagonal block, the restriction) without moving data.
//
// One wave serves a site and 8 or 16 right-hand sides, so the site's blocks are read
// once for all of them, and all loads of the neighbour products are issued before the
// first product.  Narrow batches are bound by that load latency (one launch of a 16^2
// level costs about 3 us whatever it does), wide ones by L2 traffic.  Each column is
// its own vector, 32 to 128 bytes per site at a stride of a whole vector: loads of one
// value per lane left half of every 64-byte run to a second instruction and made wide
// batches slower than one thread per row (a colour of 64^2 sites and 64 columns: 46 us
// the residual), 16-byte loads shared by lane pairs 16 us.
// Measured on the 256^2 two-spin trace (complex64, batches of 1 to 64 columns) against
// one thread per row and column: sweeps 52 -> 33 ms, residuals 21.5 -> 11.5, restriction
// 17.7 -> 6.8; complex128 on 64^2, 5 columns: sweep 6.9 -> 3.4 us, restriction 12 -> 5.
//
// Because a launch costs what it costs, a V-cycle's visit to such a level has as few as
// the red-black order allows (11 before, 8 now with two sweeps each way, 7 and 4 with
// one).  A sweep from zero is one launch on small levels: a site of the second
// colour forms its neighbours' D^-1 b again.  The residual after a sweep is zero on the
// colour solved last, so only the other colour's is formed, and restricted in the same
// launch.  Of a prolonged correction the post-smoothing's first half sweep reads the
// other colour only, and the second half overwrites that: it is added to the neighbours
// where they are read and never stored.
#include "kernels.h"
#include "vec_body.h"
#include "wilson_body.h"

namespace mlmc {
namespace {

template <typename T> using R_t = typename Traits<T>::real;

constexpr int kXcd8 = 8;
// contiguous logical blocks per XCD, so that the column groups of a site and its
// neighbours share an L2
__device__ __forceinline__ int xcd_block() {
  const int total = gridDim.x, b = blockIdx.x;
  const int x = b % kXcd8, local = b / kXcd8, q = total / kXcd8, r = total % kXcd8;
  return x * q + (x < r ? x : r) + local;
}

__device__ __forceinline__ float pair_swap(float v) {  // the value of lane ^ 1
  return __int_as_float(
      __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), 0xB1, 0xf, 0xf, false));
}
__device__ __forceinline__ double pair_swap(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = (int)(u & 0xffffffffll), hi = (int)(u >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, 0xB1, 0xf, 0xf, false);
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, 0xB1, 0xf, 0xf, false);
  return __longlong_as_double(((long long)h2 << 32) | (unsigned int)l2);
}

// the value of the lane of this row's other part (A operand: xor 1 in f32, xor 8 in f64)
__device__ __forceinline__ float row_swap(float v) { return pair_swap(v); }
__device__ __forceinline__ double row_swap(double v) {
  const long long u = __double_as_longlong(v);
  const int lo = (int)(u & 0xffffffffll), hi = (int)(u >> 32);
  const int l2 = __builtin_amdgcn_update_dpp(lo, lo, 0x128, 0xf, 0xf, false);  // row_ror:8
  const int h2 = __builtin_amdgcn_update_dpp(hi, hi, 0x128, 0xf, 0xf, false);
  return __longlong_as_double(((long long)h2 << 32) | (unsigned int)l2);
}

// this lane's place: A row (unknown ai, part ap), column (kc, part), group g
template <typename R, int DOF>
struct Place {
  static_assert(DOF == 4 || DOF == 8, "four or eight unknowns per site");
  static constexpr int NE = DOF / 4;  // unknowns per lane
  int g, kc, part, ai, ap;
  __device__ Place() {
    const int lane = threadIdx.x & 63, m = lane & 15;
    g = lane >> 4;
    kc = m >> 1;
    part = m & 1;
    ai = sizeof(R) == 4 ? (DOF == 8 ? m >> 1 : m >> 2) : m & (DOF - 1);
    ap = sizeof(R) == 4 ? m & 1 : m >> 3;
  }
  __device__ int unknown(int e) const { return sizeof(R) == 4 && DOF == 8 ? 2 * g + e : g + 4 * e; }
};

// the complex products of this lane's unknowns (conj: of the conjugated A)
template <typename R, int NE, bool CONJ, typename Acc>
__device__ __forceinline__ void combine(const Acc& acc, int part, R* out) {
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    const R re = sizeof(R) == 4 ? acc[2 * e] : acc[e];
    const R t = pair_swap(sizeof(R) == 4 ? acc[2 * e + 1] : acc[e + 2]);
    out[e] = ((part != 0) != CONJ) ? re + t : re - t;
  }
}

// Shared loads: an item is W consecutive complex values (16 bytes, or 8 of one complex64)
// of which this lane wants one part each.  Of two items each lane of a pair loads one
// and hands the other lane its part, so a wave reads whole runs with a quarter or half
// of the load instructions.
template <typename R, int W>
struct Item {
  using vec = R __attribute__((ext_vector_type(2 * W), aligned(sizeof(R))));
};

// out[W u + s] = part-th component of value s of item u at ptr(u); AROW: pairs of the
// A operand's rows, else of the B operand's columns
template <typename R, int N, int W, bool AROW, typename P>
__device__ __forceinline__ void load_items(P ptr, int part, R* out) {
  using vec = typename Item<R, W>::vec;
  vec v[N / 2 + 1];
#pragma unroll
  for (int h = 0; h < N / 2; ++h) {
    const R *p0 = ptr(2 * h), *p1 = ptr(2 * h + 1);
    v[h] = *reinterpret_cast<const vec*>(part ? p1 : p0);
  }
  if (N & 1) {
    const R* p0 = ptr(N - 1);
#pragma unroll
    for (int s = 0; s < W; ++s) out[W * (N - 1) + s] = p0[2 * s + part];
  }
#pragma unroll
  for (int h = 0; h < N / 2; ++h) {
#pragma unroll
    for (int s = 0; s < W; ++s) {
      const R keep = part ? v[h][2 * s + 1] : v[h][2 * s];
      const R give = part ? v[h][2 * s] : v[h][2 * s + 1];
      const R got = AROW ? row_swap(give) : pair_swap(give);
      out[W * 2 * h + s] = part ? got : keep;
      out[W * (2 * h + 1) + s] = part ? keep : got;
    }
  }
}

// values per item of a site's unknowns: two neighbours share a lane group in f32 with 8
template <typename R, int DOF>
constexpr int unknown_width() {
  return sizeof(R) == 4 && DOF == 8 ? 2 : 1;
}

// this lane's unknowns of N site vectors (at(q): the site's 2 DOF reals), out[q NE + e]
template <typename R, int DOF, int N, typename P>
__device__ __forceinline__ void load_unknowns(P at, const Place<R, DOF>& pl, R* out) {
  constexpr int W = unknown_width<R, DOF>(), NI = Place<R, DOF>::NE / W;
  load_items<R, N * NI, W, false>(
      [&](int u) { return at(u / NI) + 2 * pl.unknown(u % NI); }, pl.part, out);
}

// this lane's entries (row ai, columns unknown(e)) of N row-major blocks, out[q NE + e]
template <typename R, int DOF, int N, typename P>
__device__ __forceinline__ void load_blocks(P at, const Place<R, DOF>& pl, R* out) {
  constexpr int W = unknown_width<R, DOF>(), NI = Place<R, DOF>::NE / W;
  load_items<R, N * NI, W, true>(
      [&](int u) { return at(u / NI) + 2 * (pl.ai * DOF + pl.unknown(u % NI)); }, pl.ap, out);
}

// a site's unknowns back to memory; with two per lane each lane of a pair stores one
template <typename R, int DOF, typename Ro>
__device__ __forceinline__ void store_unknowns(Ro* at, const Place<R, DOF>& pl, const R* out,
                                               bool on) {
  if constexpr (DOF == 8) {
    using V = Ro __attribute__((ext_vector_type(2), aligned(sizeof(Ro))));
    const R keep = pl.part ? out[1] : out[0];
    const R got = pair_swap(pl.part ? out[0] : out[1]);
    V v;
    v[0] = (Ro)(pl.part ? got : keep);
    v[1] = (Ro)(pl.part ? keep : got);
    if (on) *reinterpret_cast<V*>(at + 2 * pl.unknown(pl.part)) = v;
  } else {
    if (on) at[2 * pl.g + pl.part] = (Ro)out[0];
  }
}

// the columns of a lane: right-hand sides (group CG + q) 8 + kc
template <int CG>
struct Cols {
  int64_t col[CG];
  bool on[CG], live;
  __device__ Cols(int group, int kc, int nb, const int* active) {
    bool any = false;
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      const int k = (group * CG + q) * 8 + kc;
      on[q] = k < nb && (!active || active[k]);
      col[q] = k < nb ? k : 0;
      any = any || on[q];
    }
    // narrow batches don't wait for the flags before their loads: inactive columns are
    // only not stored
    live = CG == 1 || __any(any);
  }
};

__device__ __forceinline__ int neighbour(int X, int Y, int d, int Nc) {
  switch (d) {
    case 1: return Y * Nc + (X + 1 == Nc ? 0 : X + 1);
    case 2: return Y * Nc + (X == 0 ? Nc - 1 : X - 1);
    case 3: return (Y + 1 == Nc ? 0 : Y + 1) * Nc + X;
    case 4: return (Y == 0 ? Nc - 1 : Y - 1) * Nc + X;
    default: return Y * Nc + X;
  }
}

// acc[q] += sum over the NB blocks a (of a site's row) times the vectors v
template <typename R, int NE, int CG, int NB, typename Acc>
__device__ __forceinline__ void multiply(Acc (&acc)[CG], const R* a, const R* v) {
#pragma unroll
  for (int d = 0; d < NB; ++d)
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int q = 0; q < CG; ++q)
        acc[q] = body::Mfma<R>::step(a[d * NE + e], v[(d * CG + q) * NE + e], acc[q]);
}

// acc[q] = sum over the directions D0 .. 4 of block d times the neighbour's vector
template <typename R, int DOF, int CG, int D0, typename Acc>
__device__ __forceinline__ void stencil(Acc (&acc)[CG], const R* __restrict__ B, const R* x, int S,
                                        const int (&tn)[5], int64_t vs, const Place<R, DOF>& pl,
                                        const Cols<CG>& cols) {
  constexpr int NE = Place<R, DOF>::NE, ND = 5 - D0;
  R a[ND * NE], v[ND * CG * NE];
  load_unknowns<R, DOF, ND * CG>(
      [&](int u) { return x + cols.col[u % CG] * vs + (int64_t)tn[D0 + u / CG] * (2 * DOF); }, pl,
      v);
  load_blocks<R, DOF, ND>([&](int d) { return B + ((int64_t)S * 5 + D0 + d) * (2 * DOF * DOF); },
                          pl, a);
#pragma unroll
  for (int q = 0; q < CG; ++q) acc[q] = Acc{0, 0, 0, 0};
  multiply<R, NE, CG, ND>(acc, a, v);
}

// where the neighbours of a half sweep come from
enum Source {
  kFromX,        // x (or zero: nothing is read)
  kFromZero,     // Dinv b of the neighbour, both colours of a sweep from zero in one launch
  kFromProlong,  // x + omega P xc, the correction of the coarse level below
};

// one colour (kFromZero: both) of a red-black block Gauss-Seidel sweep, in place:
// x_S = Dinv_S (b_S - sum_{d != self} B[S][d] x_nbr)
template <typename T, int DOF, int CG, int SRC>
__global__ __launch_bounds__(kThreads) void k_bsr8_gs(const T* __restrict__ b, T* x,
                                                      const T* __restrict__ B,
                                                      const T* __restrict__ Dinv,
                                                      const T* __restrict__ Q,
                                                      const T* __restrict__ xc, R_t<T> omega,
                                                      int blk, int Nc, int colour, int zero_nbrs,
                                                      int nb, int groups, const int* active,
                                                      int* tlog) {
  using R = R_t<T>;
  using Acc = typename body::Mfma<R>::acc_t;
  constexpr int NE = Place<R, DOF>::NE, NM = 2 * DOF * DOF;
  const int t0 = xcd_block(), group = t0 % groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (tlog && t0 < groups && threadIdx.x < 8 * CG && group * 8 * CG + (int)threadIdx.x < nb)
    tlog[group * 8 * CG + threadIdx.x] = active ? active[group * 8 * CG + threadIdx.x] : 1;
  int t = (t0 / groups) * (kThreads / 64) + wave;
  const int hc = Nc >> 1;
  bool nbrs = !zero_nbrs;
  if (SRC == kFromZero) {  // the second colour's waves first
    if (t >= Nc * Nc) return;
    nbrs = t < Nc * hc;
    if (nbrs)
      colour = 1 - colour;
    else
      t -= Nc * hc;
  } else if (t >= Nc * hc) {
    return;
  }
  const Place<R, DOF> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  if (!cols.live) return;
  const int Y = t / hc, X = 2 * (t - Y * hc) + ((colour + Y) & 1), S = Y * Nc + X;
  const int64_t vs = (int64_t)Nc * Nc * (2 * DOF);
  const R* br = reinterpret_cast<const R*>(b);
  R* xr = reinterpret_cast<R*>(x);
  const R* Br = reinterpret_cast<const R*>(B);
  const R* Dr = reinterpret_cast<const R*>(Dinv);
  int tn[5];
#pragma unroll
  for (int d = 0; d < 5; ++d) tn[d] = neighbour(X, Y, d, Nc);
  R rhs[CG * NE], a2[NE];
  load_blocks<R, DOF, 1>([&](int) { return Dr + (int64_t)S * NM; }, pl, a2);
  load_unknowns<R, DOF, CG>(
      [&](int q) { return br + cols.col[q] * vs + (int64_t)S * (2 * DOF); }, pl, rhs);
  if (nbrs) {
    Acc acc[CG];
    if constexpr (SRC == kFromX) {
      stencil<R, DOF, CG, 1>(acc, Br, xr, S, tn, vs, pl, cols);
    } else {
      // the neighbours' vectors: M_nbr w, plus x_nbr
      const R* Mr = SRC == kFromZero ? Dr : reinterpret_cast<const R*>(Q);
      const int NcC = SRC == kFromZero ? 0 : Nc / blk;
      const int64_t vc = (int64_t)NcC * NcC * (2 * DOF);
      R m[4 * NE], w[4 * CG * NE], a[4 * NE], v[4 * CG * NE];
      load_unknowns<R, DOF, 4 * CG>(
          [&](int u) {
            const int n = tn[1 + u / CG];
            if (SRC == kFromZero) return br + cols.col[u % CG] * vs + (int64_t)n * (2 * DOF);
            const int ny = n / Nc, nx = n - ny * Nc;
            return reinterpret_cast<const R*>(xc) + cols.col[u % CG] * vc +
                   (int64_t)((ny / blk) * NcC + nx / blk) * (2 * DOF);
          },
          pl, w);
      load_blocks<R, DOF, 4>([&](int d) { return Mr + (int64_t)tn[1 + d] * NM; }, pl, m);
      if (SRC == kFromProlong)
        load_unknowns<R, DOF, 4 * CG>(
            [&](int u) {
              return xr + cols.col[u % CG] * vs + (int64_t)tn[1 + u / CG] * (2 * DOF);
            },
            pl, v);
      load_blocks<R, DOF, 4>([&](int d) { return Br + ((int64_t)S * 5 + 1 + d) * NM; }, pl, a);
#pragma unroll
      for (int u = 0; u < 4 * CG; ++u) {
        Acc h[1] = {Acc{0, 0, 0, 0}};
        multiply<R, NE, 1, 1>(h, m + (u / CG) * NE, w + u * NE);
        R o[NE];
        combine<R, NE, false>(h[0], pl.part, o);
#pragma unroll
        for (int e = 0; e < NE; ++e)
          v[u * NE + e] = SRC == kFromZero ? o[e] : v[u * NE + e] + omega * o[e];
      }
#pragma unroll
      for (int q = 0; q < CG; ++q) acc[q] = Acc{0, 0, 0, 0};
      multiply<R, NE, CG, 4>(acc, a, v);
    }
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R h[NE];
      combine<R, NE, false>(acc[q], pl.part, h);
#pragma unroll
      for (int e = 0; e < NE; ++e) rhs[q * NE + e] -= h[e];
    }
  }
#pragma unroll
  for (int q = 0; q < CG; ++q) {
    Acc o[1] = {Acc{0, 0, 0, 0}};
    multiply<R, NE, 1, 1>(o, a2, rhs + q * NE);
    R out[NE];
    combine<R, NE, false>(o[0], pl.part, out);
    store_unknowns<R, DOF, R>(xr + cols.col[q] * vs + (int64_t)S * (2 * DOF), pl, out, cols.on[q]);
  }
}

// r = b - A x (b == nullptr: r = A x); spw sites per wave; partials (nullable) of
// |r|^2 (or Re conj(x)^T A x) per column and block
template <typename T, typename Tr, int DOF, int CG>
__global__ __launch_bounds__(kThreads) void k_bsr8_residual(const T* __restrict__ b,
                                                            const T* __restrict__ x,
                                                            Tr* __restrict__ r,
                                                            const T* __restrict__ B, int Nc,
                                                            int nb, int groups, int spw,
                                                            const int* active, c64* partials) {
  using R = R_t<T>;
  using Rr = R_t<Tr>;
  constexpr int NE = Place<R, DOF>::NE;
  __shared__ double red[kThreads / 64][CG * 8];
  const int t0 = xcd_block(), group = t0 % groups, blk = t0 / groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ns = Nc * Nc;
  const Place<R, DOF> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  const int64_t vs = (int64_t)ns * (2 * DOF);
  const R* xr = reinterpret_cast<const R*>(x);
  const R* br = reinterpret_cast<const R*>(b);
  Rr* rr = reinterpret_cast<Rr*>(r);
  double sum[CG];
#pragma unroll
  for (int q = 0; q < CG; ++q) sum[q] = 0.0;
  for (int j = 0; j < spw; ++j) {
    const int S = (blk * (kThreads / 64) + wave) * spw + j;
    if (S >= ns || !cols.live) break;
    const int Y = S / Nc, X = S - Y * Nc;
    int tn[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) tn[d] = neighbour(X, Y, d, Nc);
    R w[CG * NE];
    if (b || partials)
      load_unknowns<R, DOF, CG>(
          [&](int q) {
            const int64_t at = cols.col[q] * vs + (int64_t)S * (2 * DOF);
            return b ? br + at : xr + at;
          },
          pl, w);
    typename body::Mfma<R>::acc_t acc[CG];
    stencil<R, DOF, CG, 0>(acc, reinterpret_cast<const R*>(B), xr, S, tn, vs, pl, cols);
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R h[NE];
      combine<R, NE, false>(acc[q], pl.part, h);
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        if (b) {
          h[e] = w[q * NE + e] - h[e];
          sum[q] += (double)h[e] * h[e];
        } else if (partials) {
          sum[q] += (double)w[q * NE + e] * h[e];
        }
      }
      store_unknowns<R, DOF, Rr>(rr + cols.col[q] * vs + (int64_t)S * (2 * DOF), pl, h,
                                 cols.on[q]);
    }
  }
  if (partials) {
    // over the two parts and the four lane groups of a column, then the waves
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      double s = sum[q];
      s += __shfl_xor(s, 1, 64);
      s += __shfl_xor(s, 16, 64);
      s += __shfl_xor(s, 32, 64);
      if (pl.g == 0 && pl.part == 0) red[wave][q * 8 + pl.kc] = s;
    }
    __syncthreads();
    if ((int)threadIdx.x < CG * 8) {
      const int k = group * CG * 8 + threadIdx.x;
      double s = red[0][threadIdx.x];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) s += red[w][threadIdx.x];
      if (k < nb && (!active || active[k]))
        partials[(int64_t)k * (gridDim.x / groups) + blk] = {s, 0.0};
    }
  }
}

// xc = P^H (b - A x) where the residual of the other colour is zero (x comes from a sweep
// that ended with it): a block per aggregate and 8 CG columns, its waves share the
// aggregate's sites of the given colour, whose residual stays in registers
template <typename T, int DOF, int CG>
__global__ __launch_bounds__(kThreads) void k_bsr8_residual_restrict(
    const T* __restrict__ b, const T* __restrict__ x, T* __restrict__ xc,
    const T* __restrict__ B, const T* __restrict__ Q, int Nc, int blk, int colour, int nb,
    int groups, const int* active) {
  using R = R_t<T>;
  using Acc = typename body::Mfma<R>::acc_t;
  constexpr int NE = Place<R, DOF>::NE, NW = kThreads / 64;
  __shared__ R red[NW][CG * NE][64];
  const int t0 = xcd_block(), group = t0 % groups, agg = t0 / groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const Place<R, DOF> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  if (!cols.live) return;  // the whole block: its waves have the same columns
  const int NcC = Nc / blk, Y0 = agg / NcC * blk, X0 = agg % NcC * blk;
  const int64_t vs = (int64_t)Nc * Nc * (2 * DOF), vc = (int64_t)NcC * NcC * (2 * DOF);
  const R* xr = reinterpret_cast<const R*>(x);
  const R* br = reinterpret_cast<const R*>(b);
  const R* qr = reinterpret_cast<const R*>(Q);
  Acc sum[CG];
#pragma unroll
  for (int q = 0; q < CG; ++q) sum[q] = Acc{0, 0, 0, 0};
  for (int t = wave; t < blk * blk; t += NW) {
    const int yy = t / blk, Y = Y0 + yy, X = X0 + t - yy * blk, S = Y * Nc + X;
    if (((X + Y) & 1) != colour) continue;
    int tn[5];
#pragma unroll
    for (int d = 0; d < 5; ++d) tn[d] = neighbour(X, Y, d, Nc);
    R w[CG * NE], a[NE];
    load_unknowns<R, DOF, CG>(
        [&](int q) { return br + cols.col[q] * vs + (int64_t)S * (2 * DOF); }, pl, w);
#pragma unroll
    for (int e = 0; e < NE; ++e)
      a[e] = qr[(((int64_t)S * DOF + pl.unknown(e)) * DOF + pl.ai) * 2 + pl.ap];
    Acc acc[CG];
    stencil<R, DOF, CG, 0>(acc, reinterpret_cast<const R*>(B), xr, S, tn, vs, pl, cols);
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R h[NE];
      combine<R, NE, false>(acc[q], pl.part, h);
#pragma unroll
      for (int e = 0; e < NE; ++e) sum[q] = body::Mfma<R>::step(a[e], w[q * NE + e] - h[e], sum[q]);
    }
  }
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int q = 0; q < CG; ++q) {
    R h[NE];
    combine<R, NE, true>(sum[q], pl.part, h);
#pragma unroll
    for (int e = 0; e < NE; ++e) red[wave][q * NE + e][lane] = h[e];
  }
  __syncthreads();
  if (wave >= CG) return;
  // wave q finishes column group q
  R h[NE];
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    h[e] = red[0][wave * NE + e][lane];
#pragma unroll
    for (int i = 1; i < NW; ++i) h[e] += red[i][wave * NE + e][lane];
  }
  R* out = reinterpret_cast<R*>(xc);
#pragma unroll
  for (int q = 0; q < CG; ++q)
    if (q == wave)
      store_unknowns<R, DOF, R>(out + cols.col[q] * vc + (int64_t)agg * (2 * DOF), pl, h,
                                cols.on[q]);
}

// xc = P^H (b - D x) from the two-spin lattice, where the residual is zero on the colour
// solved last (colour: the other): a wave per aggregate (blk even) and 8 CG columns.  A
// lane of a pair forms the residual of one site, both spins, and the pair shares them as
// the loads above, so the residual is neither stored nor read.  64^2 sites, 5 complex128
// columns: 4.6 us against 3.1 + 4.0; 256^2 sites, 64 complex64 columns 34 against 31 + 16.
template <typename T, int DOF, int CG>
__global__ __launch_bounds__(kThreads) void k_wilson_residual_restrict(
    const T* __restrict__ b, const T* __restrict__ x, T* __restrict__ xc,
    const T* __restrict__ U, const T* __restrict__ Q, R_t<T> diag, int N, int blk, int colour,
    int nb, int groups, const int* active) {
  using R = R_t<T>;
  using Acc = typename body::Mfma<R>::acc_t;
  constexpr int NE = Place<R, DOF>::NE;
  const int t0 = xcd_block(), group = t0 % groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int Nc = N / blk, S = (t0 / groups) * (kThreads / 64) + wave;
  if (S >= Nc * Nc) return;
  const Place<R, DOF> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  if (!cols.live) return;
  const int Y0 = S / Nc * blk, X0 = S % Nc * blk, hb = blk >> 1, sites = blk * hb;
  const int64_t vf = (int64_t)N * N * 2, vc = (int64_t)Nc * Nc * (2 * DOF);
  const R* qr = reinterpret_cast<const R*>(Q);
  // site t of the colour in the aggregate
  auto site = [&](int t, int& sx, int& sy) {
    const int yy = t / hb;
    sy = Y0 + yy;
    sx = X0 + 2 * (t - yy * hb) + ((colour + yy) & 1);
  };
  Acc acc[CG];
#pragma unroll
  for (int q = 0; q < CG; ++q) acc[q] = Acc{0, 0, 0, 0};
  for (int i0 = 0; i0 < sites; i0 += 8) {  // two items of four sites, one per lane group
    const int mine = i0 + 4 * pl.part + pl.g;
    int sx, sy;
    site(mine < sites ? mine : 0, sx, sy);
    const int s = sy * N + sx;
    T r[CG][2];
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      const T* xk = x + cols.col[q] * vf;
      const T* bk = b + cols.col[q] * vf;
      T h0, h1;
      wil::wilson_hop(xk, U, N, sx, sy, h0, h1);
      const R half = (R)0.5;
      r[q][0] = bk[2 * s] - (diag * xk[2 * s] - half * h0);
      r[q][1] = bk[2 * s + 1] - (diag * xk[2 * s + 1] - half * h1);
    }
    R a[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int t = i0 + 4 * u + pl.g;
      int ux, uy;
      site(t < sites ? t : 0, ux, uy);
#pragma unroll
      for (int e = 0; e < 2; ++e)
        a[u][e] = t < sites ? qr[(((int64_t)(uy * N + ux) * 2 + e) * DOF + pl.ai) * 2 + pl.ap] : (R)0;
    }
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R v[2][2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const T w = mine < sites ? r[q][e] : zero_of(T());
        const R keep = pl.part ? w.im : w.re, got = pair_swap(pl.part ? w.re : w.im);
        v[0][e] = pl.part ? got : keep;
        v[1][e] = pl.part ? keep : got;
      }
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int e = 0; e < 2; ++e) acc[q] = body::Mfma<R>::step(a[u][e], v[u][e], acc[q]);
    }
  }
  R* out = reinterpret_cast<R*>(xc);
#pragma unroll
  for (int q = 0; q < CG; ++q) {
    R h[NE];
    combine<R, NE, true>(acc[q], pl.part, h);
    store_unknowns<R, DOF, R>(out + cols.col[q] * vc + (int64_t)S * (2 * DOF), pl, h, cols.on[q]);
  }
}

// xc = P^H x: a wave per aggregate (blk x blk fine sites of dofF unknowns, rows of
// blk dofF contiguous ones, a multiple of eight) and 8 CG columns
template <typename T, int DOF, int CG>
__global__ __launch_bounds__(kThreads) void k_agg8_restrict(const T* __restrict__ x,
                                                            T* __restrict__ xc,
                                                            const T* __restrict__ q8, int Nf,
                                                            int dofF, int blk, int nb, int groups,
                                                            const int* active) {
  using R = R_t<T>;
  constexpr int NE = Place<R, DOF>::NE;
  constexpr int W = sizeof(R) == 4 ? 2 : 1, KI = 4 * W;  // unknowns an item covers over the groups
  const int t0 = xcd_block(), group = t0 % groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int Nc = Nf / blk, S = (t0 / groups) * (kThreads / 64) + wave;
  if (S >= Nc * Nc) return;
  const Place<R, DOF> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  if (!cols.live) return;
  const int Y = S / Nc, X = S - Y * Nc;
  const int wr = blk * dofF, items = blk * wr / KI, per_row = wr / KI;
  const int64_t vf = (int64_t)Nf * Nf * dofF * 2, vc = (int64_t)Nc * Nc * (2 * DOF);
  const R* xr = reinterpret_cast<const R*>(x);
  const R* qr = reinterpret_cast<const R*>(q8);
  typename body::Mfma<R>::acc_t acc[CG];
#pragma unroll
  for (int c = 0; c < CG; ++c) acc[c] = {0, 0, 0, 0};
  auto first = [&](int item) {  // this lane's first unknown of an item
    const int yy = item / per_row;
    return ((int64_t)(Y * blk + yy) * Nf + X * blk) * dofF + (item - yy * per_row) * KI + W * pl.g;
  };
  auto run = [&](auto n, int item) {
    constexpr int U = decltype(n)::value;
    R a[U * W], v[CG * U * W];
    load_items<R, CG * U, W, false>(
        [&](int u) { return xr + cols.col[u % CG] * vf + first(item + u / CG) * 2; }, pl.part, v);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < W; ++s)
        a[u * W + s] = qr[((first(item + u) + s) * DOF + pl.ai) * 2 + pl.ap];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < W; ++s)
#pragma unroll
        for (int c = 0; c < CG; ++c)
          acc[c] = body::Mfma<R>::step(a[u * W + s], v[(u * CG + c) * W + s], acc[c]);
  };
  constexpr int U = 8 / W;
  int it = 0;
  for (; it + U <= items; it += U) run(std::integral_constant<int, U>(), it);
  for (; it < items; ++it) run(std::integral_constant<int, 1>(), it);
  R* out = reinterpret_cast<R*>(xc);
#pragma unroll
  for (int c = 0; c < CG; ++c) {
    R h[NE];
    combine<R, NE, true>(acc[c], pl.part, h);
    store_unknowns<R, DOF, R>(out + cols.col[c] * vc + (int64_t)S * (2 * DOF), pl, h, cols.on[c]);
  }
}

// ---- dense complex products ------------------------------------------------------
// z = M b per column for the coarsest inverse M (n a multiple of 8): a block per RT
// tiles of 8 rows and 8 CG columns, its sixteen waves share the reduction index in ranges
// of chunks of 16; the partial tiles are summed in wave order.  M comes in the order the
// products need it (pack_dense): 16 bytes per lane and chunk in f32, 32 in f64.
// The real representation this replaces has each entry twice: n = 2048, up to 16
// complex64 columns 12.2 us (64 MB, at the memory's rate), 64 columns 91; now 8.2 (8 columns), 12.3 (16) and
// 60 (64).
constexpr int kDenseWaves = 16, kDenseBlock = kDenseWaves * 64;

// the reduction index of lane group g, step s of chunk c
template <typename R>
__device__ __forceinline__ int dense_k(int c, int g, int s) {
  return sizeof(R) == 4 ? 16 * c + 8 * (s >> 1) + 2 * g + (s & 1) : 16 * c + 4 * s + g;
}

template <typename T, int RT, int CG>
__global__ __launch_bounds__(kDenseBlock) void k_dense_complex(const R_t<T>* __restrict__ M,
                                                               const T* __restrict__ b,
                                                               T* __restrict__ z, int n, int nb,
                                                               const int* active) {
  using R = R_t<T>;
  using Acc = typename body::Mfma<R>::acc_t;
  using V4 = R __attribute__((ext_vector_type(4)));
  constexpr int NE = 2, W = sizeof(R) == 4 ? 2 : 1, NI = 4 / W;
  __shared__ R part[kDenseWaves][NE][64];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const Place<R, 8> pl;
  const Cols<CG> cols(blockIdx.y, pl.kc, nb, active);
  if (!cols.live) return;  // the whole block
  const int tiles = n >> 3, chunks = (n + 15) >> 4;
  const int t0 = blockIdx.x * RT;
  const R* br = reinterpret_cast<const R*>(b);
  const int c0 = wave * chunks / kDenseWaves, c1 = (wave + 1) * chunks / kDenseWaves;
  Acc acc[RT][CG];
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int q = 0; q < CG; ++q) acc[t][q] = Acc{0, 0, 0, 0};
  auto run = [&](auto un, int c) {
    constexpr int U = decltype(un)::value;
    V4 a[U][RT];
    R v[U * CG * 4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < RT; ++t) {
        const int tile = t0 + t < tiles ? t0 + t : t0;
        a[u][t] = *reinterpret_cast<const V4*>(M + (((int64_t)tile * chunks + c + u) * 64 + lane) * 4);
      }
    load_items<R, U * CG * NI, W, false>(
        [&](int i) {
          // beyond n (the last chunk of an odd multiple of 8) M is zero
          const int k = dense_k<R>(c + i / (CG * NI), pl.g, W * (i % NI));
          return br + (cols.col[i / NI % CG] * n + (k < n ? k : 0)) * 2;
        },
        pl.part, v);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < CG; ++q)
#pragma unroll
          for (int t = 0; t < RT; ++t)
            acc[t][q] = body::Mfma<R>::step(a[u][t][s], v[(u * CG + q) * 4 + s], acc[t][q]);
  };
  constexpr int U = RT * CG <= 2 ? 4 : RT * sizeof(R) < 16 ? 2 : 1;
  int c = c0;
  for (; c + U <= c1; c += U) run(std::integral_constant<int, U>(), c);
  for (; c < c1; ++c) run(std::integral_constant<int, 1>(), c);
#pragma unroll
  for (int t = 0; t < RT; ++t)
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R h[NE];
      combine<R, NE, false>(acc[t][q], pl.part, h);
      if (t + q > 0) __syncthreads();
#pragma unroll
      for (int e = 0; e < NE; ++e) part[wave][e][lane] = h[e];
      __syncthreads();
      if (wave == (t * CG + q) % kDenseWaves) {
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          h[e] = part[0][e][lane];
#pragma unroll
          for (int w = 1; w < kDenseWaves; ++w) h[e] += part[w][e][lane];
        }
        store_unknowns<R, 8, R>(reinterpret_cast<R*>(z) + (cols.col[q] * n + 8 * (t0 + t)) * 2, pl,
                                h, cols.on[q] && t0 + t < tiles);
      }
    }
}

// M from the transposed matrix At[j][i]
template <typename T>
__global__ void k_pack_dense(const T* __restrict__ At, R_t<T>* __restrict__ M, int n, int chunks) {
  using R = R_t<T>;
  const Place<R, 8> pl;
  const int c = blockIdx.x, i = 8 * blockIdx.y + pl.ai;
  for (int s = 0; s < 4; ++s) {
    const int k = dense_k<R>(c, pl.g, s);
    R v = 0;
    if (k < n) v = pl.ap ? At[(int64_t)k * n + i].im : At[(int64_t)k * n + i].re;
    M[(((int64_t)blockIdx.y * chunks + c) * 64 + threadIdx.x) * 4 + s] = v;
  }
}

// right-hand sides per wave: 8 for batches up to 8 (the second group would be empty),
// 16 beyond: the blocks, twice the size of a column's site vector times eight, are then
// read half as often
template <typename F>
void with_groups(int nb, F&& f) {
  if (nb <= 8)
    f(std::integral_constant<int, 1>(), (nb + 7) / 8);
  else
    f(std::integral_constant<int, 2>(), (nb + 15) / 16);
}
template <typename F>
void with_form(int dof, int nb, F&& f) {
  with_groups(nb, [&](auto cg, int groups) {
    if (dof == 8)
      f(std::integral_constant<int, 8>(), cg, groups);
    else
      f(std::integral_constant<int, 4>(), cg, groups);
  });
}

// sites per wave of the residual: one without partial sums; with them as many as keep
// the blocks, one partial each, within kMaxPartials
int sites_per_wave(int Nc) {
  int spw = 1;
  while ((Nc * Nc + kThreads / 64 * spw - 1) / (kThreads / 64 * spw) > kMaxPartials) spw *= 2;
  return spw;
}

constexpr int kOneLaunchWaves = 2048;  // two per SIMD

}  // namespace

int bsr8_residual_blocks(int Nc) {
  const int per = kThreads / 64 * sites_per_wave(Nc);
  return (Nc * Nc + per - 1) / per;
}

template <typename T>
void bsr8_rbgs(const T* b, T* x, const T* B, const T* Dinv, int Nc, int dof, int nb,
               const int* active, bool zero_init, bool reverse, hipStream_t s) {
  const int first = reverse ? 1 : 0;
  const T* none = nullptr;
  with_form(dof, nb, [&](auto d, auto cg, int groups) {
    constexpr int CG = decltype(cg)::value, DOF = decltype(d)::value;
    // One launch from zero while its waves (a site and column group each) are all resident:
    // 4.3 us instead of 2.3 + 3.4 on 16^2 sites and 5 complex128 columns.  Beyond, the
    // neighbours' second reading of D^-1 and b costs more than a launch: 64^2 sites, 13
    // complex64 columns 9.5 us against 3 + 4.6, 64 columns 53 against 35.
    if (zero_init && Nc * Nc * groups <= kOneLaunchWaves) {
      MLMC_LAUNCH((k_bsr8_gs<T, DOF, CG, kFromZero>), dim3((unsigned)((Nc * Nc + 3) / 4 * groups)),
                  dim3(kThreads), 0, s, b, x, B, Dinv, none, none, (R_t<T>)0, 1, Nc, first, 0, nb,
                  groups, active, timing_log());
      return;
    }
    const dim3 g((unsigned)((Nc * Nc / 2 + 3) / 4 * groups));
    MLMC_LAUNCH((k_bsr8_gs<T, DOF, CG, kFromX>), g, dim3(kThreads), 0, s, b, x, B, Dinv, none,
                none, (R_t<T>)0, 1, Nc, first, zero_init ? 1 : 0, nb, groups, active,
                timing_log());
    MLMC_LAUNCH((k_bsr8_gs<T, DOF, CG, kFromX>), g, dim3(kThreads), 0, s, b, x, B, Dinv, none,
                none, (R_t<T>)0, 1, Nc, 1 - first, 0, nb, groups, active, (int*)nullptr);
  });
}

template <typename T>
void bsr8_prolong_rbgs(const T* xc, const T* Q, int blk, double omega, const T* b, T* x,
                       const T* B, const T* Dinv, int Nc, int dof, int nb, const int* active,
                       bool reverse, hipStream_t s) {
  const int first = reverse ? 1 : 0;
  with_form(dof, nb, [&](auto d, auto cg, int groups) {
    constexpr int CG = decltype(cg)::value, DOF = decltype(d)::value;
    const dim3 g((unsigned)((Nc * Nc / 2 + 3) / 4 * groups));
    MLMC_LAUNCH((k_bsr8_gs<T, DOF, CG, kFromProlong>), g, dim3(kThreads), 0, s, b, x, B, Dinv, Q,
                xc, (R_t<T>)omega, blk, Nc, first, 0, nb, groups, active, timing_log());
    MLMC_LAUNCH((k_bsr8_gs<T, DOF, CG, kFromX>), g, dim3(kThreads), 0, s, b, x, B, Dinv,
                (const T*)nullptr, (const T*)nullptr, (R_t<T>)0, 1, Nc, 1 - first, 0, nb, groups,
                active, (int*)nullptr);
  });
}

template <typename T, typename Tr>
void bsr8_residual(const T* b, const T* x, Tr* r, const T* B, int Nc, int dof, int nb,
                   const int* active, c64* partials, hipStream_t s) {
  with_form(dof, nb, [&](auto d, auto cg, int groups) {
    constexpr int CG = decltype(cg)::value, DOF = decltype(d)::value;
    const int spw = partials ? sites_per_wave(Nc) : 1, per = kThreads / 64 * spw;
    hipLaunchKernelGGL((k_bsr8_residual<T, Tr, DOF, CG>),
                       dim3((unsigned)((Nc * Nc + per - 1) / per * groups)), dim3(kThreads), 0, s,
                       b, x, r, B, Nc, nb, groups, spw, active, partials);
  });
}

template <typename T>
void bsr8_residual_restrict(const T* b, const T* x, T* xc, const T* B, const T* Q, int Nc, int dof,
                            int blk, int nb, const int* active, bool reverse, hipStream_t s) {
  with_form(dof, nb, [&](auto d, auto cg, int groups) {
    constexpr int CG = decltype(cg)::value, DOF = decltype(d)::value;
    hipLaunchKernelGGL((k_bsr8_residual_restrict<T, DOF, CG>),
                       dim3((unsigned)((Nc / blk) * (Nc / blk) * groups)), dim3(kThreads), 0, s, b,
                       x, xc, B, Q, Nc, blk, reverse ? 1 : 0, nb, groups, active);
  });
}

template <typename T>
void wilson_residual_restrict(const T* b, const T* x, T* xc, const T* U, const T* Q, int N,
                              double diag, int blk, int dofC, int nb, const int* active,
                              bool reverse, hipStream_t s) {
  const int Nc = N / blk;
  with_form(dofC, nb, [&](auto d, auto cg, int groups) {
    constexpr int CG = decltype(cg)::value, DOF = decltype(d)::value;
    hipLaunchKernelGGL((k_wilson_residual_restrict<T, DOF, CG>),
                       dim3((unsigned)((Nc * Nc + 3) / 4 * groups)), dim3(kThreads), 0, s, b, x,
                       xc, U, Q, (R_t<T>)diag, N, blk, reverse ? 1 : 0, nb, groups, active);
  });
}

template <typename T>
void agg8_restrict(const T* x, T* xc, const T* q, int Nf, int dofF, int blk, int dofC, int nb,
                   const int* active, hipStream_t s) {
  const int Nc = Nf / blk;
  with_form(dofC, nb, [&](auto d, auto cg, int groups) {
    constexpr int CG = decltype(cg)::value, DOF = decltype(d)::value;
    hipLaunchKernelGGL((k_agg8_restrict<T, DOF, CG>),
                       dim3((unsigned)((Nc * Nc + 3) / 4 * groups)), dim3(kThreads), 0, s, x, xc,
                       q, Nf, dofF, blk, nb, groups, active);
  });
}

int64_t dense_complex_elems(int n) { return (int64_t)(n / 8) * ((n + 15) / 16) * 256; }

template <typename T>
void dense_complex_pack(const T* At, typename Traits<T>::real* M, int n, hipStream_t s) {
  const int chunks = (n + 15) / 16;
  hipLaunchKernelGGL(k_pack_dense<T>, dim3(chunks, n / 8), dim3(64), 0, s, At, M, n, chunks);
}

template <typename T>
void dense_complex_apply(const typename Traits<T>::real* M, const T* b, T* z, int n, int nb,
                         const int* active, hipStream_t s) {
  const unsigned tiles = (unsigned)(n / 8);
  auto go = [&](auto rt, auto cg) {
    constexpr int RT = decltype(rt)::value, CG = decltype(cg)::value;
    hipLaunchKernelGGL((k_dense_complex<T, RT, CG>), dim3((tiles + RT - 1) / RT, (nb + 8 * CG - 1) / (8 * CG)),
                       dim3(kDenseBlock), 0, s, M, b, z, n, nb, active);
  };
  std::integral_constant<int, 1> one;
  std::integral_constant<int, 2> two;
  std::integral_constant<int, 4> four;
  // as many columns as there are per reading of M, up to 32; beyond, two row tiles per
  // block halve the readings of the columns instead
  if (nb <= 8)
    go(one, one);
  else if (nb <= 16)
    go(one, two);
  else if (nb <= 32 || sizeof(T) == sizeof(c64))  // two tiles spill in f64
    go(one, four);
  else if constexpr (sizeof(T) == sizeof(c32))
    go(two, four);
}

#define BSR8_INST(T)                                                                            \
  template void bsr8_rbgs<T>(const T*, T*, const T*, const T*, int, int, int, const int*, bool,  \
                             bool, hipStream_t);                                                \
  template void bsr8_prolong_rbgs<T>(const T*, const T*, int, double, const T*, T*, const T*,    \
                                     const T*, int, int, int, const int*, bool, hipStream_t);   \
  template void bsr8_residual<T, T>(const T*, const T*, T*, const T*, int, int, int, const int*, \
                                    c64*, hipStream_t);                                         \
  template void bsr8_residual_restrict<T>(const T*, const T*, T*, const T*, const T*, int, int,  \
                                          int, int, const int*, bool, hipStream_t);             \
  template void wilson_residual_restrict<T>(const T*, const T*, T*, const T*, const T*, int,     \
                                            double, int, int, int, const int*, bool,            \
                                            hipStream_t);                                       \
  template void agg8_restrict<T>(const T*, T*, const T*, int, int, int, int, int, const int*,    \
                                 hipStream_t);                                                  \
  template void dense_complex_pack<T>(const T*, Traits<T>::real*, int, hipStream_t);             \
  template void dense_complex_apply<T>(const Traits<T>::real*, const T*, T*, int, int,           \
                                       const int*, hipStream_t);
BSR8_INST(c32)
BSR8_INST(c64)
template void bsr8_residual<c64, c32>(const c64*, const c64*, c32*, const c64*, int, int, int,
                                      const int*, c64*, hipStream_t);

}  // namespace mlmc
