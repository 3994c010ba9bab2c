// Block stencils and aggregation restriction with eight complex unknowns per coarse
// site on the matrix cores (v_mfma_{f32,f64}_16x16x4).
//
// A block row is an 8 x 8 complex block per neighbour.  Its real and imaginary parts
// are stacked as the 16 rows of the A operand and eight right-hand sides, real and
// imaginary parts next to each other, are the 16 columns of the B operand: one
// product gives A_re x_re, A_re x_im, A_im x_re and A_im x_im without the doubled
// matrix of a real representation, and the complex result is a sum of two
// accumulators of neighbouring lanes.  The rows are ordered so that a lane's four
// accumulators are the real and imaginary rows of two unknowns:
//   f32 (accumulator r of lane group g is row 4 g + r): row 2 i + p,
//   f64 (row 4 r + g):                                   row i + 8 p,
// p = 0 real, 1 imaginary, so after the sum lane group g holds the unknowns 2 g, 2 g + 1
// (f32) or g, g + 4 (f64), which is the B operand of the next product (the inverted
// diagonal block) without moving data.
//
// One wave serves a site and 8 or 16 right-hand sides, so the site's blocks are read
// once for all of them, and all loads of the neighbour products are issued before the
// first product.  Narrow batches are bound by that load latency (one launch of a 16^2
// level costs about 3 us whatever it does), wide ones by L2 traffic.  Each column is
// its own vector, 64 or 128 bytes per site at a stride of a whole vector: loads of one
// value per lane left half of every 64-byte run to a second instruction and made wide
// batches slower than one thread per row (a colour of 64^2 sites and 64 columns: 46 us
// the residual), 16-byte loads shared by lane pairs 16 us.
// Measured on the 256^2 two-spin trace (complex64, batches of 1 to 64 columns) against
// one thread per row and column: sweeps 52 -> 33 ms, residuals 21.5 -> 11.5, restriction
// 17.7 -> 6.8; complex128 on 64^2, 5 columns: sweep 6.9 -> 3.4 us, restriction 12 -> 5.
#include "kernels.h"
#include "vec_body.h"

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
template <typename R>
struct Place {
  int g, kc, part, ai, ap;
  __device__ Place() {
    const int lane = threadIdx.x & 63, m = lane & 15;
    g = lane >> 4;
    kc = m >> 1;
    part = m & 1;
    ai = sizeof(R) == 4 ? m >> 1 : m & 7;
    ap = sizeof(R) == 4 ? m & 1 : m >> 3;
  }
  __device__ int unknown(int e) const { return sizeof(R) == 4 ? 2 * g + e : g + 4 * e; }
};

// the complex products of this lane's unknowns (conj: of the conjugated A)
template <typename R, bool CONJ, typename Acc>
__device__ __forceinline__ void combine(const Acc& acc, int part, R* out) {
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const R re = sizeof(R) == 4 ? acc[2 * e] : acc[e];
    const R t = pair_swap(sizeof(R) == 4 ? acc[2 * e + 1] : acc[e + 2]);
    out[e] = ((part != 0) != CONJ) ? re + t : re - t;
  }
}

// Sixteen-byte loads: an item is 16 bytes of consecutive complex values (two in f32,
// one in f64) of which this lane wants one part each.  Of two items each lane of a
// pair loads one and hands the other lane its part, so a wave reads whole 64-byte
// runs with a quarter (f32) or half (f64) of the load instructions.
template <typename R>
struct Item;
template <>
struct Item<float> {
  static constexpr int W = 2;
  using vec = float __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct Item<double> {
  static constexpr int W = 1;
  using vec = double __attribute__((ext_vector_type(2), aligned(8)));
};

// out[W u + s] = part-th component of value s of item u at ptr(u); AROW: pairs of the
// A operand's rows, else of the B operand's columns
template <typename R, int N, bool AROW, typename P>
__device__ __forceinline__ void load_items(P ptr, int part, R* out) {
  constexpr int W = Item<R>::W;
  typename Item<R>::vec v[N / 2 + 1];
#pragma unroll
  for (int h = 0; h < N / 2; ++h) {
    const R *p0 = ptr(2 * h), *p1 = ptr(2 * h + 1);
    v[h] = *reinterpret_cast<const typename Item<R>::vec*>(part ? p1 : p0);
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

// this lane's two unknowns of N columns' site vectors (at(q): the site's 16 reals)
template <typename R, int N, typename P>
__device__ __forceinline__ void load_unknowns(P at, const Place<R>& pl, R* out) {
  if (sizeof(R) == 4)
    load_items<R, N, false>([&](int u) { return at(u) + 4 * pl.g; }, pl.part, out);
  else
    load_items<R, 2 * N, false>([&](int u) { return at(u >> 1) + 2 * (pl.g + 4 * (u & 1)); },
                                pl.part, out);
}

// the same back: each lane of a pair stores one whole unknown
template <typename R, typename Ro>
__device__ __forceinline__ void store_unknowns(Ro* at, const Place<R>& pl, const R* out, bool on) {
  using V = Ro __attribute__((ext_vector_type(2), aligned(sizeof(Ro))));
  const R keep = pl.part ? out[1] : out[0];
  const R got = pair_swap(pl.part ? out[0] : out[1]);
  V v;
  v[0] = (Ro)(pl.part ? got : keep);
  v[1] = (Ro)(pl.part ? keep : got);
  if (on) *reinterpret_cast<V*>(at + 2 * pl.unknown(pl.part)) = v;
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
    live = __any(any);
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

// acc[q] = sum over the directions D0 .. 4 of block d times the neighbour's vector;
// k runs over the two consecutive unknowns 2 g, 2 g + 1 of a lane group
template <typename T, int CG, int D0, typename Acc>
__device__ __forceinline__ void stencil(Acc (&acc)[CG], const R_t<T>* __restrict__ B,
                                        const R_t<T>* x, int S, int X, int Y, int Nc,
                                        const Place<R_t<T>>& pl, const Cols<CG>& cols) {
  using R = R_t<T>;
  constexpr int ND = 5 - D0, IP = 2 / Item<R>::W;  // items per (block, lane)
  const int64_t vs = (int64_t)Nc * Nc * 16;        // reals per column
  R a[2 * ND], v[CG * 2 * ND];
  int tn[ND];
#pragma unroll
  for (int d = 0; d < ND; ++d) tn[d] = neighbour(X, Y, D0 + d, Nc);
  load_items<R, CG * ND * IP, false>(
      [&](int u) {
        // the pairs are the two column groups (CG 2) or neighbours, and values in f64
        const int q = IP == 2 ? u / (2 * ND) : u % CG, d = IP == 2 ? (u / 2) % ND : u / CG;
        return x + cols.col[q] * vs + (int64_t)tn[d] * 16 + 4 * pl.g + (IP == 2 ? 2 * (u & 1) : 0);
      },
      pl.part, v);
  load_items<R, ND * IP, true>(
      [&](int u) {
        const int d = u / IP;
        return B + (((int64_t)S * 5 + D0 + d) * 64 + pl.ai * 8 + 2 * pl.g + (IP == 2 ? u & 1 : 0)) * 2;
      },
      pl.ap, a);
#pragma unroll
  for (int q = 0; q < CG; ++q) acc[q] = Acc{0, 0, 0, 0};
#pragma unroll
  for (int d = 0; d < ND; ++d)
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int q = 0; q < CG; ++q)
        acc[q] = body::Mfma<R>::step(a[2 * d + s],
                                     v[IP == 2 ? (q * ND + d) * 2 + s : (d * CG + q) * 2 + s], acc[q]);
}

// one colour of a red-black block Gauss-Seidel sweep, in place:
// x_S = Dinv_S (b_S - sum_{d != self} B[S][d] x_nbr)
template <typename T, int CG>
__global__ __launch_bounds__(kThreads) void k_bsr8_gs(const T* __restrict__ b, T* x,
                                                      const T* __restrict__ B,
                                                      const T* __restrict__ Dinv, int Nc,
                                                      int colour, int zero_nbrs, int nb,
                                                      int groups, const int* active, int* tlog) {
  using R = R_t<T>;
  const int t0 = xcd_block(), group = t0 % groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (tlog && t0 < groups && threadIdx.x < 8 * CG && group * 8 * CG + (int)threadIdx.x < nb)
    tlog[group * 8 * CG + threadIdx.x] = active ? active[group * 8 * CG + threadIdx.x] : 1;
  const int t = (t0 / groups) * (kThreads / 64) + wave;
  const int hc = Nc >> 1;
  if (t >= Nc * hc) return;
  const Place<R> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  if (!cols.live) return;
  const int Y = t / hc, X = 2 * (t - Y * hc) + ((colour + Y) & 1), S = Y * Nc + X;
  const int64_t vs = (int64_t)Nc * Nc * 16;
  const R* br = reinterpret_cast<const R*>(b);
  R* xr = reinterpret_cast<R*>(x);
  const R* Dr = reinterpret_cast<const R*>(Dinv);
  R rhs[2 * CG], a2[2];
#pragma unroll
  for (int e = 0; e < 2; ++e)
    a2[e] = Dr[((int64_t)S * 64 + pl.ai * 8 + pl.unknown(e)) * 2 + pl.ap];
  load_unknowns<R, CG>([&](int q) { return br + cols.col[q] * vs + (int64_t)S * 16; }, pl, rhs);
  typename body::Mfma<R>::acc_t acc[CG];
  if (!zero_nbrs) {
    stencil<T, CG, 1>(acc, reinterpret_cast<const R*>(B), xr, S, X, Y, Nc, pl, cols);
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R h[2];
      combine<R, false>(acc[q], pl.part, h);
      rhs[2 * q] -= h[0];
      rhs[2 * q + 1] -= h[1];
    }
  }
#pragma unroll
  for (int q = 0; q < CG; ++q) {
    typename body::Mfma<R>::acc_t o = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 2; ++e) o = body::Mfma<R>::step(a2[e], rhs[2 * q + e], o);
    R out[2];
    combine<R, false>(o, pl.part, out);
    store_unknowns<R, R>(xr + cols.col[q] * vs + (int64_t)S * 16, pl, out, cols.on[q]);
  }
}

// r = b - A x (b == nullptr: r = A x); spw sites per wave; partials (nullable) of
// |r|^2 (or Re conj(x)^T A x) per column and block
template <typename T, typename Tr, int CG>
__global__ __launch_bounds__(kThreads) void k_bsr8_residual(const T* __restrict__ b,
                                                            const T* __restrict__ x,
                                                            Tr* __restrict__ r,
                                                            const T* __restrict__ B, int Nc,
                                                            int nb, int groups, int spw,
                                                            const int* active, c64* partials) {
  using R = R_t<T>;
  using Rr = R_t<Tr>;
  __shared__ double red[kThreads / 64][CG * 8];
  const int t0 = xcd_block(), group = t0 % groups, blk = t0 / groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int ns = Nc * Nc;
  const Place<R> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  const int64_t vs = (int64_t)ns * 16;
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
    R w[2 * CG];
    if (b || partials)
      load_unknowns<R, CG>(
          [&](int q) {
            const int64_t at = cols.col[q] * vs + (int64_t)S * 16;
            return b ? br + at : xr + at;
          },
          pl, w);
    typename body::Mfma<R>::acc_t acc[CG];
    stencil<T, CG, 0>(acc, reinterpret_cast<const R*>(B), xr, S, X, Y, Nc, pl, cols);
#pragma unroll
    for (int q = 0; q < CG; ++q) {
      R h[2];
      combine<R, false>(acc[q], pl.part, h);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        if (b) {
          h[e] = w[2 * q + e] - h[e];
          sum[q] += (double)h[e] * h[e];
        } else if (partials) {
          sum[q] += (double)w[2 * q + e] * h[e];
        }
      }
      store_unknowns<R, Rr>(rr + cols.col[q] * vs + (int64_t)S * 16, pl, h, cols.on[q]);
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

// xc = P^H x: a wave per aggregate (blk x blk fine sites of dofF unknowns, rows of
// blk dofF contiguous ones, a multiple of eight) and 8 CG columns
template <typename T, int CG>
__global__ __launch_bounds__(kThreads) void k_agg8_restrict(const T* __restrict__ x,
                                                            T* __restrict__ xc,
                                                            const T* __restrict__ q8, int Nf,
                                                            int dofF, int blk, int nb, int groups,
                                                            const int* active) {
  using R = R_t<T>;
  constexpr int W = Item<R>::W, KI = 4 * W;  // unknowns an item covers over the groups
  const int t0 = xcd_block(), group = t0 % groups;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int Nc = Nf / blk, S = (t0 / groups) * (kThreads / 64) + wave;
  if (S >= Nc * Nc) return;
  const Place<R> pl;
  const Cols<CG> cols(group, pl.kc, nb, active);
  if (!cols.live) return;
  const int Y = S / Nc, X = S - Y * Nc;
  const int wr = blk * dofF, items = blk * wr / KI, per_row = wr / KI;
  const int64_t vf = (int64_t)Nf * Nf * dofF * 2, vc = (int64_t)Nc * Nc * 16;
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
    load_items<R, CG * U, false>(
        [&](int u) { return xr + cols.col[u % CG] * vf + first(item + u / CG) * 2; }, pl.part, v);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int s = 0; s < W; ++s)
        a[u * W + s] = qr[((first(item + u) + s) * 8 + pl.ai) * 2 + pl.ap];
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
    R h[2];
    combine<R, true>(acc[c], pl.part, h);
    store_unknowns<R, R>(out + cols.col[c] * vc + (int64_t)S * 16, pl, h, cols.on[c]);
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

// sites per wave of the residual: one without partial sums; with them as many as keep
// the blocks, one partial each, within kMaxPartials
int sites_per_wave(int Nc) {
  int spw = 1;
  while ((Nc * Nc + kThreads / 64 * spw - 1) / (kThreads / 64 * spw) > kMaxPartials) spw *= 2;
  return spw;
}

}  // namespace

int bsr8_residual_blocks(int Nc) {
  const int per = kThreads / 64 * sites_per_wave(Nc);
  return (Nc * Nc + per - 1) / per;
}

template <typename T>
void bsr8_rbgs(const T* b, T* x, const T* B, const T* Dinv, int Nc, int nb, const int* active,
               bool zero_init, bool reverse, hipStream_t s) {
  const int first = reverse ? 1 : 0;
  with_groups(nb, [&](auto cg, int groups) {
    constexpr int CG = decltype(cg)::value;
    const dim3 g((unsigned)((Nc * Nc / 2 + 3) / 4 * groups));
    MLMC_LAUNCH((k_bsr8_gs<T, CG>), g, dim3(kThreads), 0, s, b, x, B, Dinv, Nc, first,
                zero_init ? 1 : 0, nb, groups, active, timing_log());
    MLMC_LAUNCH((k_bsr8_gs<T, CG>), g, dim3(kThreads), 0, s, b, x, B, Dinv, Nc, 1 - first, 0, nb,
                groups, active, (int*)nullptr);
  });
}

template <typename T, typename Tr>
void bsr8_residual(const T* b, const T* x, Tr* r, const T* B, int Nc, int nb, const int* active,
                   c64* partials, hipStream_t s) {
  with_groups(nb, [&](auto cg, int groups) {
    constexpr int CG = decltype(cg)::value;
    const int spw = partials ? sites_per_wave(Nc) : 1, per = kThreads / 64 * spw;
    hipLaunchKernelGGL((k_bsr8_residual<T, Tr, CG>), dim3((unsigned)((Nc * Nc + per - 1) / per * groups)),
                       dim3(kThreads), 0, s, b, x, r, B, Nc, nb, groups, spw, active, partials);
  });
}

template <typename T>
void agg8_restrict(const T* x, T* xc, const T* q, int Nf, int dofF, int blk, int nb,
                   const int* active, hipStream_t s) {
  const int Nc = Nf / blk;
  with_groups(nb, [&](auto cg, int groups) {
    constexpr int CG = decltype(cg)::value;
    hipLaunchKernelGGL((k_agg8_restrict<T, CG>), dim3((unsigned)((Nc * Nc + 3) / 4 * groups)),
                       dim3(kThreads), 0, s, x, xc, q, Nf, dofF, blk, nb, groups, active);
  });
}

#define BSR8_INST(T)                                                                            \
  template void bsr8_rbgs<T>(const T*, T*, const T*, const T*, int, int, const int*, bool, bool, \
                             hipStream_t);                                                      \
  template void bsr8_residual<T, T>(const T*, const T*, T*, const T*, int, int, const int*,   \
                                       c64*, hipStream_t);                                      \
  template void agg8_restrict<T>(const T*, T*, const T*, int, int, int, int, const int*,         \
                                 hipStream_t);
BSR8_INST(c32)
BSR8_INST(c64)
template void bsr8_residual<c64, c32>(const c64*, const c64*, c32*, const c64*, int, int,
                                           const int*, c64*, hipStream_t);

}  // namespace mlmc
