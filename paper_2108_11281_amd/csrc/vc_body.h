// Device bodies of the 3D 7-point variable-coefficient stencil kernels.  Each
// body takes its block index (and, where a workgroup runs more than one block,
// its thread index) as arguments, so that the one-problem launches and the
// grouped and persistent launches over several problems run the same
// operations in the same order and give identical results.
#pragma once

#include "common.h"
#include "lanes.h"

namespace mlmc {
namespace vcb {

template <typename T> using R_t = typename Traits<T>::real;
constexpr int kNT = 256;  // threads of a (virtual) block of the cell-parallel bodies

// Stencil kernels read the level's couplings in a cell-major layout:
// kl[d][i] = coefficient of the face below cell i in direction d (x, y, z),
// zero on the boundary, each of the three arrays padded with N^2 zeros, so that
// the six couplings of cell i are kl[0][i], kl[0][i+1], kl[1][i], kl[1][i+N],
// kl[2][i], kl[2][i+N^2] -- coalesced and branch-free.  Neighbour loads use
// clamped indices (their coupling is zero wherever the clamp acts).  A thread
// serves COLS right-hand sides, so the couplings are loaded once per COLS
// columns.
template <typename R>
struct Couplings {
  R cx0, cx1, cy0, cy1, cz0, cz1, d;
  int64_t im1, ip1, imN, ipN, imNN, ipNN;
};

template <typename R>
__device__ __forceinline__ Couplings<R> couplings(const R* __restrict__ kl,
                                                  const R* __restrict__ dg, int64_t i, int N) {
  const int64_t n = (int64_t)N * N * N, NN = (int64_t)N * N, stride = n + NN;
  Couplings<R> c;
  c.cx0 = kl[i];
  c.cx1 = kl[i + 1];
  c.cy0 = kl[stride + i];
  c.cy1 = kl[stride + i + N];
  c.cz0 = kl[2 * stride + i];
  c.cz1 = kl[2 * stride + i + NN];
  c.d = dg[i];
  c.im1 = i > 0 ? i - 1 : 0;
  c.ip1 = i + 1 < n ? i + 1 : n - 1;
  c.imN = i >= N ? i - N : 0;
  c.ipN = i + N < n ? i + N : n - 1;
  c.imNN = i >= NN ? i - NN : 0;
  c.ipNN = i + NN < n ? i + NN : n - 1;
  return c;
}

// coupling times neighbour value, selected (not multiplied) to zero where the
// coupling is zero: a clamped index may point at a cell that the current sweep
// has not written yet, whose stale contents need not be finite
template <typename T, typename R>
__device__ __forceinline__ T term(R cf, T v) {
  return cf != (R)0 ? cf * v : zero_of(T());
}

// sum of the six couplings times the neighbours of u (one column)
template <typename T, typename R>
__device__ __forceinline__ T nbr_sum(const T* __restrict__ u, const Couplings<R>& c) {
  return term(c.cx0, u[c.im1]) + term(c.cx1, u[c.ip1]) + term(c.cy0, u[c.imN]) +
         term(c.cy1, u[c.ipN]) + term(c.cz0, u[c.imNN]) + term(c.cz1, u[c.ipNN]);
}

__device__ __forceinline__ bool col_on(const int* active, int col, int nb) {
  return col < nb && (!active || active[col]);
}

// wave sums, then the waves' sums in wave order by thread 0 (the kernels'
// block_sum2 for blocks of kNT threads)
__device__ __forceinline__ void bsum2(double& a, double& b, double* lds) {
  block_sum2<kNT>(a, b, lds);
}

// r = b - A x (or r = A x when b is null); partials: per column and block of
// |r|^2 (or conj(x)^T r).  Block (bx, by) of a grid with nblk blocks of kNT
// cells; COLS columns from by * COLS.
template <typename Tb, typename T, typename Tr, int COLS>
__device__ __forceinline__ void vc_residual(const Tb* __restrict__ b, const T* __restrict__ x,
                                            Tr* __restrict__ r, const R_t<T>* __restrict__ kl,
                                            const R_t<T>* __restrict__ dg, int N, int nb,
                                            const int* active, c64* partials, int* tlog, int bx,
                                            int by, int nblk, double* red) {
  const int col0 = by * COLS;
  if (tlog && bx == 0 && threadIdx.x < COLS && col0 + (int)threadIdx.x < nb)
    tlog[col0 + threadIdx.x] = active ? active[col0 + threadIdx.x] : 1;
  const int64_t n = (int64_t)N * N * N;
  const int64_t i = (int64_t)bx * kNT + threadIdx.x;
  const bool in = i < n;
  Couplings<R_t<T>> c = couplings(kl, dg, in ? i : 0, N);
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    const int col = col0 + q;
    if (!col_on(active, col, nb)) continue;  // uniform over the block
    const int64_t off = (int64_t)col * n;
    double dre = 0.0, dim = 0.0;
    if (in) {
      const T* xc = x + off;
      T v = c.d * xc[i] - nbr_sum(xc, c);
      if (b) {
        v = convert<T, Tb>(b[off + i]) - v;
        cdot_acc(dre, dim, v, v);
      } else {
        cdot_acc(dre, dim, xc[i], v);
      }
      r[off + i] = convert<Tr, T>(v);
    }
    if (partials) {
      bsum2(dre, dim, red);
      if (threadIdx.x == 0) partials[(int64_t)col * nblk + bx] = {dre, dim};
    }
  }
}

// p_new = z + beta p_old ; q = A p_new ; partials of conj(p_new)^T q.  The
// neighbours' p_new values are recomputed from z and p_old, so the update and
// the operator need a single pass.  Block (bx, by) as in vc_residual.
template <typename T, int COLS>
__device__ __forceinline__ void vc_update_apply(const T* __restrict__ p_old,
                                                const T* __restrict__ z,
                                                const c64* __restrict__ beta,
                                                T* __restrict__ p_new, T* __restrict__ q,
                                                const R_t<T>* __restrict__ kl,
                                                const R_t<T>* __restrict__ dg, int N, int nb,
                                                const int* active, c64* partials, int* tlog,
                                                int bx, int by, int nblk, double* red) {
  const int col0 = by * COLS;
  if (tlog && bx == 0 && threadIdx.x < COLS && col0 + (int)threadIdx.x < nb)
    tlog[col0 + threadIdx.x] = active ? active[col0 + threadIdx.x] : 1;
  const int64_t n = (int64_t)N * N * N;
  const int64_t i = (int64_t)bx * kNT + threadIdx.x;
  const bool in = i < n;
  Couplings<R_t<T>> c = couplings(kl, dg, in ? i : 0, N);
#pragma unroll
  for (int qq = 0; qq < COLS; ++qq) {
    const int col = col0 + qq;
    if (!col_on(active, col, nb)) continue;
    const int64_t off = (int64_t)col * n;
    const R_t<T> bt = (R_t<T>)beta[col].re;
    const T* zc = z + off;
    const T* pc = p_old + off;
    double dre = 0.0, dim = 0.0;
    if (in) {
      auto P = [&](int64_t j) { return zc[j] + bt * pc[j]; };
      const T pi = P(i);
      const T s = term(c.cx0, P(c.im1)) + term(c.cx1, P(c.ip1)) + term(c.cy0, P(c.imN)) +
                  term(c.cy1, P(c.ipN)) + term(c.cz0, P(c.imNN)) + term(c.cz1, P(c.ipNN));
      const T qv = c.d * pi - s;
      p_new[off + i] = pi;
      q[off + i] = qv;
      cdot_acc(dre, dim, pi, qv);
    }
    bsum2(dre, dim, red);
    if (threadIdx.x == 0) partials[(int64_t)col * nblk + bx] = {dre, dim};
  }
}

// rc = R (b - A x) for 2x2x2 aggregates (1/sqrt(8)): coarse cell
// I = bx * NT + tid (a thread per coarse cell, no barrier), COLS columns from
// by * COLS.  HALF: x has just left a forward sweep, so the residual is zero on the
// second colour and only the first colour's four cells are formed (96^3, 32 FP32
// columns: 97 us instead of 109, 56^3 33 instead of 41)
template <typename T, int COLS, int NT, bool HALF>
__device__ __forceinline__ void vc_res_restrict(const T* __restrict__ b, const T* __restrict__ x,
                                                T* __restrict__ rc,
                                                const R_t<T>* __restrict__ kl,
                                                const R_t<T>* __restrict__ dg, int N, int nb,
                                                const int* active, int* tlog, int bx, int by,
                                                int tid) {
  using R = R_t<T>;
  const int col0 = by * COLS;
  if (tlog && bx == 0 && tid < COLS && col0 + tid < nb)
    tlog[col0 + tid] = active ? active[col0 + tid] : 1;
  const int Nc = N >> 1;
  const int nc = Nc * Nc * Nc;
  const int I = bx * NT + tid;
  if (I >= nc) return;
  const int Z = I / (Nc * Nc);
  const int rem = I - Z * Nc * Nc;
  const int Y = rem / Nc, X = rem - Y * Nc;
  const int x0 = 2 * X;
  const int NN = N * N;
  const int64_t n = (int64_t)NN * N, stride = n + NN;
  const T zero = zero_of(T());
  T acc[COLS];
#pragma unroll
  for (int q = 0; q < COLS; ++q) acc[q] = zero;
#pragma unroll
  for (int dz = 0; dz < 2; ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy) {
      const int y = 2 * Y + dy, z = 2 * Z + dz;
      const int64_t i = ((int64_t)z * N + y) * N + x0;
      // couplings of the pair (faces below each cell and the ones above, which
      // are the faces below the next cells; zero on the boundary, padded)
      const R kx0 = kl[i], kx1 = kl[i + 1], kx2 = kl[i + 2];
      const R ky0 = kl[stride + i], ky1 = kl[stride + i + 1];
      const R kyu0 = kl[stride + i + N], kyu1 = kl[stride + i + N + 1];
      const R kz0 = kl[2 * stride + i], kz1 = kl[2 * stride + i + 1];
      const R kzu0 = kl[2 * stride + i + NN], kzu1 = kl[2 * stride + i + NN + 1];
      const R d0 = dg[i], d1 = dg[i + 1];
      const bool xl_in = x0 > 0, xr_in = x0 + 2 < N;
      const bool yl_in = y > 0, yu_in = y + 1 < N, zl_in = z > 0, zu_in = z + 1 < N;
#pragma unroll
      for (int q = 0; q < COLS; ++q) {
        const int col = col0 + q;
        if (!col_on(active, col, nb)) continue;  // uniform over the block
        const T* xc = x + (int64_t)col * n;
        const T* bc = b + (int64_t)col * n;
        if constexpr (HALF) {
          if ((dy + dz) % 2 == 0) {
            const T xl = xl_in ? xc[i - 1] : zero, yl = yl_in ? xc[i - N] : zero,
                    yu = yu_in ? xc[i + N] : zero, zl = zl_in ? xc[i - NN] : zero,
                    zu = zu_in ? xc[i + NN] : zero;
            acc[q] += bc[i] - (d0 * xc[i] - (kx0 * xl + kx1 * xc[i + 1] + ky0 * yl + kyu0 * yu +
                                             kz0 * zl + kzu0 * zu));
          } else {
            const T xr = xr_in ? xc[i + 2] : zero, yl = yl_in ? xc[i - N + 1] : zero,
                    yu = yu_in ? xc[i + N + 1] : zero, zl = zl_in ? xc[i - NN + 1] : zero,
                    zu = zu_in ? xc[i + NN + 1] : zero;
            acc[q] += bc[i + 1] - (d1 * xc[i + 1] - (kx1 * xc[i] + kx2 * xr + ky1 * yl +
                                                     kyu1 * yu + kz1 * zl + kzu1 * zu));
          }
          continue;
        }
        const T c0 = xc[i], c1 = xc[i + 1];
        const T xl = xl_in ? xc[i - 1] : zero, xr = xr_in ? xc[i + 2] : zero;
        const T yl0 = yl_in ? xc[i - N] : zero, yl1 = yl_in ? xc[i - N + 1] : zero;
        const T yu0 = yu_in ? xc[i + N] : zero, yu1 = yu_in ? xc[i + N + 1] : zero;
        const T zl0 = zl_in ? xc[i - NN] : zero, zl1 = zl_in ? xc[i - NN + 1] : zero;
        const T zu0 = zu_in ? xc[i + NN] : zero, zu1 = zu_in ? xc[i + NN + 1] : zero;
        const T r0 = bc[i] - (d0 * c0 - (kx0 * xl + kx1 * c1 + ky0 * yl0 + kyu0 * yu0 +
                                          kz0 * zl0 + kzu0 * zu0));
        const T r1 = bc[i + 1] - (d1 * c1 - (kx1 * c0 + kx2 * xr + ky1 * yl1 + kyu1 * yu1 +
                                              kz1 * zl1 + kzu1 * zu1));
        acc[q] += r0;
        acc[q] += r1;
      }
    }
#pragma unroll
  for (int q = 0; q < COLS; ++q) {
    const int col = col0 + q;
    if (!col_on(active, col, nb)) continue;
    rc[(int64_t)col * nc + I] = (R)0.35355339059327373 * acc[q];  // 1/sqrt(8)
  }
}

// ---------------------------------------------------------------------------
// One fused red-black sweep, out of place, marching along z:
//   x_out = S(x_in + ws * P ec ; b)      (ws = omega / sqrt(8); F = first colour)
// A workgroup of 8 waves owns TY = 8 RPW - 2 consecutive rows y0 .. y0+TY-1
// of COLS right-hand sides and walks a segment of SZ planes.  It holds the
// rows y0-1 .. y0+TY as lane pairs (x = 2*pl, 2*pl+1), RPW rows per wave of
// 64/RPW lanes each (2*64/RPW >= N, so a row needs no x halo; a wave's rows
// have one parity), with five planes of each row in registers.  At step p a
// wave loads plane p+2, updates the first colour on plane p and the second
// colour on plane p-1, and writes plane p-1 (owned rows).  In a row both
// updates of a step hit the same element of the pair, and the y-neighbours each
// needs are one value per lane of the rows above and below: the rows swap them
// through LDS (double-buffered, one barrier per step); the two outermost rows
// also load the row beyond them.  Cells outside the grid read as zero, so no
// coupling ever multiplies a value that was not written.
// ---------------------------------------------------------------------------
// Bound by vector instructions: with register moves, 64-bit addresses and two divisions
// per step 96^3 cells and 32 FP32 columns took 131 us from zero and 181 us after a coarse
// correction; with the ring of slots, plane pointers in scalar registers and stored
// reciprocals 105 and 147.
// couplings of a row pair on one plane; d0, d1 hold 1 / diagonal
template <typename R>
struct PlaneK {
  R kx0, kx1, kyl0, kyl1, kyu0, kyu1, kz0, kz1, d0, d1;
};

constexpr int kMarchWaves = 8;

// LDS elements of vc_march<T, COLS, RPW, ...>
template <typename T, int COLS, int RPW>
__host__ __device__ constexpr int vc_march_lds() {
  return 2 * 2 * (kMarchWaves * RPW) * COLS * (64 / RPW);
}

template <typename T, int COLS, int RPW, bool HX, bool HE, int F>
__device__ __forceinline__ void vc_march(const T* __restrict__ xin, const T* __restrict__ b,
                                         T* __restrict__ xout, const T* __restrict__ ec,
                                         R_t<T> ws, const R_t<T>* __restrict__ kl,
                                         const R_t<T>* __restrict__ dg, int N, int SZ, int nb,
                                         const int* active, int* tlog, int bx, int by, int bz,
                                         T* lds) {
  using R = R_t<T>;
  constexpr int RW = kMarchWaves * RPW;  // rows held, incl. one halo row each side
  constexpr int TY = RW - 2;             // rows owned
  constexpr int LPR = 64 / RPW;          // lanes (pairs) per row
  // a row's second-colour cell at plane p (x_in) and first-colour cell at
  // plane p-1 (updated): vc_march_lds<T, COLS, RPW>() elements of LDS
  T (*xa)[RW][COLS][LPR] = reinterpret_cast<T (*)[RW][COLS][LPR]>(lds);
  T (*xb)[RW][COLS][LPR] = reinterpret_cast<T (*)[RW][COLS][LPR]>(lds + 2 * RW * COLS * LPR);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int col0 = by * COLS;
  if (tlog && bx == 0 && bz == 0 && threadIdx.x < COLS &&
      col0 + (int)threadIdx.x < nb)
    tlog[col0 + threadIdx.x] = active ? active[col0 + threadIdx.x] : 1;
  bool con[COLS];
  bool any = false;
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    con[c] = col_on(active, col0 + c, nb);
    any = any || con[c];
  }
  if (!any) return;  // uniform over the workgroup
  const int seg = lane / LPR, pl = lane - seg * LPR;
  // row slot: wave w holds slots of parity w & 1 (so e below is wave-uniform)
  const int r = (w & 1) + 2 * (seg + RPW * (w >> 1));
  const int y = bx * TY - 1 + r;
  // a row of the wave's parity (uniform; y has this parity in every lane)
  const int ybase = __builtin_amdgcn_readfirstlane((int)(bx * TY - 1 + (w & 1)));
  const int x0 = 2 * pl;
  const bool xok = x0 < N;
  const bool row_in = y >= 0 && y < N;
  const bool edge = (r == 0) || (r == RW - 1);
  const int ye = (r == 0) ? y - 1 : y + 1;  // the outermost rows' outer neighbour row
  const bool eok = edge && ye >= 0 && ye < N;
  const bool inner = r >= 1 && r <= TY;
  const bool store = inner && row_in && xok;
  const bool has_r = x0 + 2 < N;
  const int NN = N * N;
  const int64_t n = (int64_t)NN * N, stride = n + NN;
  const int Nc = N >> 1;
  const T zero = zero_of(T());

  // Per-lane byte offsets within a plane, from uniform plane pointers: the loads take
  // them as they are.  Lanes outside the grid load the nearest cell inside; their rows
  // publish zeros below, their columns reach no other lane, and neither is stored.
  auto clampi = [](int v, int hi) { return v < 0 ? 0 : (v > hi ? hi : v); };
  const int yc = clampi(y, N - 1), yec = clampi(ye, N - 1), xcl = xok ? x0 : 0;
  const uint32_t at = (uint32_t)(yc * N + xcl), ate = (uint32_t)(yec * N + xcl);
  const uint32_t offx = at * sizeof(T), offe = ate * sizeof(T), offk = at * sizeof(R),
                 offku = (at + N) * sizeof(R);
  const uint32_t offc = (uint32_t)((yc >> 1) * Nc + (xcl >> 1)) * sizeof(T),
                 offce = (uint32_t)((yec >> 1) * Nc + (xcl >> 1)) * sizeof(T);
  // column base pointers (inactive columns point at column 0 and are never stored)
  const T* xc[COLS];
  const T* bc[COLS];
  const T* ecc[COLS];
  T* xo[COLS];
#pragma unroll
  for (int c = 0; c < COLS; ++c) {
    const int64_t col = con[c] ? col0 + c : 0;
    xc[c] = xin + (HX ? col * n : 0);
    bc[c] = b + col * n;
    ecc[c] = ec + (HE ? col * (int64_t)Nc * Nc * Nc : 0);
    xo[c] = xout + col * n;
  }
  auto ld2 = [](const auto* base, uint32_t off, auto& v0, auto& v1) {
    const auto* q = reinterpret_cast<decltype(base)>(reinterpret_cast<const char*>(base) + off);
    v0 = q[0];
    v1 = q[1];
  };

  // planes p+2 (loads in flight), p+1, p, p-1 in a ring of four slots that the loop
  // below unrolls, so that a step moves no registers: x_in / x, right-hand side,
  // couplings; on the edge rows the outer row.  Xq: x of plane p-2.
  T X0[4][COLS], X1[4][COLS], E[4][COLS], B0[4][COLS], B1[4][COLS];
  T Xq0[COLS], Xq1[COLS];
  PlaneK<R> K[4];
  auto clear = [&](int s) {
#pragma unroll
    for (int c = 0; c < COLS; ++c)
      X0[s][c] = X1[s][c] = E[s][c] = B0[s][c] = B1[s][c] = zero;
    K[s] = PlaneK<R>{};
  };
  auto load_plane = [&](int s, int z) {
    if (z >= N) {  // uniform
      clear(s);
      return;
    }
    int64_t zo = (int64_t)z * NN, zc = (int64_t)(z >> 1) * Nc * Nc;
    // not to be turned into one running 64-bit pointer per lane and array
    asm volatile("" : "+s"(zo), "+s"(zc));
    const int ez = (F + ybase + z) & 1;  // the element of the outer row that plane z's update reads
#pragma unroll
    for (int c = 0; c < COLS; ++c) {
      X0[s][c] = X1[s][c] = E[s][c] = zero;
      if constexpr (HX) {
        ld2(xc[c] + zo, offx, X0[s][c], X1[s][c]);
        E[s][c] = *reinterpret_cast<const T*>(reinterpret_cast<const char*>(xc[c] + zo + ez) + offe);
      }
      ld2(bc[c] + zo, offx, B0[s][c], B1[s][c]);
      if constexpr (HE) {
        const char* ep = reinterpret_cast<const char*>(ecc[c] + zc);
        const T e = *reinterpret_cast<const T*>(ep + offc);
        const T eo = *reinterpret_cast<const T*>(ep + offce);
        X0[s][c] += ws * e;
        X1[s][c] += ws * e;
        E[s][c] += ws * eo;
      }
    }
    PlaneK<R>& k = K[s];
    ld2(kl + zo, offk, k.kx0, k.kx1);
    ld2(kl + stride + zo, offk, k.kyl0, k.kyl1);
    ld2(kl + stride + zo, offku, k.kyu0, k.kyu1);
    ld2(kl + 2 * stride + zo, offk, k.kz0, k.kz1);
    ld2(dg + n + zo, offk, k.d0, k.d1);  // the diagonal's reciprocals lie behind it
  };

  // this workgroup's planes zs .. ze-1 (segments of SZ): the march starts one
  // plane early (first colour only there) and reads one plane more below it
  const int zs = bz * SZ;
  const int ze = zs + SZ < N ? zs + SZ : N;
  const int p0 = zs > 0 ? zs - 1 : 0;
  const int pe = ze < N ? ze : N;
  // plane z is in slot (z - p0) & 3
#pragma unroll
  for (int c = 0; c < COLS; ++c) Xq0[c] = Xq1[c] = zero;
  if (p0 >= 1)
    load_plane(3, p0 - 1);
  else
    clear(3);
  clear(2);
  load_plane(0, p0);
  load_plane(1, p0 + 1);
  for (int pb = p0; pb <= pe; pb += 4) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int p = pb + u;
      if (p > pe) break;  // uniform
      const int sm = (u + 2) & 3, sn = (u + 1) & 3, sc = u, sp = (u + 3) & 3;
      // plane p-2 leaves its slot to plane p+2, loaded a step ahead of its first use
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        Xq0[c] = X0[sm][c];
        Xq1[c] = X1[sm][c];
      }
      load_plane(sm, p + 2);  // zeros beyond the last plane
      // element of the pair updated in this step (first colour on plane p,
      // second colour on plane p-1): e = (F + y + p) & 1, uniform per wave
      const int e = (F + ybase + p) & 1;
      const int buf = p & 1;
      // publish: this row's second-colour cell of plane p (x_in, element 1-e) and
      // first-colour cell of plane p-1 (updated last step, element 1-e)
#pragma unroll
      for (int c = 0; c < COLS; ++c) {
        const T va = e ? X0[sc][c] : X1[sc][c], vb = e ? X0[sp][c] : X1[sp][c];
        xa[buf][r][c][pl] = row_in ? va : zero;
        xb[buf][r][c][pl] = row_in ? vb : zero;
      }
      __syncthreads();
      const PlaneK<R>&Kc = K[sc], &Kn = K[sn], &Kp = K[sp];
      // first colour on plane p, element e (all rows of the workgroup)
      if (p < N) {
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
          const T alo = xa[buf][r > 0 ? r - 1 : 0][c][pl];
          const T ahi = xa[buf][r < RW - 1 ? r + 1 : RW - 1][c][pl];
          const T ev = eok ? E[sc][c] : zero;
          const T ylo = r > 0 ? alo : ev;
          const T yhi = r < RW - 1 ? ahi : ev;
          if (e == 0) {
            const T sh = wave_shr1(X1[sc][c]);
            const T l = pl > 0 ? sh : zero;
            const T v = B0[sc][c] + Kc.kx0 * l + Kc.kx1 * X1[sc][c] + Kc.kyl0 * ylo +
                        Kc.kyu0 * yhi + Kc.kz0 * X0[sp][c] + Kn.kz0 * X0[sn][c];
            X0[sc][c] = Kc.d0 * v;
          } else {
            const T sh = wave_shl1(X0[sc][c]);
            const R shk = wave_shl1(Kc.kx0);
            const T rr = has_r ? sh : zero;
            const R kr = has_r ? shk : (R)0;
            const T v = B1[sc][c] + Kc.kx1 * X0[sc][c] + kr * rr + Kc.kyl1 * ylo +
                        Kc.kyu1 * yhi + Kc.kz1 * X1[sp][c] + Kn.kz1 * X1[sn][c];
            X1[sc][c] = Kc.d1 * v;
          }
        }
      }
      // second colour on plane p-1, element e (rows y0 .. y0+TY-1), and output
      if (p - 1 >= zs) {
        int64_t zo = (int64_t)(p - 1) * NN;
        asm volatile("" : "+s"(zo));
#pragma unroll
        for (int c = 0; c < COLS; ++c) {
          const T ylo = xb[buf][r > 0 ? r - 1 : 0][c][pl];
          const T yhi = xb[buf][r < RW - 1 ? r + 1 : RW - 1][c][pl];
          if (e == 0) {
            const T sh = wave_shr1(X1[sp][c]);
            const T l = pl > 0 ? sh : zero;
            const T v = B0[sp][c] + Kp.kx0 * l + Kp.kx1 * X1[sp][c] + Kp.kyl0 * ylo +
                        Kp.kyu0 * yhi + Kp.kz0 * Xq0[c] + Kc.kz0 * X0[sc][c];
            if (inner) X0[sp][c] = Kp.d0 * v;
          } else {
            const T sh = wave_shl1(X0[sp][c]);
            const R shk = wave_shl1(Kp.kx0);
            const T rr = has_r ? sh : zero;
            const R kr = has_r ? shk : (R)0;
            const T v = B1[sp][c] + Kp.kx1 * X0[sp][c] + kr * rr + Kp.kyl1 * ylo +
                        Kp.kyu1 * yhi + Kp.kz1 * Xq1[c] + Kc.kz1 * X1[sc][c];
            if (inner) X1[sp][c] = Kp.d1 * v;
          }
          if (store && con[c]) {
            T* q = reinterpret_cast<T*>(reinterpret_cast<char*>(xo[c] + zo) + offx);
            q[0] = X0[sp][c];
            q[1] = X1[sp][c];
          }
        }
      }
    }
  }
}

}  // namespace vcb
}  // namespace mlmc
