// The two-spin hop term of a lattice site, shared by the kernels that apply it.
#pragma once
#include "common.h"

namespace mlmc {
namespace wil {

__host__ __device__ __forceinline__ c32 mk(float re, float im) { return {re, im}; }
__host__ __device__ __forceinline__ c64 mk(double re, double im) { return {re, im}; }
template <typename T> __device__ __forceinline__ T times_i(T a) { return mk(-a.im, a.re); }
template <typename T> __device__ __forceinline__ T cmul_conj(T u, T a) {  // conj(u) * a
  return mk(u.re * a.re + u.im * a.im, u.re * a.im - u.im * a.re);
}

// hop term H x at a site (the sum in D = (m0+2) I - H/2), 2 spins, from the
// links u (+x: U_0(s), -x: U_0(s-x), +y: U_1(s), -y: U_1(s-y)) and the
// neighbours' spin pairs xp (s+x), xm (s-x), yp (s+y), ym (s-y)
template <typename T>
__device__ __forceinline__ void wilson_hop_sum(T upx, T xp0, T xp1, T umx, T xm0, T xm1, T upy,
                                               T yp0, T yp1, T umy, T ym0, T ym1, T& h0,
                                               T& h1) {
  // +x: (I - s1) U_0(s) x_{s+x}
  {
    const T a0 = upx * xp0, a1 = upx * xp1;
    h0 = a0 - a1;
    h1 = a1 - a0;
  }
  // -x: (I + s1) conj(U_0(s-x)) x_{s-x}
  {
    const T a0 = cmul_conj(umx, xm0), a1 = cmul_conj(umx, xm1);
    h0 += a0 + a1;
    h1 += a1 + a0;
  }
  // +y: (I - s2) U_1(s) x_{s+y};  (I - s2) v = (v0 - i v1, v1 + i v0)
  {
    const T a0 = upy * yp0, a1 = upy * yp1;
    h0 += a0 - times_i(a1);
    h1 += a1 + times_i(a0);
  }
  // -y: (I + s2) conj(U_1(s-y)) x_{s-y};  (I + s2) v = (v0 + i v1, v1 - i v0)
  {
    const T a0 = cmul_conj(umy, ym0), a1 = cmul_conj(umy, ym1);
    h0 += a0 + times_i(a1);
    h1 += a1 - times_i(a0);
  }
}

// hop term at site (sx, sy) with x read from the column's global vector
template <typename T>
__device__ __forceinline__ void wilson_hop(const T* __restrict__ x, const T* __restrict__ U, int N,
                                           int sx, int sy, T& h0, T& h1) {
  const int n2 = N * N;
  const int xp = sx + 1 == N ? 0 : sx + 1, xm = sx == 0 ? N - 1 : sx - 1;
  const int yp = sy + 1 == N ? 0 : sy + 1, ym = sy == 0 ? N - 1 : sy - 1;
  const int s = sy * N + sx;
  const int tpx = sy * N + xp, tmx = sy * N + xm, tpy = yp * N + sx, tmy = ym * N + sx;
  wilson_hop_sum(U[s], x[2 * tpx], x[2 * tpx + 1], U[tmx], x[2 * tmx], x[2 * tmx + 1],
                 U[n2 + s], x[2 * tpy], x[2 * tpy + 1], U[n2 + tmy], x[2 * tmy], x[2 * tmy + 1],
                 h0, h1);
}

}  // namespace wil
}  // namespace mlmc
