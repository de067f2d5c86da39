// smear_kernels.hpp -- the smearing-step kernel (launcher in k_smear.hip).
#pragma once

#include "internal.hpp"
#include "smear.hpp"

namespace mcg {

// A thread per link: over-improved stout (OI), and stout where k_smear_stout's blocks are too coarse
// (stout_in_blocks).  CS = 1: also store the staple sums Cp (and Cr, OI) of every link in Cst, as two link
// fields [Cp | Cr], for the adjoint's first pass
template <typename T, bool OI, int CS = 0>
__global__ __launch_bounds__(128, sizeof(T) == 4 ? (OI ? 2 : 3) : 1) void k_smear(Geom g, const V2<T> *__restrict__ U,
                                               V2<T> *__restrict__ out, T rho, T wp, T wr,
                                               V2<T> *__restrict__ Cst = nullptr) {
  // one block per (tile, direction, parity), the tiles as gather_site lays them out; the eight blocks
  // of a tile follow each other and each XCD takes a contiguous range of tiles (xcd_range), so the
  // staple links that the eight share, and those of the neighbouring tiles along z and t, are mostly
  // still in that XCD's L2
  const int w = xcd_range((int)blockIdx.x, (int)gridDim.x);
  const int h = gather_site(g, w >> 3, (int)threadIdx.x);
  if (h < 0) return;
  const int mu = (w & 7) >> 1, par = w & 1;
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  M3<T> Cp, Cr;
  staples<T, OI>(g, L, par, h, mu, Cp, Cr);
  if constexpr (CS != 0) {
    Links<T>{Cst, g.Vh}.store(mu, par, h, Cp);
    if (OI) Links<T>{Cst + (size_t)72 * g.Vh, g.Vh}.store(mu, par, h, Cr);
  }
  M3<T> C;
#pragma unroll
  for (int k = 0; k < 9; k++) {
    C.e[k] = rho * (wp * Cp.e[k]);
    if (OI) C.e[k] = rho * (wp * Cp.e[k] + wr * Cr.e[k]);
  }
  const M3<T> u = L.load(mu, par, h);
  const M3<T> E = exp_su3(ta(mul_nd(C, u)));
  Links<T>{out, g.Vh}.store(mu, par, h, mul(E, u));
}

// Stout: one block per 64 half-sites of one parity, wave mu the links of direction mu.  Waves mu and
// nu = mu ^ j take the direction nu and mu of their plane together and read U_nu(x) and U_nu(x+mu) from each
// other through LDS, so that a link takes 13 matrices from the caches instead of 19 (11.5 GB per
// 32^3x64 FP32 step, 14 TB/s, was what the step had waited for).  FP32 runs four waves per SIMD (126
// registers), and tiles in groups of four t-slices, the 64-site tiles of eight being more than an
// XCD's L2 holds.  CS = 1: also store Cp in Cst.
// 32^3x64 FP32, per step: 0.802 ms with a wave per link and 19 loads, 0.767 with the exchange at three
// waves per SIMD, 0.747 at four, 0.713 with the groups of four (of two: 0.744): 76 % of the VALU issue
// rate.  FP64, 20^3x40 and 16^4: 0.136 -> 0.123 ms on average.  The sums
// of k_smear<T, false>, in another order.
template <typename T, int CS = 0>
__global__ __launch_bounds__(256, sizeof(T) == 4 ? 4 : 2) void k_smear_stout(Geom g, const V2<T> *__restrict__ U, V2<T> *__restrict__ out,
                                                     T rho, T wp, V2<T> *__restrict__ Cst = nullptr) {
  __shared__ V2<T> own[4][9][64], ahead[4][9][64];  // U_mu(x); U_mu(x + (mu ^ j)) of the step
  const int w = xcd_range((int)blockIdx.x, (int)gridDim.x);
  const int lane = (int)threadIdx.x & 63, mu = wave_uniform((int)threadIdx.x >> 6), par = w & 1;
  const int site = gather_site<64, 4>(g, w >> 1, lane);
  const bool live = site >= 0;
  const int h = live ? site : 0;  // idle lanes follow along on the first site
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  auto put = [&](V2<T>(*m)[64], const M3<T> &a) {
#pragma unroll
    for (int k = 0; k < 9; k++) {
      V2<T> v;
      v.x = a.e[k].re;
      v.y = a.e[k].im;
      m[k][lane] = v;
    }
  };
  auto get = [&](const V2<T>(*m)[64]) -> M3<T> {
    M3<T> a;
#pragma unroll
    for (int k = 0; k < 9; k++) {
      const V2<T> v = m[k][lane];
      a.e[k] = cx<T>{v.x, v.y};
    }
    return a;
  };
  int c[4];
  coords_of(g, par, h, c);
  const Around<T> x0(L, par, h);
  const int m1 = move_by<T>(g, c, mu, +1);
  put(own[mu], L.load_off(mu, x0.even(0)));
  M3<T> Cp = m_zero<T>();
  for (int j = 1; j < 4; j++) {
    const int nu = mu ^ j;
    const Around<T> x = opaque_site(x0);
    const int n1 = move_by<T>(g, c, nu, +1), n_1 = move_by<T>(g, c, nu, -1);
    M3<T> umu_xpn = L.load_off(mu, x.odd(n1));
    M3<T> unu_xmn = L.load_off(nu, x.odd(n_1)), umu_xmn = L.load_off(mu, x.odd(n_1)),
          unu_xmnpm = L.load_off(nu, x.even(n_1 + m1));
    if constexpr (sizeof(T) == 4) {  // held until all are in, as in staples
      opaque_m3(umu_xpn);
      opaque_m3(unu_xmn);
      opaque_m3(umu_xmn);
      opaque_m3(unu_xmnpm);
    }
    if (j > 1) __syncthreads();  // the last step's matrices have been read
    put(ahead[mu], umu_xpn);
    __syncthreads();
    mac_nd(mul(get(own[nu]), umu_xpn), get(ahead[nu]), Cp);  // U_nu(x) U_mu(x+nu) U_nu(x+mu)^dag
    mac(mul_dn(unu_xmn, umu_xmn), unu_xmnpm, Cp);           // U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu)
  }
  if (!live) return;
  if constexpr (CS != 0) Links<T>{Cst, g.Vh}.store(mu, par, h, Cp);
  M3<T> C;
#pragma unroll
  for (int k = 0; k < 9; k++) C.e[k] = rho * (wp * Cp.e[k]);
  const M3<T> u = get(own[mu]);
  const M3<T> E = exp_su3(ta(mul_nd(C, u)));
  Links<T>{out, g.Vh}.store(mu, par, h, mul(E, u));
}

}  // namespace mcg
