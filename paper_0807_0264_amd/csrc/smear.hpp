// smear.hpp -- device pieces of stout and over-improved stout smearing
// (Sec. II.B of arXiv:0807.0264; parameters of Sec. III): the staple sum of
// one link and exp of a traceless anti-Hermitian 3x3 matrix through the
// Cayley-Hamilton relation Q^3 = c1 Q + c0 (Q = -iA Hermitian traceless,
// c1 = tr(Q^2)/2, c0 = det Q).
#pragma once

#include "common.hpp"

namespace mcg {

// Powers of Q reduce to Q^n = a_n + b_n Q + d_n Q^2 with the real recursion
// a_{n+1} = c0 d_n, b_{n+1} = a_n + c1 d_n, d_{n+1} = b_n (from Q^3 = c1 Q + c0),
// so exp(iQ) = f0 + f1 Q + f2 Q^2 with f_j = sum_n (i^n / n!) {a,b,d}_n.
// The derivatives of the f_j with respect to c0 and c1 follow from the same
// recursion differentiated term by term (used by the adjoint).
template <typename T> struct CHCoef {
  cx<T> f[3];
  cx<T> df0[3];  // d f_j / d c0
  cx<T> df1[3];  // d f_j / d c1
};

template <typename T, int N, bool DERIV>
__device__ __forceinline__ void ch_series(T c0, T c1, CHCoef<T> &o) {
  T a = T(1), b = T(0), d = T(0);
  T a0 = T(0), b0 = T(0), d0 = T(0);  // d/dc0 of a, b, d
  T a1 = T(0), b1 = T(0), d1 = T(0);  // d/dc1 of a, b, d
  T wre = T(1), wim = T(0);
  o.f[0] = cx<T>{T(1), T(0)};
  o.f[1] = o.f[2] = cx<T>{T(0), T(0)};
  if (DERIV) {
#pragma unroll
    for (int j = 0; j < 3; j++) o.df0[j] = o.df1[j] = cx<T>{T(0), T(0)};
  }
#pragma unroll
  for (int n = 1; n <= N; n++) {
    const T an = c0 * d, bn = a + c1 * d, dn = b;
    if (DERIV) {
      const T a0n = c0 * d0 + d, b0n = a0 + c1 * d0, d0n = b0;
      const T a1n = c0 * d1, b1n = a1 + c1 * d1 + d, d1n = b1;
      a0 = a0n; b0 = b0n; d0 = d0n;
      a1 = a1n; b1 = b1n; d1 = d1n;
    }
    a = an;
    b = bn;
    d = dn;
    const T inv = T(1) / T(n);
    const T nre = -wim * inv, nim = wre * inv;  // w <- w * i / n
    wre = nre;
    wim = nim;
    o.f[0] = o.f[0] + cx<T>{wre * a, wim * a};
    o.f[1] = o.f[1] + cx<T>{wre * b, wim * b};
    o.f[2] = o.f[2] + cx<T>{wre * d, wim * d};
    if (DERIV) {
      o.df0[0] = o.df0[0] + cx<T>{wre * a0, wim * a0};
      o.df0[1] = o.df0[1] + cx<T>{wre * b0, wim * b0};
      o.df0[2] = o.df0[2] + cx<T>{wre * d0, wim * d0};
      o.df1[0] = o.df1[0] + cx<T>{wre * a1, wim * a1};
      o.df1[1] = o.df1[1] + cx<T>{wre * b1, wim * b1};
      o.df1[2] = o.df1[2] + cx<T>{wre * d1, wim * d1};
    }
  }
}

// Q = -iA for anti-Hermitian A
template <typename T> __device__ __forceinline__ M3<T> minus_i(const M3<T> &A) {
  M3<T> Q;
#pragma unroll
  for (int k = 0; k < 9; k++) Q.e[k] = cx<T>{A.e[k].im, -A.e[k].re};
  return Q;
}

// c1 = tr(Q^2)/2 and c0 = det Q = tr(Q^3)/3 for traceless Hermitian Q
template <typename T>
__device__ __forceinline__ void ch_invariants(const M3<T> &Q, const M3<T> &Q2, T &c0, T &c1) {
  c1 = T(0.5) * (Q2.e[0].re + Q2.e[4].re + Q2.e[8].re);
  T t3 = T(0);
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int j = 0; j < 3; j++) t3 += (Q.e[3 * i + j] * Q2.e[3 * j + i]).re;
  c0 = t3 * T(1.0 / 3.0);
}

template <typename T> struct ExpTerms;
template <> struct ExpTerms<float> { static constexpr int N = 14; };
template <> struct ExpTerms<double> { static constexpr int N = 22; };

// exp(A) for A in su(3).  Q is scaled by 2^-s until the bound sqrt(4 c1/3)
// on its spectral radius is at most 1; the series is summed for the scaled
// matrix and the result squared s times.
template <typename T> __device__ __forceinline__ M3<T> exp_su3(const M3<T> &A) {
  const M3<T> Q = minus_i(A);
  const M3<T> Q2 = mul(Q, Q);
  T c0, c1;
  ch_invariants(Q, Q2, c0, c1);
  int s = 0;
  T r2 = T(4.0 / 3.0) * c1;
  T sc = T(1);
  while (r2 > T(1) && s < 40) {
    r2 *= T(0.25);
    sc *= T(0.5);
    s++;
  }
  const T sc2 = sc * sc;
  CHCoef<T> co;
  ch_series<T, ExpTerms<T>::N, false>(c0 * sc2 * sc, c1 * sc2, co);
  const cx<T> g1 = sc * co.f[1], g2 = sc2 * co.f[2];
  M3<T> E;
#pragma unroll
  for (int k = 0; k < 9; k++) E.e[k] = g1 * Q.e[k] + g2 * Q2.e[k];
  E.e[0] = E.e[0] + co.f[0];
  E.e[4] = E.e[4] + co.f[0];
  E.e[8] = E.e[8] + co.f[0];
  for (int q = 0; q < s; q++) E = mul(E, E);
  return E;
}

// Byte offsets of the sites x + a mu + b nu (|a|, |b| <= 2) around a site x of parity par, half index h
// and coordinates c, into the planes of a link field.  Lx is even, so a step along y, z or t moves the
// half index by a stride whatever x is, a step along x by what (x >> 1) moves, and steps along
// different directions add: two selections per (direction, steps) and one addition per site, where
// going from coordinates to an index took three 32-bit multiplications (a quarter of the FMA rate) per
// site, a tenth of the instructions: per wave, over-improved 9,703 -> 8,845, stout 2,581 -> 2,367.  Stout
// 32^3x64 FP32 0.823 -> 0.802 ms a step; the over-improved step and the loop gather, which run at the
// clock that their FMAs allow, 0 and 2.5 % faster.
template <typename T> struct Around {
  unsigned same, other;  // x as a site of its own parity; the same half index of the other parity
  __device__ __forceinline__ Around(const Links<T> &L, int par, int h) : same(L.off(par, h)), other(L.off(1 - par, h)) {}
  // the offset after an odd (or even) number of steps that moved by d
  __device__ __forceinline__ unsigned odd(int d) const { return other + (unsigned)d; }
  __device__ __forceinline__ unsigned even(int d) const { return same + (unsigned)d; }
};
// what `step` (|step| <= 2, at most the extent) along direction d moves, in bytes
template <typename T> __device__ __forceinline__ int move_by(const Geom &g, const int c[4], int d, int step) {
  const int x = d == 0 ? c[0] : d == 1 ? c[1] : d == 2 ? c[2] : c[3], n = g.L[d];
  if (d == 0) {
    int v = x + step;
    v = v >= n ? v - n : v;
    v = v < 0 ? v + n : v;
    return ((v >> 1) - (x >> 1)) * (int)sizeof(V2<T>);
  }
  int st = g.hx * (int)sizeof(V2<T>);
  if (d > 1) st *= g.L[1];
  if (d > 2) st *= g.L[2];
  const bool wrap = step > 0 ? x + step >= n : x + step < 0;
  return wrap ? (step > 0 ? step - n : step + n) * st : step * st;
}
// Make the compiler treat a site's offsets as freshly produced (see staples).
template <typename T> __device__ __forceinline__ Around<T> opaque_site(Around<T> x) {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__ volatile("" : "+v"(x.same), "+v"(x.other));
#endif
  return x;
}

// ... and, with m, as known only once all of m is: loads from x are not issued before m is computed.
template <typename T> __device__ __forceinline__ Around<T> opaque_site(Around<T> x, M3<T> &m) {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__ volatile(""
                   : "+v"(x.same), "+v"(x.other), "+v"(m.e[0].re), "+v"(m.e[0].im), "+v"(m.e[1].re),
                     "+v"(m.e[1].im), "+v"(m.e[2].re), "+v"(m.e[2].im), "+v"(m.e[3].re), "+v"(m.e[3].im));
  __asm__ volatile(""
                   : "+v"(x.same), "+v"(x.other), "+v"(m.e[4].re), "+v"(m.e[4].im), "+v"(m.e[5].re),
                     "+v"(m.e[5].im), "+v"(m.e[6].re), "+v"(m.e[6].im), "+v"(m.e[7].re), "+v"(m.e[7].im),
                     "+v"(m.e[8].re), "+v"(m.e[8].im));
#else
  (void)m;
#endif
  return x;
}

// Make the compiler treat a loaded matrix as produced here: every load into it is complete at this
// point (see staples).
template <typename T> __device__ __forceinline__ void opaque_m3(M3<T> &m) {
#if defined(__HIP_DEVICE_COMPILE__)
#pragma unroll
  for (int k = 0; k < 9; k++) __asm__ volatile("" : "+v"(m.e[k].re), "+v"(m.e[k].im));
#else
  (void)m;
#endif
}

// Plaquette part Cp and rectangle part Cr (OI only) of the staple sum of
// link (c, mu): paths from x to x+mu.  Per nu != mu and per sign of nu: the
// plaquette staple and the rectangles 2x1 ahead, 2x1 behind (long in mu) and
// 1x2 (long in nu).  Rectangles that end on the same link share the last
// product: the 2x1-behind and 1x2 paths of one nu and sign both end on the
// link into x+mu along nu, and every 2x1-ahead path ends on U_mu(x+mu)^dag, so
// their prefixes are summed first and multiplied by that link once.
template <typename T, bool OI>
__device__ __forceinline__ void staples(const Geom &g, const Links<T> &L, int par, int h, int mu, M3<T> &Cp,
                                        M3<T> &Cr) {
  Cp = m_zero<T>();
  Cr = m_zero<T>();
  M3<T> ahead = m_zero<T>();  // OI: sum of the 2x1-ahead prefixes, closed by U_mu(x+mu)^dag at the end
  int c[4];
  coords_of(g, par, h, c);
  const Around<T> x0(L, par, h);
  const int m1 = move_by<T>(g, c, mu, +1);
  if constexpr (!OI) {
    // Stout, for small launches and for the adjoint where the forward pass's staple sums did not fit:
    // the six links of a direction are loaded together and (FP32) held until all six are in, so a wave
    // has six loads in flight instead of three.  Unrolled, nu is known when the kernel is compiled and a
    // direction's offsets need no look-up of its extent: k_smear, 4^4 FP32 9.3 -> 8.7 us, 8^4 9.6 -> 8.9,
    // FP64 10.6 -> 9.4, against directions taken as mu ^ 1, mu ^ 2, mu ^ 3 in a loop.
#pragma unroll
    for (int nu = 0; nu < 4; nu++) {
      if (nu == mu) continue;
      const Around<T> x = opaque_site(x0);
      const int n1 = move_by<T>(g, c, nu, +1), n_1 = move_by<T>(g, c, nu, -1);
      M3<T> unu_x = L.load_off(nu, x.even(0)), umu_xpn = L.load_off(mu, x.odd(n1)),
            unu_xpm = L.load_off(nu, x.odd(m1));  // +nu side
      M3<T> unu_xmn = L.load_off(nu, x.odd(n_1)), umu_xmn = L.load_off(mu, x.odd(n_1)),
            unu_xmnpm = L.load_off(nu, x.even(n_1 + m1));  // -nu
      if constexpr (sizeof(T) == 4) {
        opaque_m3(unu_x);
        opaque_m3(umu_xpn);
        opaque_m3(unu_xpm);
        opaque_m3(unu_xmn);
        opaque_m3(umu_xmn);
        opaque_m3(unu_xmnpm);
      }
      mac_nd(mul(unu_x, umu_xpn), unu_xpm, Cp);       // U_nu(x) U_mu(x+nu) U_nu(x+mu)^dag
      mac(mul_dn(unu_xmn, umu_xmn), unu_xmnpm, Cp);  // U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu)
    }
    return;
  }
  const int m_1 = move_by<T>(g, c, mu, -1), m2 = move_by<T>(g, c, mu, +2);
  if constexpr (sizeof(T) == 8) {
    // FP64 multiplies the two links of a long side first, so that every path is three factors: the
    // same number of products, with the 2x1-behind paths too summed without their common first
    // link.  A side then has few matrices live at once, and the compiler keeps its order of loads without
    // the pins that FP32 needs below (whose moves of 64-bit pairs cost more than they hid): 20^3x40 1.00 ->
    // 0.70 ms a step, 16^4 170 -> 140 us, 8^4 39 -> 31 (the order below without pins: 0.89 ms,
    // 152, 35; the pins with this order: 1.00-1.22 ms).  FP32 takes as long with a fifth of its products
    // left out (0.37 ms at 20^3x40): it waits for the 63 matrices of a link at 16 TB/s of cache reads, and
    // this order with pins or without takes 0.40-0.44 ms.
    M3<T> behind = m_zero<T>();  // sum of the 2x1-behind paths without U_mu(x-mu)^dag
    auto two = [&](int d, unsigned a, unsigned b) -> M3<T> { return mul(L.load_off(d, a), L.load_off(d, b)); };
    for (int nu = 0; nu < 4; nu++) {
      if (nu == mu) continue;
      {  // +nu
        const Around<T> x = opaque_site(x0, Cr);
        const int n1 = move_by<T>(g, c, nu, +1), n2 = move_by<T>(g, c, nu, +2);
        const M3<T> unu_x = L.load_off(nu, x.even(0)), umu_xpn = L.load_off(mu, x.odd(n1)),
                    unu_xpm = L.load_off(nu, x.odd(m1));
        const M3<T> a1 = L.load_off(mu, x.even(n1 + m1)), a2 = L.load_off(nu, x.even(m2));
        M3<T> t = mul(unu_x, umu_xpn);
        const M3<T> b1 = L.load_off(nu, x.odd(m_1)), b2 = two(mu, x.even(m_1 + n1), x.odd(n1));
        mac_nd(t, unu_xpm, Cp);  // U_nu(x) U_mu(x+nu) U_nu(x+mu)^dag
        t = mul(t, a1);
        const M3<T> d1 = two(nu, x.even(0), x.odd(n1)), d2 = L.load_off(mu, x.even(n2)),
                    d3 = two(nu, x.odd(m1), x.even(m1 + n1));
        mac_nd(t, a2, ahead);  // U_nu(x) U_mu(x+nu) U_mu(x+nu+mu) U_nu(x+2mu)^dag [U_mu(x+mu)^dag]
        t = mul(b1, b2);
        mac_nd(t, unu_xpm, behind);  // [U_mu(x-mu)^dag] U_nu(x-mu) (U_mu U_mu)(x-mu+nu) U_nu(x+mu)^dag
        t = mul(d1, d2);
        mac_nd(t, d3, Cr);  // (U_nu U_nu)(x) U_mu(x+2nu) (U_nu U_nu)(x+mu)^dag
      }
      {  // -nu
        const Around<T> x = opaque_site(x0, Cr);
        const int n_1 = move_by<T>(g, c, nu, -1), n_2 = move_by<T>(g, c, nu, -2);
        const M3<T> unu_xmn = L.load_off(nu, x.odd(n_1)), umu_xmn = L.load_off(mu, x.odd(n_1)),
                    unu_xmnpm = L.load_off(nu, x.even(n_1 + m1));
        const M3<T> a1 = L.load_off(mu, x.even(n_1 + m1)), a2 = L.load_off(nu, x.odd(n_1 + m2));
        M3<T> t = mul_dn(unu_xmn, umu_xmn);
        const M3<T> b1 = L.load_off(nu, x.even(m_1 + n_1)), b2 = two(mu, x.even(m_1 + n_1), x.odd(n_1));
        mac(t, unu_xmnpm, Cp);  // U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu)
        t = mul(t, a1);
        const M3<T> d1 = two(nu, x.even(n_2), x.odd(n_1)), d2 = L.load_off(mu, x.even(n_2)),
                    d3 = two(nu, x.odd(n_2 + m1), x.even(n_1 + m1));
        mac(t, a2, ahead);  // U_nu(x-nu)^dag U_mu(x-nu) U_mu(x-nu+mu) U_nu(x-nu+2mu) [U_mu(x+mu)^dag]
        t = mul_dn(b1, b2);
        mac(t, unu_xmnpm, behind);  // [U_mu(x-mu)^dag] U_nu(x-mu-nu)^dag (U_mu U_mu)(x-mu-nu) U_nu(x-nu+mu)
        t = mul_dn(d1, d2);
        mac(t, d3, Cr);  // (U_nu U_nu)(x-2nu)^dag U_mu(x-2nu) (U_nu U_nu)(x-2nu+mu)
      }
    }
    add_to(mul_dn(L.load_off(mu, x0.odd(m_1)), behind), Cr);
    mac_nd(ahead, L.load_off(mu, x0.odd(m1)), Cr);
    return;
  }
  // FP32 from here on
  const M3<T> umu_xmm = L.load_off(mu, x0.odd(m_1));  // U_mu(x-mu)
  for (int nu = 0; nu < 4; nu++) {
    if (nu == mu) continue;
    // Each side of the direction starts from opaque copies of the site's offsets, so the
    // compiler forms its addresses and loads where they are used rather than all at once (a
    // register-pressure hint with no run-time cost); the sums are taken in the same order.
    {  // +nu
      Around<T> x = opaque_site(x0, Cr);
      const int n1 = move_by<T>(g, c, nu, +1), n2 = move_by<T>(g, c, nu, +2);
      const M3<T> unu_x = L.load_off(nu, x.even(0));     // U_nu(x)
      const M3<T> umu_xpn = L.load_off(mu, x.odd(n1));   // U_mu(x+nu)
      const M3<T> unu_xpm = L.load_off(nu, x.odd(m1));   // U_nu(x+mu)
      M3<T> up = mul(unu_x, umu_xpn);                    // U_nu(x) U_mu(x+nu)
      x = opaque_site(x, up);
      mac_nd(up, unu_xpm, Cp);
      M3<T> t, end;
      // 2x1 ahead: U_nu(x) U_mu(x+nu) U_mu(x+nu+mu) U_nu(x+2mu)^dag [U_mu(x+mu)^dag]
      t = mul(up, L.load_off(mu, x.even(n1 + m1)));
      x = opaque_site(x, t);
      mac_nd(t, L.load_off(nu, x.even(m2)), ahead);
      // 2x1 behind: U_mu(x-mu)^dag U_nu(x-mu) U_mu(x-mu+nu) U_mu(x+nu) [U_nu(x+mu)^dag]
      t = mul_dn(umu_xmm, L.load_off(nu, x.odd(m_1)));
      t = mul(t, L.load_off(mu, x.even(m_1 + n1)));
      end = mul(t, umu_xpn);
      x = opaque_site(x, end);
      // 1x2: U_nu(x) U_nu(x+nu) U_mu(x+2nu) U_nu(x+mu+nu)^dag [U_nu(x+mu)^dag]
      t = mul(unu_x, L.load_off(nu, x.odd(n1)));
      t = mul(t, L.load_off(mu, x.even(n2)));
      mac_nd(t, L.load_off(nu, x.even(m1 + n1)), end);
      mac_nd(end, unu_xpm, Cr);
    }
    {  // -nu
      Around<T> x = opaque_site(x0, Cr);
      const int n_1 = move_by<T>(g, c, nu, -1), n_2 = move_by<T>(g, c, nu, -2);
      const M3<T> unu_xmn = L.load_off(nu, x.odd(n_1));           // U_nu(x-nu)
      const M3<T> umu_xmn = L.load_off(mu, x.odd(n_1));           // U_mu(x-nu)
      const M3<T> unu_xmnpm = L.load_off(nu, x.even(n_1 + m1));   // U_nu(x-nu+mu)
      M3<T> dn = mul_dn(unu_xmn, umu_xmn);                        // U_nu(x-nu)^dag U_mu(x-nu)
      x = opaque_site(x, dn);
      mac(dn, unu_xmnpm, Cp);
      M3<T> t, end;
      // 2x1 ahead: U_nu(x-nu)^dag U_mu(x-nu) U_mu(x-nu+mu) U_nu(x-nu+2mu) [U_mu(x+mu)^dag]
      t = mul(dn, L.load_off(mu, x.even(n_1 + m1)));
      x = opaque_site(x, t);
      mac(t, L.load_off(nu, x.odd(n_1 + m2)), ahead);
      // 2x1 behind: U_mu(x-mu)^dag U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_mu(x-nu) [U_nu(x-nu+mu)]
      t = dag(mul(L.load_off(nu, x.even(m_1 + n_1)), umu_xmm));
      t = mul(t, L.load_off(mu, x.even(m_1 + n_1)));
      end = mul(t, umu_xmn);
      x = opaque_site(x, end);
      // 1x2: U_nu(x-nu)^dag U_nu(x-2nu)^dag U_mu(x-2nu) U_nu(x-2nu+mu) [U_nu(x-nu+mu)]
      t = dag(mul(L.load_off(nu, x.even(n_2)), unu_xmn));
      t = mul(t, L.load_off(mu, x.even(n_2)));
      mac(t, L.load_off(nu, x.odd(n_2 + m1)), end);
      mac(end, unu_xmnpm, Cr);
    }
  }
  mac_nd(ahead, L.load_off(mu, x0.odd(m1)), Cr);  // ... U_mu(x+mu)^dag
}

}  // namespace mcg
