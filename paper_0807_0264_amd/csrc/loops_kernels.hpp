// loops_kernels.hpp -- vortex-only / vortex-removed fields and Wilson loops
// (launchers in k_loops.hip).
#pragma once

#include "internal.hpp"

namespace mcg {

// site coordinates c moved by the spatial offset (o0, o1, o2) and dt in time,
// each |offset| < 2 L (periodic)
__device__ __forceinline__ void shifted(const Geom &g, const int c[4], int o0, int o1, int o2, int dt,
                                        int e[4]) {
  const int o[4] = {o0, o1, o2, dt};
#pragma unroll
  for (int k = 0; k < 4; k++) {
    int v = c[k] + o[k];
    v = v < 0 ? v + g.L[k] : v;
    v = v < 0 ? v + g.L[k] : v;
    v = v >= g.L[k] ? v - g.L[k] : v;
    v = v >= g.L[k] ? v - g.L[k] : v;
    e[k] = v;
  }
}

// z(m) = exp(2 pi i m / 3) for m in {-1, 0, 1}
__device__ __forceinline__ cx<double> center_elem(int m) {
  const double s3 = 0.86602540378443864676;  // sqrt(3)/2
  return m == 0 ? cx<double>{1.0, 0.0} : cx<double>{-0.5, m > 0 ? s3 : -s3};
}

// mode 0: out_mu(x) = z(m_mu(x)) 1; mode 1: out_mu(x) = conj(z(m_mu(x))) G(x) U_mu(x) G(x+mu)^dag
// (G may be null: identity).  One thread per half index h, both parities.  out may alias U: every
// element is read and written by the same thread.  Bound by HBM (mode 1: U, G and Z read and a field
// written, 724 bytes per site with FP32 links): 32^3x64 425 us with lexicographic tiles, 322 us with
// site_of_block's and streaming links.  LD, ST: loads and stores of links stream (streaming()).
template <typename T, bool LD, bool ST>
__global__ __launch_bounds__(256) void k_vortex_field(Geom g, const V2<T> *U, const double2 *__restrict__ G,
                                                      const int8_t *__restrict__ Z, int mode, V2<T> *out, int tiled) {
  const int h = site_of_block(g, tiled);
  if (h < 0) return;
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  const Links<T> O{out, g.Vh};
  const Gauge gg{const_cast<double2 *>(G), g.Vh};
  for (int par = 0; par < 2; par++) {
    int c[4];
    coords_of(g, par, h, c);
    const int i = lex_index(g, c);
    M3<double> Gx;
    if (mode == 1 && G) Gx = gg.load(par, h);
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
      const cx<double> z = center_elem(Z[(size_t)mu * g.V + i]);
      M3<double> r;
      if (mode == 0) {
        r = m_zero<double>();
        r.e[0] = r.e[4] = r.e[8] = z;
      } else {
        const M3<double> u = m_cvt<double>(L.template load_as<LD>(mu, par, h));
        if (G) {
          int e[4];
          moved(g, c, mu, +1, e);
          r = mul_nd(mul(Gx, u), gg.load(1 - par, half_index(g, e)));
        } else {
          r = u;
        }
        const cx<double> zc = conj(z);
#pragma unroll
        for (int k = 0; k < 9; k++) r.e[k] = r.e[k] * zc;
      }
      O.template store_as<ST>(mu, par, h, m_cvt<T>(r));
    }
  }
}

// For image blockIdx.y: line k of the image, out(x) = in(x) * (the path's links starting at
// x + (k - 1) d), in = line k - 1 (none for k = 1).  Line fields use the link layout with a single
// direction.  Grid: (2 * ceil(Vh / 256), images), the first half of x even sites, the second odd.
template <typename T>
__global__ __launch_bounds__(256) void k_line(Geom g, const V2<T> *__restrict__ U,
                                              const LoopImage<T> *__restrict__ imgs, int k) {
  const LoopImage<T> &im = imgs[blockIdx.y];
  const int nbp = gridDim.x >> 1;
  const int par = blockIdx.x >= nbp;
  // tiles of one parity in contiguous ranges per XCD (xcd_range)
  const int h = xcd_range((int)blockIdx.x - par * nbp, nbp) * 256 + threadIdx.x;
  if (h >= g.Vh) return;
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  const V2<T> *in = k == 1 ? nullptr : ((k & 1) ? im.b : im.a);
  V2<T> *out = (k & 1) ? im.a : im.b;
  int c[4];
  coords_of(g, par, h, c);
  M3<T> M = in ? Links<T>{const_cast<V2<T> *>(in), g.Vh}.load(0, par, h) : m_ident<T>();
  int y[4];
  shifted(g, c, (k - 1) * im.path.d[0], (k - 1) * im.path.d[1], (k - 1) * im.path.d[2], 0, y);
  for (int q = 0; q < im.path.n; q++) {
    const int st = im.path.s[q];
    const int a = (st > 0 ? st : -st) - 1;
    if (st > 0) {
      M = mul(M, L.at(g, y, a));
      int e[4];
      moved(g, y, a, +1, e);
#pragma unroll
      for (int q2 = 0; q2 < 4; q2++) y[q2] = e[q2];
    } else {
      int e[4];
      moved(g, y, a, -1, e);
#pragma unroll
      for (int q2 = 0; q2 < 4; q2++) y[q2] = e[q2];
      M = mul_nd(M, L.at(g, y, a));
    }
  }
  Links<T>{out, g.Vh}.store(0, par, h, M);
}

// For image blockIdx.y and every site x: the loops with spatial side S(x) (its line k, from x to
// x + D, D = k d) and time extents T = 1..tmax, Re tr[ S(x) B_T(x+D) S(x+T)^dag A_T(x)^dag ],
// A_T(y) = U_3(y) ... U_3(y+(T-1)), summed per block into
// part[(image * tmax + T - 1) * gridDim.x + blockIdx.x].  Each lane carries P = S(x) B_T(x+D) and
// A_T(x), one product each per T, and forms Q = A_T(x) S(x+T): Re tr(P Q^dag).
template <typename T, int BS>
__global__ __launch_bounds__(BS) void k_wloop(Geom g, const V2<T> *__restrict__ U,
                                              const LoopImage<T> *__restrict__ imgs, int k, int tmax,
                                              double *__restrict__ part) {
  const LoopImage<T> &im = imgs[blockIdx.y];
  const V2<T> *S = (k & 1) ? im.a : im.b;
  const int D0 = k * im.path.d[0], D1 = k * im.path.d[1], D2 = k * im.path.d[2];
  const int nbp = gridDim.x >> 1;
  const int par = blockIdx.x >= nbp;
  // tiles of one parity in contiguous ranges per XCD (xcd_range); the block sums are stored by tile
  const int tile = par * nbp + xcd_range((int)blockIdx.x - par * nbp, nbp);
  const int h = (tile - par * nbp) * BS + threadIdx.x;
  const bool live = h < g.Vh;
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  const Links<T> Sf{const_cast<V2<T> *>(S), g.Vh};
  int c[4] = {0, 0, 0, 0}, cd[4] = {0, 0, 0, 0};
  M3<T> P, A;
  if (live) {
    coords_of(g, par, h, c);
    shifted(g, c, D0, D1, D2, 0, cd);
    P = Sf.load(0, par, h);
    A = m_ident<T>();
  }
  double *pt = part + (size_t)blockIdx.y * tmax * gridDim.x;
  for (int t = 1; t <= tmax; t++) {
    double val = 0.0;
    if (live) {
      int e[4];
      shifted(g, c, 0, 0, 0, t - 1, e);
      A = mul(A, L.at(g, e, 3));
      shifted(g, cd, 0, 0, 0, t - 1, e);
      P = mul(P, L.at(g, e, 3));
      shifted(g, c, 0, 0, 0, t, e);
      const M3<T> Q = mul(A, Sf.load(0, parity_of(e), half_index(g, e)));
#pragma unroll
      for (int q = 0; q < 9; q++)
        val += (double)P.e[q].re * (double)Q.e[q].re + (double)P.e[q].im * (double)Q.e[q].im;
    }
    const double s = block_sum<BS>(val);
    if (threadIdx.x == 0) pt[(size_t)(t - 1) * gridDim.x + tile] = s;
  }
}

// res[t] += sum over the images, in order, of weight * sum_b part[(image * tmax + t) * nb + b]
// (each block sum in a fixed order); one block per t
template <typename T>
__global__ __launch_bounds__(256) void k_wloop_final(const double *__restrict__ part, int nb, int nimg, int tmax,
                                                     const LoopImage<T> *__restrict__ imgs, double *res) {
  double r = threadIdx.x == 0 ? res[blockIdx.x] : 0.0;
  for (int i = 0; i < nimg; i++) {
    const double s = sum_partials<256>(part + ((size_t)i * tmax + blockIdx.x) * nb, nb);
    if (threadIdx.x == 0) r += imgs[i].weight * s;
  }
  if (threadIdx.x == 0) res[blockIdx.x] = r;
}

__global__ __launch_bounds__(256) void k_zero(double *p, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

// ------------------------------------------- Wilson loops in the temporal gauge
// With h(x, 0) = 1 and h(x, t+1) = h(x, t) U_3(x, t), t running on past the period, the time sides of
// every loop become 1 and a loop is Re tr[ S(x, t) S(x, t+T)^dag ], S the lines transformed by h: a
// product of 18 reals per (site, T, image) instead of three complex 3x3 products.  It needs unitary
// time links only (k_wl_gauge checks them); the spatial links may be any matrices.  20^3x40, FP32,
// six directions up to five copies, T <= 10: 36.9 ms with k_line and k_wloop, 6.8 ms here (k_wl_corr
// 4.3, k_wl_line 1.7, k_wl_links and k_wl_gauge 0.6).  The general kernels keep what this form does not
// take: non-unitary time links, tmax too long for a block (wl_plan), too little scratch.
// Fields in this form are [t][element][s] complex, s = x + Lx (y + Ly z), t < Lt + tmax.

// Largest |(U_3 U_3^dag - 1)_ij| (real and imaginary parts) accepted.  The gauge takes each time link's
// unitary part, where the general path multiplies the link as it is.  The scale that all time links have
// in common is put back (k_wl_final); what is left out is how a link's own deviation goes with the loops
// it is in, and that no sum over sites averages away.  The lines lie where it stays below what the
// general path rounds away: largest error of W(R <= 3, T <= 10) at 20^3x40 against 64-bit mathematics, gauged
// and general, FP32 fields as given (off by 1.0e-7, transformed or vortex-removed ones by 1.7e-7) 8e-11
// and 1.1e-10, after one smearing step (4e-7) 1.4e-10 and 1.1e-10, after ten (1.2e-6) 8e-10 and 1.3e-10; FP64
// fields (1.1e-15) and after 80 smearing steps (8e-15) 1-3e-16 both ways.
template <typename T> struct WlTol;
template <> struct WlTol<float> { static constexpr double v = 2.4e-7; };
template <> struct WlTol<double> { static constexpr double v = 1e-14; };
// R: the slices of S_k that a wave holds in registers; Q: the slices t whose loops it sums (all read
// from LDS, so that every wave of a block has a share).  With these a wave needs at most 256 registers (two waves per SIMD).
template <typename T> struct WlTile;
template <> struct WlTile<float> { static constexpr int R = 8, Q = 5; };
template <> struct WlTile<double> { static constexpr int R = 4, Q = 3; };
// Waves of a block of k_wl_corr at most: four where tmax leaves a block at least half of its slices
// to sum the loops of, since two blocks then share a CU and one computes while the other waits
// for its lines or at a barrier; else eight.
constexpr int WL_WAVES = 8;
template <typename T> constexpr int wl_waves(int tmax) { return 2 * tmax <= 4 * WlTile<T>::R ? 4 : WL_WAVES; }

// one matrix of a [t][element][s] field, o = s * sizeof(complex)
template <typename V> struct wl_real;
template <> struct wl_real<float2> { using type = float; };
template <> struct wl_real<double2> { using type = double; };
template <typename V> __device__ __forceinline__ M3<typename wl_real<V>::type> wl_load(const V *f, int t, int Vs, unsigned o) {
  M3<typename wl_real<V>::type> m;
#pragma unroll
  for (int k = 0; k < 9; k++) {
    const V v = ld_plane(f + (size_t)(t * 9 + k) * Vs, o);
    m.e[k] = cx<typename wl_real<V>::type>{v.x, v.y};
  }
  return m;
}
template <typename V, typename T> __device__ __forceinline__ void wl_store(V *f, int t, int Vs, unsigned o, const M3<T> &m) {
#pragma unroll
  for (int k = 0; k < 9; k++) {
    V v;
    v.x = m.e[k].re;
    v.y = m.e[k].im;
    st_plane(f + (size_t)(t * 9 + k) * Vs, o, v);
  }
}
__device__ __forceinline__ void wl_site(const Geom &g, int s, int c[4]) {
  const int ry = s / g.L[0];
  c[0] = s - ry * g.L[0];
  c[2] = ry / g.L[1];
  c[1] = ry - c[2] * g.L[1];
}
__device__ __forceinline__ int wl_index(const Geom &g, const int c[4]) { return c[0] + g.L[0] * (c[1] + g.L[1] * c[2]); }

// h in FP64, 64 spatial sites per block.  Each product h U_3 is brought back to unitarity by one Newton
// step of the polar decomposition, so h stays unitary to FP64 rounding however far it runs, and what U_3
// itself is off by, which is measured there, is left out.  The chain of products along t is cut into
// WL_WAVES pieces: each wave multiplies its piece out, takes the pieces before it from LDS and goes
// through its piece again (50 slices: 59 us as one chain).
template <typename T>
__global__ __launch_bounds__(64 * WL_WAVES) void k_wl_gauge(Geom g, const V2<T> *__restrict__ U,
                                                           double2 *__restrict__ H, int TE, double *__restrict__ dev, int *bad_out) {
  __shared__ double2 piece[WL_WAVES - 1][9][64];
  const int Vs = g.L[0] * g.L[1] * g.L[2];
  const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6);
  const bool live = (int)blockIdx.x * 64 + lane < Vs;
  const int s = live ? (int)blockIdx.x * 64 + lane : 0;
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  int c[4];
  wl_site(g, s, c);
  const int p0 = (c[0] + c[1] + c[2]) & 1, Sh = Vs >> 1, n = (TE + WL_WAVES - 1) / WL_WAVES;
  const int lo = wave * n < TE ? wave * n : TE, hi = lo + n < TE ? lo + n : TE;
  bool bad = false;
  double tr = 0.0, off = 0.0;  // tr(U U^dag - 1) of the last link; of the block's own links
  auto link = [&](int te) -> M3<T> {
    const int t = te % g.L[3];
    return L.load(3, (p0 + t) & 1, t * Sh + (s >> 1));
  };
  // the unitary part of m: (3 - m m^dag) / 2 m
  auto unitary = [&](const M3<double> &m) -> M3<double> {
    M3<double> q = mul_nd(m, m);
    tr = (q.e[0].re - 1.0) + (q.e[4].re - 1.0) + (q.e[8].re - 1.0);
#pragma unroll
    for (int k = 0; k < 9; k++) {
      const double one = k % 4 == 0 ? 1.0 : 0.0;
      bad = bad || !(fabs(q.e[k].re - one) <= WlTol<T>::v) || !(fabs(q.e[k].im) <= WlTol<T>::v);
      q.e[k] = cx<double>{1.5 * one - 0.5 * q.e[k].re, -0.5 * q.e[k].im};
    }
    return mul(q, m);
  };
  M3<double> h = m_ident<double>();
  if (wave < WL_WAVES - 1) {
    for (int te = lo; te < hi; te++) h = unitary(mul(h, m_cvt<double>(link(te))));
#pragma unroll
    for (int k = 0; k < 9; k++) piece[wave][k][lane] = make_double2(h.e[k].re, h.e[k].im);
  }
  __syncthreads();
  h = m_ident<double>();
  for (int w = 0; w < wave; w++) {
    M3<double> p;
#pragma unroll
    for (int k = 0; k < 9; k++) {
      const double2 v = piece[w][k][lane];
      p.e[k] = cx<double>{v.x, v.y};
    }
    h = mul(h, p);
  }
  h = unitary(h);
  for (int te = lo; te < hi; te++) {
    const M3<T> u = link(te);
    if (live) wl_store(H, te, Vs, (unsigned)s * 16u, h);
    h = unitary(mul(h, m_cvt<double>(u)));
    if (live && te < g.L[3]) off += tr;
  }
  off = block_sum<64 * WL_WAVES>(off);
  if (threadIdx.x == 0) dev[blockIdx.x] = off;
  if (bad) *bad_out = 1;  // the same value from every lane
}

// The spatial links in the gauge, h(x, t) U_j(x, t) h(x+j, t)^dag for t < TE (links at t modulo Lt),
// formed in FP64 and rounded once: N + j TE 9 Vs.  One block per (256 spatial sites, t).
template <typename T>
__global__ __launch_bounds__(256) void k_wl_links(Geom g, const V2<T> *__restrict__ U,
                                                  const double2 *__restrict__ H, int TE, V2<T> *__restrict__ N) {
  const int Vs = g.L[0] * g.L[1] * g.L[2], nsb = (Vs + 255) / 256;
  const int te = (int)blockIdx.x / nsb, s = ((int)blockIdx.x - te * nsb) * 256 + (int)threadIdx.x;
  if (s >= Vs) return;
  const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
  int c[4];
  wl_site(g, s, c);
  c[3] = te % g.L[3];
  const M3<double> hx = wl_load(H, te, Vs, (unsigned)s * 16u);
#pragma unroll
  for (int j = 0; j < 3; j++) {
    int e[4];
    moved(g, c, j, +1, e);
    const M3<double> hd = wl_load(H, te, Vs, (unsigned)wl_index(g, e) * 16u);
    const M3<T> r = m_cvt<T>(mul_nd(mul(hx, m_cvt<double>(L.at(g, c, j))), hd));
    wl_store(N + (size_t)j * TE * 9 * Vs, te, Vs, (unsigned)s * (unsigned)sizeof(V2<T>), r);
  }
}

// S_1(x, t): the image's path from x in the gauged links, for every image and t < TE; one block per
// (256 spatial sites, t, image).  Bound by its loads from the caches, one matrix per step of the path
// (15 GB in 1.7 ms at 20^3x40).
template <typename T>
__global__ __launch_bounds__(256) void k_wl_line(Geom g, const V2<T> *__restrict__ N, LoopImages imgs, int TE,
                                                 V2<T> *__restrict__ A) {
  const LoopPath &im = imgs.img[blockIdx.y];
  const int Vs = g.L[0] * g.L[1] * g.L[2], nsb = (Vs + 255) / 256;
  const int blk = xcd_range((int)blockIdx.x, (int)gridDim.x);
  const int te = blk / nsb, s = (blk - te * nsb) * 256 + (int)threadIdx.x;
  if (s >= Vs) return;
  int y[4];
  wl_site(g, s, y);
  y[3] = te;
  // the link of step q, from y, which moves on to the step's end; the next step's link is loaded
  // before the product with this one
  auto step = [&](int q) -> M3<T> {
    const int st = im.s[q], a = (st > 0 ? st : -st) - 1;
    int e[4];
    moved(g, y, a, st > 0 ? +1 : -1, e);
    const unsigned o = (unsigned)wl_index(g, st > 0 ? y : e) * (unsigned)sizeof(V2<T>);
#pragma unroll
    for (int q2 = 0; q2 < 3; q2++) y[q2] = e[q2];
    return wl_load(N + (size_t)a * TE * 9 * Vs, te, Vs, o);
  };
  M3<T> M = step(0);
  if (im.n == 1) {
    if (im.s[0] < 0) M = dag(M);
  } else {
    M3<T> u = step(1);
    if (im.s[0] < 0) M = dag(M);
    for (int q = 1; q < im.n; q++) {
      M3<T> next = u;
      if (q + 1 < im.n) next = step(q + 1);
      M = im.s[q] > 0 ? mul(M, u) : mul_nd(M, u);
      u = next;
    }
  }
  wl_store(A + (size_t)blockIdx.y * TE * 9 * Vs, te, Vs, (unsigned)s * (unsigned)sizeof(V2<T>), M);
}

// Sums of N values per lane over the 64 lanes of a wave (N a power of two up to 16): at each step the
// two halves of the lanes keep one half of the values each, so N + 5 - log2(N) exchanges do instead of
// 6 N.  The total of value i ends in the lanes whose upper bits spell i; returns that value's index.
template <int N, int OFF = 32> __device__ __forceinline__ int wave_sum_many(double *v) {
  if constexpr (N > 1) {
    constexpr int n = N / 2;
    const bool up = ((int)threadIdx.x & OFF) != 0;
#pragma unroll
    for (int i = 0; i < n; i++) {
      const double send = up ? v[i] : v[i + n], keep = up ? v[i + n] : v[i];
      v[i] = keep + __shfl_xor(send, OFF, 64);
    }
    return (up ? n : 0) + wave_sum_many<n, OFF / 2>(v);
  } else {
#pragma unroll
    for (int off = OFF; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
    return 0;
  }
}

// the compiler may not compute what follows from x before y is known (a register-pressure hint)
template <typename T, typename S> __device__ __forceinline__ void opaque_after(T &x, S &y) {
#if defined(__HIP_DEVICE_COMPILE__)
  __asm__ volatile("" : "+v"(x), "+v"(y));
#else
  (void)x;
  (void)y;
#endif
}

// part[((image * rmax + k - 1) * tmax + T - 1) * gridDim.x + block] = sums of Re tr[S_k(x, t) S_k(x, t+T)^dag]
// over the block's 64 spatial sites and its own range of t, for every k <= rmax and T <= tmax.
// A wave holds S_k for R consecutive slices of 64 spatial sites in registers through all k
// (S_k(x) = S_{k-1}(x) S_1(x + (k-1) d): one matrix load and one product per site and k); the block's
// waves cover the block's range of t and the tmax slices after it.  The correlations take one element
// of the matrices at a time: every wave leaves its R slices' element in LDS and sums the loops of Q
// slices t from there.  Products and sums in FP64, for TC extents T at once (TC >= tmax, or 16 and
// several rounds).
// Bound by both its VALU (3,000 instructions per wave and k, 2.4 of its 4.3 ms at 20^3x40, a third of
// them FP64 FMAs) and the read of each image's line once per k from beyond L2 (17 GB, 4 TB/s): with
// two waves per SIMD the two overlap only in part.
template <typename T, int TC, int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_wl_corr(Geom g, const V2<T> *__restrict__ A, LoopImages imgs,
                                                          int TE, int own, int rmax, int tmax,
                                                          double *__restrict__ part) {
  constexpr int R = WlTile<T>::R, Q = WlTile<T>::Q;
  constexpr int ROWS = NW * R + Q + TC;  // read past the slices held, for extents above tmax or with x = 0
  constexpr int TP = TC > 8 ? 16 : TC;
  __shared__ V2<T> ex[2][ROWS * 64];
  const LoopPath &im = imgs.img[blockIdx.y];
  const int Vs = g.L[0] * g.L[1] * g.L[2], nsc = (Vs + 63) / 64;
  const int lane = threadIdx.x & 63, wave = wave_uniform(threadIdx.x >> 6), nw = blockDim.x >> 6;
  // each XCD takes a contiguous range of (t range, spatial chunk), so the shifted lines are shared
  const int blk = xcd_range((int)blockIdx.x, (int)gridDim.x), seg = blk / nsc;
  const int s = (blk - seg * nsc) * 64 + lane;
  const bool live = s < Vs;
  const int tb = seg * own, tend = tb + own < g.L[3] ? tb + own : g.L[3];
  const int t0 = tb + wave * R;  // the first slice held
  const int u0 = wave * Q;       // the first row whose loops are summed
  int c[4];
  wl_site(g, s, c);
  c[3] = 0;
  const V2<T> *a = A + (size_t)blockIdx.y * TE * 9 * Vs;
  auto shift = [&](int k) -> unsigned {
    if (!live) return 0u;
    int e[4];
    shifted(g, c, (k - 1) * im.d[0], (k - 1) * im.d[1], (k - 1) * im.d[2], 0, e);
    return (unsigned)wl_index(g, e) * (unsigned)sizeof(V2<T>);
  };
  // rows past the field and idle lanes hold zeros
  for (int i = nw * R * 64 + (int)threadIdx.x; i < ROWS * 64; i += (int)blockDim.x) ex[0][i] = ex[1][i] = V2<T>{};
  M3<T> S[R];
  for (int k = 1; k <= rmax; k++) {
    unsigned o = shift(k);
#pragma unroll
    for (int r = 0; r < R; r++) {
      M3<T> m = m_zero<T>();
      if (r > 2) opaque_after(o, S[r - 3].e[8].im);  // three matrices in flight, not all R
      if (live && t0 + r < TE) m = wl_load(a, t0 + r, Vs, o);
      if (k == 1) S[r] = m;
      else S[r] = mul(S[r], m);
    }
    for (int base = 0; base < tmax; base += TC) {
      double acc[TP];
#pragma unroll
      for (int i = 0; i < TP; i++) acc[i] = 0.0;
#pragma unroll
      for (int q = 0; q < 9; q++) {
#pragma unroll
        for (int r = 0; r < R; r++) {
          V2<T> v;
          v.x = S[r].e[q].re;
          v.y = S[r].e[q].im;
          ex[q & 1][(wave * R + r) * 64 + lane] = v;
        }
        __syncthreads();
        if (tb + u0 < tend) {
          double xr[Q], xi[Q];
#pragma unroll
          for (int r = 0; r < Q; r++) {
            const bool in = tb + u0 + r < tend;
            const V2<T> v = ex[q & 1][(u0 + r) * 64 + lane];
            xr[r] = in ? (double)v.x : 0.0;
            xi[r] = in ? (double)v.y : 0.0;
          }
#pragma unroll
          for (int j = 1; j < Q + TC; j++) {  // row u0 + base + j
            const V2<T> v = ex[q & 1][(u0 + base + j) * 64 + lane];
            const double wr = (double)v.x, wi = (double)v.y;
#pragma unroll
            for (int r = (j - TC > 0 ? j - TC : 0); r < (j < Q ? j : Q); r++) {
              acc[j - r - 1] = fma_t(xr[r], wr, acc[j - r - 1]);
              acc[j - r - 1] = fma_t(xi[r], wi, acc[j - r - 1]);
            }
          }
        }
      }
      // the waves' sums through buffer 1, last read before the barrier of the ninth element
      double *red = (double *)ex[1];
      const int i = wave_sum_many<TP>(acc);
      if ((lane & (64 / TP - 1)) == 0) red[wave * TP + i] = acc[0];
      __syncthreads();
      if ((int)threadIdx.x < TC && base + (int)threadIdx.x < tmax) {
        double v = 0.0;
        for (int w = 0; w < nw; w++) v += red[w * TP + threadIdx.x];
        part[((size_t)((int)blockIdx.y * rmax + k - 1) * tmax + base + threadIdx.x) * gridDim.x + blk] = v;
      }
    }
  }
}

// res[i] += sum over the images of weight * sum over the blocks of part, i = (k - 1) tmax + T - 1: one
// block per i, terms in a fixed order.  The 2 T time links of a loop carry the mean scale that the gauge
// left out, 1 + norm * sum of dev.
__global__ __launch_bounds__(256) void k_wl_final(const double *__restrict__ part, int nb, LoopImages imgs, int nres,
                                                  int tmax, const double *__restrict__ dev, int ndev, double norm,
                                                  double *res) {
  double v = 0.0, e = 0.0;
  for (int b = threadIdx.x; b < ndev; b += 256) e += dev[b];
  e = block_sum<256>(e);
  for (int i = 0; i < imgs.n; i++) {
    const double *p = part + ((size_t)i * nres + blockIdx.x) * nb;
    const double w = imgs.img[i].weight;
    for (int b = threadIdx.x; b < nb; b += 256) v += w * p[b];
  }
  v = block_sum<256>(v);
  if (threadIdx.x == 0) res[blockIdx.x] += v * exp(2.0 * (blockIdx.x % tmax + 1) * log1p(norm * e));
}

}  // namespace mcg
