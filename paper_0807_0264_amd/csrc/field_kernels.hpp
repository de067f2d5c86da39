// field_kernels.hpp -- layout conversion, gauge utilities and field sums (launchers in k_field.hip).
#pragma once

#include "internal.hpp"

namespace mcg {

// Layout conversion of NM matrices per site (4: links, 1: a transform).  A block takes the 2H sites
// of H half indices through LDS, so that both sides of the copy move in runs: whole sites on the
// interchange side, H consecutive complex numbers per (mu, parity, k) plane on the other.  Written
// per link from registers, each lane walked 72 bytes (FP32) of the interchange side by itself and a
// wave wrote runs of 64 bytes.  24^3x48, FP32 links: pack 87 -> 81 us, unpack 120 -> 68 us; a
// transform 53 -> 37 us either way (191 MB of links and 96 MB of transform each read and written).  32
// half indices: with 64 FP32 links take 82 and 77 us, and a small field waits for the few blocks' longer
// rounds, 8^3x16 pack 3.8 us with 32, 4.7 with 64, unpack 3.7 and 6.1 (3.6 and 4.3 from registers).
// LDS holds the matrices of a site at a stride that spreads the sites over the banks.
// A thread has up to nine loads in flight on either side.
template <typename T, int NM> struct PackTile {
  static constexpr int H = 32, N = 9 * NM, STRIDE = N | 1;
  static constexpr int AOS = (2 * H * N + 255) / 256, SOA = (2 * N * H + 255) / 256;  // rounds of 256 on each side
};
// the parity of a pair's first site (even x)
__device__ __forceinline__ int pair_parity(const Geom &g, int h) {
  const int r = h / g.hx, r2 = r / g.L[1], t = r2 / g.L[2];
  return ((r - r2 * g.L[1]) + (r2 - t * g.L[2]) + t) & 1;
}
template <typename Tin, typename Tout, int NM>
__global__ __launch_bounds__(256) void k_pack(Geom g, const V2<Tin> *__restrict__ src, V2<Tout> *__restrict__ dst) {
  using P = PackTile<Tout, NM>;
  constexpr int H = P::H, N = P::N, ST = P::STRIDE;
  __shared__ V2<Tout> m[2 * H * ST];  // [first or second site of the pair][pair][element]
  const int h0 = blockIdx.x * H, nh = g.Vh - h0 < H ? g.Vh - h0 : H;
  const V2<Tin> *in = src + (size_t)h0 * 2 * N;
#pragma unroll
  for (int r0 = 0; r0 < P::AOS; r0 += 9) {
    V2<Tin> v[9];
#pragma unroll
    for (int r = 0; r < 9; r++) {
      const int e = (r0 + r) * 256 + threadIdx.x;
      v[r] = in[r0 + r < P::AOS && e < nh * 2 * N ? e : 0];
    }
#pragma unroll
    for (int r = 0; r < 9; r++) {
      const int e = (r0 + r) * 256 + threadIdx.x, i = e / N, j = e - i * N;
      if (r0 + r < P::AOS && e < nh * 2 * N) {
        V2<Tout> w;
        w.x = (Tout)v[r].x;
        w.y = (Tout)v[r].y;
        m[((i & 1) * H + (i >> 1)) * ST + j] = w;
      }
    }
  }
  __syncthreads();
  const int hh = threadIdx.x & (H - 1);
  if (hh >= nh) return;
  const int p0 = pair_parity(g, h0 + hh);
#pragma unroll
  for (int r = 0; r < P::SOA; r++) {
    const int q = threadIdx.x / H + r * (256 / H);  // plane (mu, parity, k)
    const int mu = q / 18, par = (q - mu * 18) / 9, k = q - mu * 18 - par * 9;
    if (q < 2 * N) dst[(size_t)q * g.Vh + h0 + hh] = m[((par ^ p0) * H + hh) * ST + mu * 9 + k];
  }
}
template <typename Tin, typename Tout, int NM>
__global__ __launch_bounds__(256) void k_unpack(Geom g, const V2<Tin> *__restrict__ src, V2<Tout> *__restrict__ dst) {
  using P = PackTile<Tin, NM>;
  constexpr int H = P::H, N = P::N, ST = P::STRIDE;
  __shared__ V2<Tin> m[2 * H * ST];
  const int h0 = blockIdx.x * H, nh = g.Vh - h0 < H ? g.Vh - h0 : H;
  const int hh = threadIdx.x & (H - 1);
  if (hh < nh) {
    const int p0 = pair_parity(g, h0 + hh);
#pragma unroll
    for (int r0 = 0; r0 < P::SOA; r0 += 9) {
      V2<Tin> v[9];
#pragma unroll
      for (int r = 0; r < 9; r++) {
        const int q = threadIdx.x / H + (r0 + r) * (256 / H);
        v[r] = src[(size_t)(r0 + r < P::SOA && q < 2 * N ? q : 0) * g.Vh + h0 + hh];
      }
#pragma unroll
      for (int r = 0; r < 9; r++) {
        const int q = threadIdx.x / H + (r0 + r) * (256 / H);
        const int mu = q / 18, par = (q - mu * 18) / 9, k = q - mu * 18 - par * 9;
        if (r0 + r < P::SOA && q < 2 * N) m[((par ^ p0) * H + hh) * ST + mu * 9 + k] = v[r];
      }
    }
  }
  __syncthreads();
  V2<Tout> *out = dst + (size_t)h0 * 2 * N;
#pragma unroll
  for (int r = 0; r < P::AOS; r++) {
    const int e = r * 256 + threadIdx.x, i = e / N, j = e - i * N;
    if (e < nh * 2 * N) {
      const V2<Tin> v = m[((i & 1) * H + (i >> 1)) * ST + j];
      V2<Tout> w;
      w.x = (Tout)v.x;
      w.y = (Tout)v.y;
      out[e] = w;
    }
  }
}

// what: 0 = identity, 1 = re-unitarise
__global__ __launch_bounds__(256) void k_gauge_op(Geom g, double2 *G, int what) {
  const int h = blockIdx.x * 256 + threadIdx.x;
  if (h >= g.Vh) return;
  const Gauge gg{G, g.Vh};
  for (int par = 0; par < 2; par++) {
    M3<double> m;
    if (what == 0) {
      m = m_ident<double>();
    } else {
      m = gg.load(par, h);
      reunit(m);
    }
    gg.store(par, h, m);
  }
}

// LD, ST: the links' loads and stores stream (streaming())
template <typename T, bool LD, bool ST>
__global__ __launch_bounds__(256) void k_apply_gauge(Geom g, const V2<T> *U, const double2 *__restrict__ G,
                                                     V2<T> *out, int tiled) {
  const int h = site_of_block(g, tiled);
  if (h < 0) return;
  const Links<T> Ui{const_cast<V2<T> *>(U), g.Vh}, O{out, g.Vh};
  const Gauge gg{const_cast<double2 *>(G), g.Vh};
  for (int par = 0; par < 2; par++) {
    int c[4];
    coords_of(g, par, h, c);
    const M3<double> Gx = gg.load(par, h);
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
      int e[4];
      moved(g, c, mu, +1, e);
      const M3<double> Gn = gg.load(1 - par, half_index(g, e));
      const M3<double> u = m_cvt<double>(Ui.template load_as<LD>(mu, par, h));
      O.template store_as<ST>(mu, par, h, m_cvt<T>(mul_nd(mul(Gx, u), Gn)));
    }
  }
}

// what: 0 = sum |tr U|^2, 1 = sum_{mu<nu} Re tr U_P
template <typename T>
__global__ __launch_bounds__(256) void k_field_sum(Geom g, const V2<T> *__restrict__ U, double *part,
                                                   int what) {
  const int h = blockIdx.x * 256 + threadIdx.x;
  double r = 0.0;
  if (h < g.Vh) {
    const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
    for (int par = 0; par < 2; par++) {
      if (what == 0) {
#pragma unroll
        for (int mu = 0; mu < 4; mu++) r += tr2(L.load(mu, par, h));
      } else {
        int c[4];
        coords_of(g, par, h, c);
        M3<T> u[4];
#pragma unroll
        for (int mu = 0; mu < 4; mu++) u[mu] = L.load(mu, par, h);
#pragma unroll
        for (int mu = 0; mu < 4; mu++) {
          int e[4];
          moved(g, c, mu, +1, e);
#pragma unroll
          for (int nu = mu + 1; nu < 4; nu++) {
            int f[4];
            moved(g, c, nu, +1, f);
            // Re tr(U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag) = Re tr(P Q^dag)
            const M3<T> P = mul(u[mu], L.at(g, e, nu));
            const M3<T> Q = mul(u[nu], L.at(g, f, mu));
            r += (double)rdot(Q, P);
          }
        }
      }
    }
  }
  const double s = block_sum<256>(r);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// max over the nmu matrices per site (4: links, 1: a gauge field, FP64) of max_ij |(M M^dag - 1)_ij|,
// computed in FP64; a NaN anywhere in a matrix counts as +inf.  Per-block maxima into part.
template <typename T>
__global__ __launch_bounds__(256) void k_unitarity(Geom g, const V2<T> *__restrict__ U, int nmu, double *part) {
  const int h = blockIdx.x * 256 + threadIdx.x;
  double dev = 0.0;
  if (h < g.Vh) {
    const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
    for (int par = 0; par < 2; par++)
      for (int mu = 0; mu < nmu; mu++) {
        const M3<double> m = m_cvt<double>(L.load(mu, par, h));
        const M3<double> p = mul_nd(m, m);
#pragma unroll
        for (int k = 0; k < 9; k++) {
          const double re = p.e[k].re - ((k % 4 == 0) ? 1.0 : 0.0), im = p.e[k].im;
          const double a = fmax(fabs(re), fabs(im));
          dev = (a == a) ? fmax(dev, a) : __builtin_huge_val();
        }
      }
  }
  const double mx = -block_min<256>(-dev);
  if (threadIdx.x == 0) part[blockIdx.x] = mx;
}

__global__ __launch_bounds__(256) void k_max_final(const double *part, int n, double *out) {
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) v = fmax(v, part[i]);
  v = -block_min<256>(-v);
  if (threadIdx.x == 0) *out = v;
}

__global__ __launch_bounds__(256) void k_final_sum(const double *part, int n, double scale, double *out) {
  const double s = sum_partials<256>(part, n);
  if (threadIdx.x == 0) *out = s * scale;
}

}  // namespace mcg
