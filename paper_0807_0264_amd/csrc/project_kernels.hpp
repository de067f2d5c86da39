// project_kernels.hpp -- centre projection and vortex counting kernels (launchers in k_project.hip).
#pragma once

#include "internal.hpp"

namespace mcg {

// One thread per pair of sites 2h, 2h + 1.  pairs: Z is 2-byte aligned, so the two integers of a pair
// go out in one store.  min_margin partials: one per block, in any order.  Bound by HBM: U and G once
// and Z written, 436 bytes per site (FP32 links).  32^3x64: 307 us with lexicographic tiles and byte
// stores, 228 us now (1.52 GB read, at the rate of the last-level cache).
// LD: the links' loads stream (streaming(); 16^3x32 FP32 17.9 us without, 19.8 with; without G, when the
// links' diagonals alone are read, 32^3x64 FP32 60 and 75).
template <typename T, bool LD>
__global__ __launch_bounds__(256) void k_center_project(Geom g, const V2<T> *__restrict__ U,
                                                        const double2 *__restrict__ G,
                                                        int8_t *__restrict__ Z, double *part, int pairs,
                                                        int tiled) {
  const int h = site_of_block(g, tiled);
  double mmin = 10.0;
  if (h >= 0) {
    const Links<T> L{const_cast<V2<T> *>(U), g.Vh};
    const Gauge gg{const_cast<double2 *>(G), g.Vh};
    const double s3 = 0.86602540378443864676;  // sqrt(3)/2
    int zz[4] = {0, 0, 0, 0};  // the integers of both sites, one byte each
    for (int par = 0; par < 2; par++) {
      int c[4];
      coords_of(g, par, h, c);
      const int i = lex_index(g, c);
      M3<double> Gx;
      if (G) Gx = gg.load(par, h);
#pragma unroll
      for (int mu = 0; mu < 4; mu++) {
        const M3<double> u = m_cvt<double>(L.template load_as<LD>(mu, par, h));
        cx<double> t;
        if (G) {
          int e[4];
          moved(g, c, mu, +1, e);
          const M3<double> Gn = gg.load(1 - par, half_index(g, e));
          const M3<double> a = mul(Gx, u);
          // tr(a Gn^dag) = sum_ij a_ij conj(Gn_ij)
          t = cx<double>{0.0, 0.0};
#pragma unroll
          for (int k = 0; k < 9; k++) t = t + mulc(a.e[k], Gn.e[k]);
        } else {
          t = trace(u);
        }
        int m = 0;
        double margin = 0.0;
        if (t.re != 0.0 || t.im != 0.0) {
          const double r0 = t.re, rp = -0.5 * t.re + s3 * t.im, rm = -0.5 * t.re - s3 * t.im;
          double best = r0;
          if (rp > best) { best = rp; m = 1; }
          if (rm > best) { best = rm; m = -1; }
          // t e^{-2 pi i m/3}
          cx<double> rot = t;
          if (m == 1) rot = t * cx<double>{-0.5, -s3};
          if (m == -1) rot = t * cx<double>{-0.5, s3};
          margin = 1.04719755119659774615 - fabs(atan2(rot.im, rot.re));
        }
        if (pairs) zz[mu] |= (m & 0xff) << (8 * (i & 1));
        else Z[(size_t)mu * g.V + i] = (int8_t)m;
        mmin = fmin(mmin, margin);
      }
    }
    if (pairs) {
#pragma unroll
      for (int mu = 0; mu < 4; mu++) ((uint16_t *)(Z + (size_t)mu * g.V))[h] = (uint16_t)zz[mu];
    }
  }
  const double s = block_min<256>(mmin);
  if (threadIdx.x == 0) part[blockIdx.x] = s;
}

// 1024 threads: the partials of 32^3x64 arrive in one round trip of four loads per thread
__global__ __launch_bounds__(1024) void k_min_final(const double *part, int n, double *out) {
  double v = 10.0;
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 1024) v = fmin(v, part[i]);
  v = block_min<1024>(v);
  if (threadIdx.x == 0) *out = v;
}

// the n = 1 and n = 2 counts of a thread's sites: added over the wave, then over the four waves through
// LDS, and at most 12 atomic additions per block
__device__ __forceinline__ void add_counts(const unsigned int cnt[12], unsigned long long *counts) {
  __shared__ unsigned int wsum[4][12];
#pragma unroll
  for (int k = 0; k < 12; k++) {
    unsigned int v = cnt[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 12) {
    const unsigned long long v = (unsigned long long)wsum[0][threadIdx.x] + wsum[1][threadIdx.x] +
                                 wsum[2][threadIdx.x] + wsum[3][threadIdx.x];
    if (v) atomicAdd(&counts[threadIdx.x], v);
  }
}

// Four sites along x per thread, for Lx a multiple of 4 and Z 4-byte aligned: the integers come as
// words, 16 loads for four sites instead of 64 loads of a byte (the +x neighbours are the words
// themselves shifted by a byte, with the first byte of the next word along x).  Any int8 values.
// Bound by latency and by its 12 reductions; 32^3x64: 42 us by bytes, 20 us.
__global__ __launch_bounds__(256) void k_count_vortices4(Geom g, const int8_t *__restrict__ Z,
                                                         unsigned long long *counts) {
  unsigned int cnt[12];
#pragma unroll
  for (int k = 0; k < 12; k++) cnt[k] = 0;
  for (int w = blockIdx.x * 256 + threadIdx.x; w < g.V / 4; w += gridDim.x * 256) {
    const int i = 4 * w;
    int c[4];
    const int r = i / g.L[0], r2 = r / g.L[1];
    c[0] = i - r * g.L[0];
    c[1] = r - r2 * g.L[1];
    c[3] = r2 / g.L[2];
    c[2] = r2 - c[3] * g.L[2];
    auto word = [&](int mu, int j) -> uint32_t { return *(const uint32_t *)(Z + (size_t)mu * g.V + j); };
    uint32_t m[4], n[4][4];  // n[mu][nu] = Z_nu at x + mu
    const int nx = c[0] + 4 == g.L[0] ? i - c[0] : i + 4;
#pragma unroll
    for (int nu = 0; nu < 4; nu++) m[nu] = word(nu, i);
#pragma unroll
    for (int nu = 1; nu < 4; nu++) n[0][nu] = (m[nu] >> 8) | (word(nu, nx) << 24);
#pragma unroll
    for (int mu = 1; mu < 4; mu++) {
      int e[4];
      moved(g, c, mu, +1, e);
      const int j = lex_index(g, e);
#pragma unroll
      for (int nu = 0; nu < 4; nu++)
        if (nu != mu) n[mu][nu] = word(nu, j);
    }
#pragma unroll
    for (int b = 0; b < 4; b++) {
      auto at = [&](uint32_t v) -> int { return (int8_t)(v >> (8 * b)); };
      int pl = 0;
#pragma unroll
      for (int mu = 0; mu < 4; mu++)
#pragma unroll
        for (int nu = mu + 1; nu < 4; nu++, pl++) {
          // + 1023 = 3 * 341 > 4 * 128: never negative
          const unsigned q = (unsigned)(at(m[mu]) + at(n[mu][nu]) - at(n[nu][mu]) - at(m[nu]) + 1023) % 3u;
          cnt[2 * pl] += q == 1u;
          cnt[2 * pl + 1] += q == 2u;
        }
    }
  }
  add_counts(cnt, counts);
}

// Each thread walks sites i, i + grid size, ... and counts in registers; the block adds its counts
// (wave shuffles, then the four waves through LDS) and makes at most 12 atomic additions, so the
// integers meet in few atomics (one per site wave had serialised on the 12 counters: ~1 ms at
// 32^3x64).  Integer sums: the result does not depend on the order.
__global__ __launch_bounds__(256) void k_count_vortices(Geom g, const int8_t *__restrict__ Z,
                                                        unsigned long long *counts) {
  unsigned int cnt[12];
#pragma unroll
  for (int k = 0; k < 12; k++) cnt[k] = 0;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < g.V; i += gridDim.x * 256) {
    int c[4];
    int r = i / g.L[0];
    c[0] = i - r * g.L[0];
    int r2 = r / g.L[1];
    c[1] = r - r2 * g.L[1];
    c[3] = r2 / g.L[2];
    c[2] = r2 - c[3] * g.L[2];
    int nb[4];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) {
      int e[4];
      moved(g, c, mu, +1, e);
      nb[mu] = lex_index(g, e);
    }
    int m[4];
#pragma unroll
    for (int mu = 0; mu < 4; mu++) m[mu] = Z[(size_t)mu * g.V + i];
    int pl = 0;
#pragma unroll
    for (int mu = 0; mu < 4; mu++)
#pragma unroll
      for (int nu = mu + 1; nu < 4; nu++, pl++) {
        const int s = m[mu] + (int)Z[(size_t)nu * g.V + nb[mu]] - (int)Z[(size_t)mu * g.V + nb[nu]] - m[nu];
        const int n = ((s % 3) + 3) % 3;
        if (n == 1) cnt[2 * pl]++;
        if (n == 2) cnt[2 * pl + 1]++;
      }
  }
  add_counts(cnt, counts);
}

}  // namespace mcg
