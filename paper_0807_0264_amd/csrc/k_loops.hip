// k_loops.hip -- the centre part of a projected field and its remainder, and
// Wilson loops W(R, T) averaged over all sites (Sec. III.B of arXiv:0807.0264).
//   vortex-only     Z_mu(x) = exp(2 pi i m_mu(x) / 3) 1
//   vortex-removed  Z_mu(x)^dag U^G_mu(x)
//   W(R, T) = < Re tr(loop) / 3 >, the spatial side a path of unit steps
//   (built as a line field by k_line), the time sides straight.

#include <algorithm>

#include "loops_kernels.hpp"

namespace mcg {

template <typename T>
hipError_t launch_vortex_field(const Geom &g, const void *U, const double *G, const int8_t *Z, int mode, void *out,
                               hipStream_t s) {
  const size_t links = (size_t)g.V * 36 * sizeof(V2<T>), transform = G ? (size_t)g.V * 9 * sizeof(double2) : 0;
  // Centres alone are written, not read: ordinary stores up to twice the cache, 20^3x40 FP32 15 us (18
  // streaming), 24^3x48 28 (38), 32^4 48 (59), FP64 24^3x48 76 (77); then 32^4 FP64 111 (107), 32^3x64 FP32
  // 116 (113) and FP64 228 (220)
  const Streaming st = mode == 0 ? Streaming{false, links > 2 * LLC_BYTES} : streaming(links + transform, links);
  const int tiled = mode != 0 && G && site_tiled(g), nb = site_blocks(g, tiled);
#define MCG_VF(LD, ST)                                                                                           \
  k_vortex_field<T, LD, ST><<<nb, 256, 0, s>>>(g, (const V2<T> *)U, (const double2 *)G, Z, mode, (V2<T> *)out, tiled)
  if (st.loads) MCG_VF(true, true);
  else if (st.stores) MCG_VF(false, true);
  else MCG_VF(false, false);
#undef MCG_VF
  return hipGetLastError();
}

int line_blocks(const Geom &g) { return 2 * ((g.Vh + 255) / 256); }

template <typename T>
hipError_t launch_lines(const Geom &g, const void *U, const LoopImage<T> *imgs, int nimg, int k, hipStream_t s) {
  k_line<T><<<dim3(line_blocks(g), nimg), 256, 0, s>>>(g, (const V2<T> *)U, imgs, k);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_wloops(const Geom &g, const void *U, const LoopImage<T> *imgs, int nimg, int k, int tmax,
                         double *part, double *res, hipStream_t s) {
  const int nb = line_blocks(g);
  k_wloop<T, 256><<<dim3(nb, nimg), 256, 0, s>>>(g, (const V2<T> *)U, imgs, k, tmax, part);
  k_wloop_final<T><<<tmax, 256, 0, s>>>(part, nb, nimg, tmax, imgs, res);
  return hipGetLastError();
}

hipError_t launch_zero(double *p, int n, hipStream_t s) {
  k_zero<<<(n + 255) / 256, 256, 0, s>>>(p, n);
  return hipGetLastError();
}

template <typename T> WlPlan wl_plan(const Geom &g, int tmax) {
  constexpr int R = WlTile<T>::R, Q = WlTile<T>::Q;
  WlPlan p{};
  const int Lt = g.L[3], Vs = g.L[0] * g.L[1] * g.L[2];
  p.TE = Lt + tmax;
  // a block holds its own slices and tmax more, and sums the loops of its own
  const int waves = wl_waves<T>(tmax), most = std::min(waves * R - tmax, waves * Q);
  if (most < Q) return p;
  p.nseg = (Lt + most - 1) / most;
  p.own = (Lt + p.nseg - 1) / p.nseg;
  p.nseg = (Lt + p.own - 1) / p.own;
  p.nw = std::max((p.own + tmax + R - 1) / R, (p.own + Q - 1) / Q);
  p.nblk = p.nseg * ((Vs + 63) / 64);
  p.ok = true;
  return p;
}

int wl_gauge_blocks(const Geom &g) { return (g.L[0] * g.L[1] * g.L[2] + 63) / 64; }
template <typename T>
hipError_t launch_wl_gauge(const Geom &g, const void *U, void *H, int TE, double *dev, int *bad, hipStream_t s) {
  k_wl_gauge<T><<<wl_gauge_blocks(g), 64 * WL_WAVES, 0, s>>>(g, (const V2<T> *)U, (double2 *)H, TE, dev, bad);
  return hipGetLastError();
}
template <typename T>
hipError_t launch_wl_links(const Geom &g, const void *U, const void *H, void *N, int TE, hipStream_t s) {
  const int Vs = g.L[0] * g.L[1] * g.L[2];
  k_wl_links<T><<<TE * ((Vs + 255) / 256), 256, 0, s>>>(g, (const V2<T> *)U, (const double2 *)H, TE, (V2<T> *)N);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_wl_loops(const Geom &g, const void *N, const LoopImages &imgs, const WlPlan &plan,
                           int rmax, int tmax, void *A, double *part, const double *dev, double *res, hipStream_t s) {
  const int Vs = g.L[0] * g.L[1] * g.L[2];
  const dim3 gl(plan.TE * ((Vs + 255) / 256), imgs.n), gc(plan.nblk, imgs.n);
  k_wl_line<T><<<gl, 256, 0, s>>>(g, (const V2<T> *)N, imgs, plan.TE, (V2<T> *)A);
#define MCG_WL(TC, NW) \
  k_wl_corr<T, TC, NW><<<gc, 64 * plan.nw, 0, s>>>(g, (const V2<T> *)A, imgs, plan.TE, plan.own, rmax, tmax, part)
// tmax from LO to HI: built for the block sizes that wl_waves gives there
#define MCG_WL_RANGE(TC, LO, HI)                                  \
  do {                                                            \
    if constexpr (wl_waves<T>(LO) == 4) { if (four) MCG_WL(TC, 4); } \
    if constexpr (wl_waves<T>(HI) == 8) { if (!four) MCG_WL(TC, 8); } \
  } while (0)
  // extents at once: the smallest set that holds tmax, else rounds of 16.  A set for 10, between the
  // powers of two: at tmax 9 and 10 3 % less time than with 12 (FP32 16^3x32, 20^3x40 and 12^3x24
  // 3.09 -> 3.00, 6.96 -> 6.76 and 1.55 -> 1.50 ms for six directions, FP64 5.12 -> 4.97, 11.5 -> 11.15 and
  // 2.13 -> 2.08)
  static_assert(WL_WAVES == 8, "the block sizes built below");
  const bool four = wl_waves<T>(tmax) == 4;
  if (tmax <= 4) MCG_WL_RANGE(4, 1, 4);
  else if (tmax <= 8) MCG_WL_RANGE(8, 5, 8);
  else if (tmax <= 10) MCG_WL_RANGE(10, 9, 10);
  else if (tmax <= 12) MCG_WL_RANGE(12, 11, 12);
  else MCG_WL_RANGE(16, 13, 1 << 16);
#undef MCG_WL_RANGE
#undef MCG_WL
  k_wl_final<<<rmax * tmax, 256, 0, s>>>(part, plan.nblk, imgs, rmax * tmax, tmax, dev, wl_gauge_blocks(g), 1.0 / (6.0 * g.V), res);
  return hipGetLastError();
}

#define MCG_LOOPS_INST(T)                                                                                  \
  template hipError_t launch_vortex_field<T>(const Geom &, const void *, const double *, const int8_t *, int, \
                                             void *, hipStream_t);                                         \
  template hipError_t launch_lines<T>(const Geom &, const void *, const LoopImage<T> *, int, int, hipStream_t); \
  template hipError_t launch_wloops<T>(const Geom &, const void *, const LoopImage<T> *, int, int, int, double *, \
                                       double *, hipStream_t);                                             \
  template WlPlan wl_plan<T>(const Geom &, int);                                                           \
  template hipError_t launch_wl_gauge<T>(const Geom &, const void *, void *, int, double *, int *, hipStream_t); \
  template hipError_t launch_wl_links<T>(const Geom &, const void *, const void *, void *, int, hipStream_t); \
  template hipError_t launch_wl_loops<T>(const Geom &, const void *, const LoopImages &, const WlPlan &, int, int, \
                                         void *, double *, const double *, double *, hipStream_t);
MCG_LOOPS_INST(float)
MCG_LOOPS_INST(double)

}  // namespace mcg
