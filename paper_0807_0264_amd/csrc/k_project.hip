// k_project.hip -- centre projection and P-vortex identification
// (Sec. II.A of arXiv:0807.0264).
//   Z_mu(x) = exp(2 pi i m / 3), m maximising Re(t e^{-2 pi i m/3}) with
//   t = tr(G(x) U_mu(x) G(x+mu)^dag) in FP64 (candidates 0, +1, -1; the first
//   wins a tie; t = 0 gives m = 0); margin = pi/3 - |arg(t e^{-2 pi i m/3})|.
//   A plaquette is a P-vortex when (m_mu(x) + m_nu(x+mu) - m_mu(x+nu) - m_nu(x))
//   mod 3 is non-zero.

#include <algorithm>

#include "project_kernels.hpp"

namespace mcg {

template <typename T>
hipError_t launch_center_project(const Geom &g, const void *U, const double *G, int8_t *Z,
                                 double *part, double *min_out, hipStream_t s) {
  const size_t links = (size_t)g.V * 36 * sizeof(V2<T>);
  const size_t read = G ? links + (size_t)g.V * 9 * sizeof(double2) : links / 3;
  const int tiled = G && site_tiled(g), nb = site_blocks(g, tiled), pairs = ((uintptr_t)Z & 1) == 0;
#define MCG_CP(LD) \
  k_center_project<T, LD><<<nb, 256, 0, s>>>(g, (const V2<T> *)U, (const double2 *)G, Z, part, pairs, tiled)
  if (streaming(read, 0).loads) MCG_CP(true);
  else MCG_CP(false);
#undef MCG_CP
  k_min_final<<<1, 1024, 0, s>>>(part, nb, min_out);
  return hipGetLastError();
}

hipError_t launch_count_vortices(const Geom &g, const int8_t *Z, unsigned long long *counts,
                                 hipStream_t s) {
  if (g.L[0] % 4 == 0 && ((uintptr_t)Z & 3) == 0) {  // four sites per thread, in words
    k_count_vortices4<<<std::min((g.V / 4 + 255) / 256, 1024), 256, 0, s>>>(g, Z, counts);
    return hipGetLastError();
  }
  // a few blocks per CU, each site visited by one thread of a grid-stride loop
  const int blocks = std::min((g.V + 255) / 256, 2048);
  k_count_vortices<<<blocks, 256, 0, s>>>(g, Z, counts);
  return hipGetLastError();
}

template hipError_t launch_center_project<float>(const Geom &, const void *, const double *, int8_t *,
                                                 double *, double *, hipStream_t);
template hipError_t launch_center_project<double>(const Geom &, const void *, const double *, int8_t *,
                                                  double *, double *, hipStream_t);

}  // namespace mcg
