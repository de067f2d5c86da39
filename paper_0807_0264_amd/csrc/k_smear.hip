// k_smear.hip -- one Jacobi step of stout (eps = 1) or over-improved stout
// smearing (Sec. II.B and Sec. III of arXiv:0807.0264):
//   C = rho (wp Cp + wr Cr),  wp = (5 - 2 eps)/3,  wr = -(1 - eps)/12
//   U'_mu(x) = exp(TA(C U_mu(x)^dag)) U_mu(x)
// One thread per link (k_smear) or one wave per direction of 64 sites
// (k_smear_stout); every new link is computed from the old field, so
// the input and output buffers are distinct.

#include "smear_kernels.hpp"

namespace mcg {

// Whether a stout step runs k_smear_stout (blocks of four waves that read 13 matrices per link) rather
// than k_smear (blocks of two, 19 matrices; one where a slice has no more than 64 half-sites).  Small
// launches are a few rounds of blocks over the 256 CUs: p of k_smear, e of k_smear_stout.  Where a CU then
// works through as many waves either way (p = 2e) the fewer reads win; with p < 2e the finer blocks leave
// it fewer waves.  From e = 4 on rounds matter little; in FP32 a single round waits for latency alone,
// which the barriers of k_smear_stout only lengthen.
// us per step, k_smear (k_smear_stout).  FP32: 4^4 8.6 (11.8), 8^4 8.8 (12.0), 12^2 10 6 (p = 2, e = 1) 11.5
// (13.2), 12^4 (3, 2) 14.4 (15.4), 12^3x16 (4, 2) 16.9 (15.4), 14^4 (5, 3) 19.1 (19.4), 16^3x12 (6, 3) 20.6
// (20.6), 16^4 (8, 4) 27.5 (23.9).  FP64: 4^4 9.2 (11.0), 8^4 9.4 (12.5), 12^2 10 6 15.6 (14.7), 12^4 16.6
// (18.7), 12^3x16 20.4 (19.6), 14^4 27.7 (28.6), 16^3x12 29.9 (29.4), 16^4 39.8 (38.2).
template <typename T> static bool stout_in_blocks(const Geom &g) {
  const int p = (8 * gather_tiles(g) + 255) / 256, e = (2 * gather_tiles<64>(g) + 255) / 256;
  const int waves = p * (g.Vh / g.L[3] > 64 ? 2 : 1);  // of a CU, where k_smear_stout has 4 e
  return e >= 4 || (waves >= 4 * e && (e >= 2 || sizeof(T) == 8));
}

template <typename T>
hipError_t launch_smear_step(const Geom &g, const void *U, void *out, double rho, double eps,
                             hipStream_t s, void *Cst) {
  const double wp = (5.0 - 2.0 * eps) / 3.0, wr = -(1.0 - eps) / 12.0;
  const int grid = 8 * gather_tiles(g);
  if (!out) return hipErrorInvalidValue;
  const V2<T> *u = (const V2<T> *)U;
  V2<T> *o = (V2<T> *)out, *cs = (V2<T> *)Cst;
  const T r = (T)rho, p = (T)wp, q = (T)wr;
  if (eps == 1.0 && stout_in_blocks<T>(g)) {
    const int blocks = 2 * gather_tiles<64>(g);
    if (cs) k_smear_stout<T, 1><<<blocks, 256, 0, s>>>(g, u, o, r, p, cs);
    else k_smear_stout<T><<<blocks, 256, 0, s>>>(g, u, o, r, p);
  } else if (eps == 1.0) {
    if (cs) k_smear<T, false, 1><<<grid, 128, 0, s>>>(g, u, o, r, p, q, cs);
    else k_smear<T, false><<<grid, 128, 0, s>>>(g, u, o, r, p, q);
  } else {
    if (cs) k_smear<T, true, 1><<<grid, 128, 0, s>>>(g, u, o, r, p, q, cs);
    else k_smear<T, true><<<grid, 128, 0, s>>>(g, u, o, r, p, q);
  }
  return hipGetLastError();
}

template hipError_t launch_smear_step<float>(const Geom &, const void *, void *, double, double, hipStream_t,
                                             void *);
template hipError_t launch_smear_step<double>(const Geom &, const void *, void *, double, double, hipStream_t,
                                              void *);

}  // namespace mcg
