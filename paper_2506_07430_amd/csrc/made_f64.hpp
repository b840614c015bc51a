// FP64 epilogue shared by the fused kernels: one orbital's conditional of a row at its cursor,
// and one entry's term of the local energy.
#pragma once
#include "elocal_internal.hpp"
#include "made_bf16.hpp"

namespace elocal {


// H exp(dA / 2 + i 2 pi (sigmoid(zp) - sig_x)); dA in natural-log units.
static __device__ __attribute__((noinline)) double2 ratio_term64(double hv, double zp, double sig_x, double dA) {
  const double dphi = 2.0 * M_PI * (1.0 / (1.0 + exp(-zp)) - sig_x);
  double sn, cs;
  sincos(dphi, &sn, &cs);
  const double mag = hv * exp(0.5 * dA);
  return make_double2(mag * cs, mag * sn);
}

// log p_p(s_p) of the row at the cursor's orbital (the softmax over the reachable
// occupations, shifted by their largest logit), then four orbitals on. The largest term of
// the sum is 1, so three exponentials are left, without a branch per occupation.
template <int NW>
__device__ __forceinline__ double cond_step64(RowCursor<NW>& rc, int ta, int tb, int na, int nb, const f64x4& z) {
  const uint32_t b8 = (uint32_t)rc.bits[0] & 0xFFu;
  const bool a_must = rc.cu < ta, a_may = rc.cu < na, b_must = rc.cd < tb, b_may = rc.cd < nb;
  const double y0 = !a_must && !b_must ? z[0] : -INFINITY, y1 = a_may && !b_must ? z[1] : -INFINITY;
  const double y2 = !a_must && b_may ? z[2] : -INFINITY, y3 = a_may && b_may ? z[3] : -INFINITY;
  const double h0 = fmax(y0, y1), l0 = fmin(y0, y1), h1 = fmax(y2, y3), l1 = fmin(y2, y3);
  const double m = fmax(h0, h1);
  const double sum = 1.0 + exp(fmin(h0, h1) - m) + (exp(l0 - m) + exp(l1 - m));
  const double z01 = (b8 & 1u) ? z[1] : z[0], z23 = (b8 & 1u) ? z[3] : z[2];
  const double zs = (b8 & 2u) ? z23 : z01;
  cursor_advance4<NW>(rc, b8);
  return zs - m - log(sum);
}

}  // namespace elocal
