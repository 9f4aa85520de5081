// Local exchange and correlation potentials of one grid value (device code
// shared by the pointwise kernels and the potential's phi synthesis).
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>

namespace ces {

// Slater (LDA) exchange potential V_x = -(3 rho_+ / pi)^(1/3), rho_+ =
// max(rho, 0): negative densities from quadrature noise count as zero.
__device__ __forceinline__ double slater_vx(double rho) {
  return -cbrt((3.0 / M_PI) * (rho > 0.0 ? rho : 0.0));
}

// Perdew-Zunger (1981) fit of the Ceperley-Alder correlation energy per
// electron of the unpolarised gas (the LDA of Section 2.1), r_s =
// (3 / (4 pi rho))^(1/3):
//   r_s >= 1:  eps = gamma / (1 + beta1 sqrt(r_s) + beta2 r_s)
//   r_s < 1:   eps = A ln r_s + B + C r_s ln r_s + D r_s
// v = d(rho eps)/d rho = eps - (r_s / 3) d eps / d r_s; rho <= 0 gives 0.
__device__ __forceinline__ void pz81(double rho, double& eps, double& v) {
  eps = 0.0;
  v = 0.0;
  if (!(rho > 0.0)) return;
  const double rs = cbrt(3.0 / (4.0 * M_PI * rho));
  if (rs >= 1.0) {
    const double g = -0.1423, b1 = 1.0529, b2 = 0.3334;
    const double sq = sqrt(rs), den = 1.0 + b1 * sq + b2 * rs;
    eps = g / den;
    // v = eps (1 + 7/6 b1 sqrt(r_s) + 4/3 b2 r_s) / den
    v = eps * (1.0 + (7.0 / 6.0) * b1 * sq + (4.0 / 3.0) * b2 * rs) / den;
  } else {
    const double A = 0.0311, B = -0.048, C = 0.0020, D = -0.0116;
    const double ln = log(rs);
    eps = A * ln + B + C * rs * ln + D * rs;
    v = A * ln + (B - A / 3.0) + (2.0 / 3.0) * C * rs * ln + ((2.0 * D - C) / 3.0) * rs;
  }
}

}  // namespace ces
