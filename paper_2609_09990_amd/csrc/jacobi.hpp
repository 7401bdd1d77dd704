// Rotation angle of the Jacobi subspace eigensolver.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace dmrg {

// c, s of the rotation that annihilates apq of [[app, apq], [apq, aqq]], |angle| <=
// pi / 4.  Est gives estimates of 1 / sqrt(x) and 1 / x good to some 2^-23 (the
// hardware's); two Newton steps each (error 2^-23 -> 2^-46 -> rounding) replace the
// exact roots and divisions, a chain of five that took most of a round: the tangent is
// good to a few units in the last place, and c = 1 / sqrt(1 + t^2), s = t c, so the
// rotation is orthogonal to rounding.
template <class Est>
__host__ __device__ inline void jacobi_rotation(double app, double aqq, double apq, double& c, double& s) {
  double x = aqq - app, y = 2.0 * apq;
  const double m = fmax(fabs(x), fabs(y));
  const double sc = m < 0x1p-460 ? 0x1p500 : (m > 0x1p460 ? 0x1p-600 : 1.0);  // keeps h in range
  x *= sc;
  y *= sc;
  const double h = fma(x, x, y * y);
  const double g = Est::rsq(h), hg = 0.5 * g;
  double r = h * g;
  r = fma(hg, fma(-r, r, h), r);
  r = fma(hg, fma(-r, r, h), r);
  const double den = fabs(x) + r;
  double inv = Est::rcp(den);
  inv = fma(inv, fma(-den, inv, 1.0), inv);
  inv = fma(inv, fma(-den, inv, 1.0), inv);
  const double t = (x >= 0.0 ? y : -y) * inv, w = fma(t, t, 1.0);
  double cc = Est::rsq(w);
  cc *= fma(-0.5 * w * cc, cc, 1.5);
  cc *= fma(-0.5 * w * cc, cc, 1.5);
  cc = fma(0.5 * cc, fma(-w * cc, cc, 1.0), cc);
  c = cc;
  s = t * cc;
}

}  // namespace dmrg
