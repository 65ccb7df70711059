// Refinement of a reciprocal square root estimate (host and device).
#pragma once

#include "host_device.hpp"

namespace fep3m {

// 1 / sqrt(x) from an estimate y of relative error d by the third-order step
// y (1 + e / 2 + 3 e^2 / 8), e = 1 - x y^2: it leaves 2.5 d^3, nothing against
// the rounding for an estimate of 24 bits.  The rounding is at most 1.7e-16:
// half a unit in the last place of the result and half of x y's.  Where the
// step is no number (x = 0 or infinity) the estimate is the value.
FEP3M_HOST_DEVICE inline double rsqrt_step3(double x, double y) {
  const double e = __builtin_fma(-x * y, y, 1.0);
  const double r = __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
  return e == e ? r : y;
}

}  // namespace fep3m
