// Cloud-in-cell weights of the tracers, along one axis.
//
// A particle at x lies in the cell whose lower corner is grid point
// i = floor(x / dx) (periodic, dx = 2 pi / n), at fraction f = x/dx - i of the
// cell; corner i weighs 1 - f and corner i + 1 weighs f per axis, and a corner's
// weight is the product over the axes: the volume of the opposite sub-box over the
// cell volume (trilinear interpolation).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>

namespace mhd {

constexpr double kTwoPi = 6.28318530717958647692528676655900577;

struct CicAxis {
  int i0, i1;
  double w0, w1;
};

// Positions below this many cells (every one inside the box is) are reduced in one
// round; FAR takes any.
constexpr double kCicNear = 4503599627370496.0;  // 2^52
__host__ __device__ __forceinline__ bool cic_far(int n, double x) { return !(fabs(x) * n < kCicNear); }

template <bool FAR> __host__ __device__ __forceinline__ CicAxis cic_axis(int n, double x) {
  const double s = x / (kTwoPi / n);
  const double fl = floor(s);
  // fl mod n, without a division.  The quotient is off by its own rounding: by one at
  // most up to 2^52, by |fl| / n 2^-52 beyond, which leaves a multiple of n (exactly: it
  // fits 53 bits) for a second round.
  const double inv = 1.0 / n;
  double r = fma(-floor(fl * inv), double(n), fl);
  if (FAR) r = fma(-floor(r * inv), double(n), r);
  r = r < 0.0 ? r + n : (r >= n ? r - n : r);
  // a position that is no number, or beyond 2^63 cells, still gives a grid point
  int i;
  if (FAR) {
    i = r >= 0.0 && r < n ? (int)r : 0;
  } else {
    i = r >= 0.0 ? (int)r : 0;  // r < n but for rounding: 32^3 FP64 5% faster than the test above
    i = i >= n ? n - 1 : i;
  }
  CicAxis a;
  a.i0 = i;
  a.i1 = i + 1 < n ? i + 1 : 0;
  a.w1 = s - fl;
  a.w0 = 1.0 - a.w1;
  return a;
}

}  // namespace mhd
