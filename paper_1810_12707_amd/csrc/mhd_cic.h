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
#include <cstdint>

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

// Whether a call of nsteps steps on np particles, gathering nf fields of reals of `size`
// bytes, interleaves them first (four values to a point) or gathers from the planes as
// they are synthesised.  Interleaving is a launch and a pass over the grid; what it saves
// is per particle and step, more of it with four fields, and not less per step than 28000
// particles', whose latency a smaller call has too.  Microseconds a call, planes and
// interleaved: 256^3 FP64 push 3x10^5 x 1: 371 and 493, 10^6 x 1: 599 and 580, 10^3 x 20:
// 437 and 516; velocity 3x10^5: 512 and 624, 10^6: 833 and 706; 512^3 FP32 push 10^6 x 1:
// 1570 and 1985, 10^6 x 4: 2280 and 2192; 128^3 FP32 push 10^3 x 1: 44 and 46, 10^3 x 4:
// 58 and 50; 64^3 FP64 push 10^3 x 1: 30 and 31.
constexpr bool cic_interleaves(int64_t np, int64_t nsteps, int nf, int64_t n3, int size) {
  const double particles = np > 28000 ? double(np) : 28000.0;
  return particles * double(nsteps) * (nf == 4 ? 64.0 : 36.0) >= double(n3) * (size / 4) + (1 << 19);
}

}  // namespace mhd
