// Host-side check of the tracers' cell index (cic_axis): floor(x / dx) mod n taken in
// whole numbers, for positions of every magnitude up to 2^62 cells; the index of any
// position at all (infinities and no number included) is a grid point.
#include <cstdint>
#include <cstdio>
#include <limits>

#include "mhd_cic.h"

// short calls gather from the planes, long ones interleave; no count overflows
constexpr int64_t cube(int64_t n) { return n * n * n; }
static_assert(!mhd::cic_interleaves(1000, 1, 3, cube(256), 8) && !mhd::cic_interleaves(1000, 1, 4, cube(512), 4), "");
static_assert(!mhd::cic_interleaves(1, 1, 3, cube(1024), 4) && mhd::cic_interleaves(1, 1, 3, cube(32), 8), "");
static_assert(mhd::cic_interleaves(1000003, 20, 3, cube(128), 8), "");
static_assert(mhd::cic_interleaves(int64_t(1) << 40, 2147483647, 4, cube(1024), 4), "");

int main() {
  const int sizes[] = {8, 12, 16, 24, 48, 96, 128, 192, 384, 768, 1024};
  long bad = 0;
  uint64_t z = 12345;
  for (int n : sizes) {
    for (int k = 0; k < 200000; ++k) {
      z = z * 6364136223846793005ull + 1442695040888963407ull;
      const double u = double(z >> 11) / 9007199254740992.0 * 2.0 - 1.0;
      double x = u * (mhd::kTwoPi / n) * ldexp(1.0, k % 63);
      if (k % 97 == 0) x = double((int64_t)(u * 1000.0)) * (mhd::kTwoPi / n);  // cell faces
      const mhd::CicAxis a = mhd::cic_far(n, x) ? mhd::cic_axis<true>(n, x) : mhd::cic_axis<false>(n, x);
      const double fl = floor(x / (mhd::kTwoPi / n));
      int64_t want = (int64_t)fl % n;
      if (want < 0) want += n;
      const bool ok = a.i0 == want && a.i1 == (want + 1) % n && a.w1 >= 0.0 && a.w1 <= 1.0 && a.w0 == 1.0 - a.w1;
      if (!ok && bad++ < 5) std::printf("n=%d x=%.17g: i0 %d i1 %d, want %d\n", n, x, a.i0, a.i1, (int)want);
    }
    const double inf = std::numeric_limits<double>::infinity(), nan = std::numeric_limits<double>::quiet_NaN();
    const double odd[] = {inf, -inf, nan, -nan, 1e300, -1e300, 1.7e308, -1.7e308, 1e30, -1e25, 0.0, -0.0, 5e-324, -5e-324};
    for (double x : odd) {
      const mhd::CicAxis a = mhd::cic_far(n, x) ? mhd::cic_axis<true>(n, x) : mhd::cic_axis<false>(n, x);
      if ((a.i0 < 0 || a.i0 >= n || a.i1 < 0 || a.i1 >= n) && bad++ < 5)
        std::printf("n=%d x=%g: i0 %d i1 %d\n", n, x, a.i0, a.i1);
    }
    // a particle lost on the way (no number) keeps to the near form
    const mhd::CicAxis b = mhd::cic_axis<false>(n, nan);
    if ((b.i0 < 0 || b.i0 >= n || b.i1 < 0 || b.i1 >= n) && bad++ < 5) std::printf("n=%d no number: i0 %d\n", n, b.i0);
  }
  std::printf("failing positions: %ld\n", bad);
  return bad ? 1 : 0;
}
