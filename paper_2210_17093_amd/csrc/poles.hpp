// Range of the eigensolvers' matrices and places of the poles of a divide and
// conquer merge (host and device code).
#pragma once
#include <cmath>

#if defined(__HIP__)
#define QSGW_HD __host__ __device__ __forceinline__
#else
#define QSGW_HD inline
#endif

namespace qsgw {

// |x|, infinity where x is not finite (a maximum of these shows it, which the
// maximum of two numbers does not for a NaN).
QSGW_HD double finite_magnitude(double x) {
  const double a = fabs(x);
  return a < HUGE_VAL ? a : HUGE_VAL;
}

// The reductions square and sum entries.  A matrix whose largest entry m lies
// outside [2^-400, 2^400] is multiplied by this power of two first, which brings m
// to [1/2, 1) and is exact but for entries that vanish beside m.
QSGW_HD int range_exponent(double m) {
  if (!(m > 0.0) || m >= HUGE_VAL || (m >= 0x1p-400 && m <= 0x1p400)) return 0;
  int ex = 0;
  (void)frexp(m, &ex);
  return -ex;
}
// Sums of squares up to this one count as zero: above it they keep all their
// bits, and the column that it belongs to is below 2^-80 of the largest entry.
constexpr double kTinySquare = 0x1p-960;
// The same for the entries of a tridiagonal matrix with a largest entry of about 1.
constexpr double kTinyEntry = 0x1p-480;

// Number of entries of the ascending v[0..len) below x, or not above it.
QSGW_HD int dc_count(const double* v, int len, double x, bool or_equal) {
  int lo = 0, hi = len;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    const bool below = or_equal ? v[mid] <= x : v[mid] < x;
    if (below) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// Place of pole t among the n poles d, ascending in [0, n1) and in [n1, n),
// when both are sorted together.  All places are different, and so each is taken
// once, as long as every pole is finite and each half is ascending; a NaN takes
// the place of another pole.
QSGW_HD int merged_place(const double* d, int n1, int n, int t) {
  return t < n1 ? t + dc_count(d + n1, n - n1, d[t], false) : t - n1 + dc_count(d, n1, d[t], true);
}

}  // namespace qsgw
