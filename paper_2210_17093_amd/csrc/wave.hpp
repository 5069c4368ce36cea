// Wave-level sums and the slots through which workgroups of one launch hand
// values to each other (the eigensolvers' kernels).
#pragma once
#include <hip/hip_runtime.h>

#include "poles.hpp"

namespace qsgw {

typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_add(double x) {
  // (lanes without a source add 0)
  const u32x2 b = __builtin_bit_cast(u32x2, x);
  u32x2 r;
  r[0] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b[0], CTRL, ROWS, 0xf, ROWS == 0xf);
  r[1] = (unsigned)__builtin_amdgcn_update_dpp(0, (int)b[1], CTRL, ROWS, 0xf, ROWS == 0xf);
  return x + __builtin_bit_cast(double, r);
}
__device__ __forceinline__ double read_lane(double x, int l) {
  const u32x2 b = __builtin_bit_cast(u32x2, x);
  u32x2 r;
  r[0] = (unsigned)__builtin_amdgcn_readlane((int)b[0], l);
  r[1] = (unsigned)__builtin_amdgcn_readlane((int)b[1], l);
  return __builtin_bit_cast(double, r);
}
// Sum over the 64 lanes (row shifts by 1, 2, 4, 8, then the row broadcasts), the same in every lane.
__device__ __forceinline__ double wave_total(double x) {
  x = dpp_add<0x111, 0xf>(x);
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  x = dpp_add<0x118, 0xf>(x);
  x = dpp_add<0x142, 0xa>(x);
  x = dpp_add<0x143, 0xc>(x);
  return read_lane(x, 63);
}
__device__ __forceinline__ double quad_total(double x) {
  x = dpp_add<0xB1, 0xf>(x);
  return dpp_add<0x4E, 0xf>(x);
}
// 1 / x and 1 / sqrt(x) to about one unit in the last place (two Newton steps).
__device__ __forceinline__ double fast_rcp(double x) {
  double y = __builtin_amdgcn_rcp(x);
  y = fma(fma(-x, y, 1.0), y, y);
  return fma(fma(-x, y, 1.0), y, y);
}
__device__ __forceinline__ double fast_rsqrt(double x) {
  double y = __builtin_amdgcn_rsq(x);
  y = fma(0.5 * y, fma(-x * y, y, 1.0), y);
  return fma(0.5 * y, fma(-x * y, y, 1.0), y);
}
// Householder reflector H = I - tau v v^T of a column (alpha, rest) with the rest's
// sum of squares sig: H (alpha, rest) = (beta, 0), v = (1, scale rest).  The norm
// r is corrected to its last bit, as beta goes into the reduced matrix:
//   beta = -sign(alpha) r, tau = (beta - alpha) / beta = 1 + |alpha| / r,
//   scale = 1 / (alpha - beta) = sign(alpha) / (|alpha| + r).
// sig up to kTinySquare counts as zero (H = I); a NaN passes through.
struct Reflector {
  double tau, beta, scale;
};
__device__ __forceinline__ Reflector reflector(double alpha, double sig) {
  Reflector h{0.0, alpha, 0.0};
  if (!(sig <= kTinySquare)) {
    const double x = fma(alpha, alpha, sig);
    const double ir = fast_rsqrt(x), nr = x * ir;
    const double r = fma(fma(-nr, nr, x), 0.5 * ir, nr);
    h.beta = -copysign(r, alpha);
    h.tau = fma(fabs(alpha), ir, 1.0);
    h.scale = copysign(fast_rcp(fabs(alpha) + r), alpha);
  }
  return h;
}
// Workgroup barrier for LDS traffic alone: global stores stay in flight (the
// row that one team member publishes would otherwise hold up its y by a
// store's round trip in every column).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// x and y each summed over half of the lanes: lanes 0..31 hold x's sums, 32..63 y's.
__device__ __forceinline__ double swap_add32(double x, double y) {
  const u32x2 a = __builtin_bit_cast(u32x2, x), b = __builtin_bit_cast(u32x2, y);
  const auto l = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
  const auto h = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
  return __builtin_bit_cast(double, u32x2{l[0], h[0]}) + __builtin_bit_cast(double, u32x2{l[1], h[1]});
}
// The same within each half: 16-lane rows 0 and 2 hold x's sums, 1 and 3 y's.
__device__ __forceinline__ double swap_add16(double x, double y) {
  const u32x2 a = __builtin_bit_cast(u32x2, x), b = __builtin_bit_cast(u32x2, y);
  const auto l = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto h = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return __builtin_bit_cast(double, u32x2{l[0], h[0]}) + __builtin_bit_cast(double, u32x2{l[1], h[1]});
}

// A slot holds kEmpty until its value is published; its reader polls it.  No
// flag and no fence: the value is its own arrival.
constexpr unsigned long long kEmpty = ~0ull;

__device__ __forceinline__ void publish(double* p, double x) {
  unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  if (b == kEmpty) b = 0x7ff8000000000000ull;
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), b, __ATOMIC_RELAXED,
                     __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long peek(const double* p) {
  return __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace qsgw
