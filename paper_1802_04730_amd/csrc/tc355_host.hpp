// Small helpers of the host side (no HIP in here: tests compile what uses them with a plain C++ compiler).
#pragma once
#include <cstdint>
#include <initializer_list>

namespace tc355 {

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// True if the product of the (positive) extents reaches `limit`; never overflows: it stops at the first factor
// that takes the running product there.
inline bool prod_reaches(std::initializer_list<int64_t> factors, int64_t limit) {
  int64_t p = 1;
  for (int64_t f : factors) {
    if (f >= limit || p > limit / f) return true;  // p * f > limit
    p *= f;
    if (p >= limit) return true;
  }
  return false;
}

// HIP refuses a launch of 2^32 threads or more in one dimension.  Kernels that may need more take the number of the launch's first
// workgroup and run in several launches: workgroups of `threads` threads for the next one, of `left` that are left.  (A
// multiple of 8 unless it is the last: workgroups equal modulo 8 share an XCD.)
inline int64_t next_launch(int64_t left, int threads) {
  const int64_t most = ((int64_t)1 << 31) / threads / 8 * 8;
  return left < most ? left : most;
}

}  // namespace tc355
