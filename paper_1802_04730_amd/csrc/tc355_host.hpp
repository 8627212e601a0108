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

}  // namespace tc355
