// What gemm_direct.hpp can address, and where a lane loads its 16-byte parts from.  Plain C++: the kernel compiles the second
// part for the GPU, and a test compiles all of it for the host and walks the rows of the largest operands.
#pragma once
#include <cstdint>

#include "tc355_host.hpp"

#ifdef __HIPCC__
#define TC355_HD __host__ __device__ __forceinline__
#else
#define TC355_HD inline
#endif

namespace tc355 {

// Can the kernel address an operand of `rows` rows of K elements?  Offsets are 32 bits, and a lane's part of a step of 16 k may
// begin beyond a short last row (gd_end_shift moves it back, but only in 64 bits: (rows, K) = (214748364, 5) in fp32 would be
// read in front of the operand).
inline bool gd_reaches(int64_t rows, int64_t K, int64_t size) { return (rows * K + 16) * size < ((int64_t)1 << 32); }

// Byte offset of element k of row `row`; k < 16.
TC355_HD unsigned gd_offset(int row, int k, int K, int size) { return ((unsigned)row * (unsigned)K + (unsigned)k) * (unsigned)size; }

// By how many bytes a part of the step at k0 that reaches beyond K is moved: `group` is the first k of its group of 4 within
// the step, and a group that would pass the row's end is moved back to end there.
TC355_HD int64_t gd_end_shift(int k0, int group, int K, int size) {
  const int beyond = K - 4 - (k0 + group);
  return (int64_t)(beyond < 0 ? beyond : 0) * size;
}

}  // namespace tc355
