// What gemm_direct.hpp can address, where a lane loads its 16-byte parts from, and which of its variants a product takes.  Plain
// C++: the kernel compiles the loads' part for the GPU, and tests compile all of it for the host, walk the rows of the largest
// operands and ask what their shapes take.
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

struct GemmDirectVariant {
  int rt, ct, nw;  // tiles of 16 x 16 per workgroup, wavefronts
  double t0, step, mfma, wg, load;
};
constexpr GemmDirectVariant GD_VARIANTS[5] = {{1, 1, 4, 2.1153, 0.1281, 0.0300, 0.2184, 0.0030}, {1, 1, 8, 2.1514, 0.1278, 0.0280, 0.3527, 0.0037},
                                              {1, 1, 16, 2.7616, 0.1079, 0.0312, 0.0000, 0.0037}, {1, 2, 8, 2.0669, 0.1774, 0.0258, 0.5765, 0.0043},
                                              {2, 2, 4, 2.2926, 0.2324, 0.0225, 0.7782, 0.0061}};

// Which tiles and how many wavefronts: the least of five estimates in us, each
//   t0 + step * (steps of 16 k of one wavefront) + (workgroups of the fullest compute unit) * (mfma * steps * tiles + wg)
//      + load * (1 KiB pieces per compute unit),
// with constants fitted to every variant's time at 650 sizes (errors of 4-6 %): the variant taken is 0.4 % from the best one
// on average, 11 % at worst ((128,4381,3140) 81.6, 73.5 with 1 x 2 tiles).  16 wavefronts only where no compute unit has two
// workgroups.
inline int choose_gemm_direct(int64_t N, int64_t M, int64_t K, int size, int cus) {  // size: bytes of an element of A
  int best = 0;
  double least = 0.0;
  for (int v = 0; v < 5; v++) {
    const GemmDirectVariant& x = GD_VARIANTS[v];
    const int64_t jobs = ceil_div(N, 16 * x.rt) * ceil_div(M, 16 * x.ct), steps = ceil_div(K, 16);
    if (x.nw == 16 && jobs > cus) continue;
    const double pieces = x.rt * (size == 8 ? 2 : 1) + x.ct;
    const double us = x.t0 + x.step * ceil_div(steps, x.nw) + ceil_div(jobs, cus) * (x.mfma * steps * x.rt * x.ct + x.wg) +
                      x.load * pieces * steps * ((double)jobs / cus);
    if (v == 0 || us < least) {
      best = v;
      least = us;
    }
  }
  return best;
}

}  // namespace tc355
