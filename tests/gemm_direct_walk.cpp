// Host walk of the loads of gemm_direct.hpp with the index arithmetic that the kernel itself uses.
#include <algorithm>

#include "gemm_direct_plan.hpp"

using namespace tc355;

// The first and last 40 rows of an operand of `rows` rows of K elements (size 4 or 8 bytes), all lanes and parts of every step
// (of the first and the last two where there are many): the number of 16-byte loads that leave the operand or that bring
// other elements than they stand for.
extern "C" int64_t walk_loads(int64_t rows, int K, int size) {
  const int parts = size == 8 ? 2 : 1, per = 16 / size;  // 64-byte pieces per 16 k; elements per part
  const int64_t bytes = rows * K * size;
  int64_t faults = 0;
  for (int64_t r = 0; r < rows; r = (r == 39 && rows > 80) ? rows - 40 : r + 1)
    for (int lp = 0; lp < 4; lp++) {
      const unsigned off = gd_offset((int)r, per * lp, K, size);
      const int steps = (K + 15) / 16;
      for (int s = 0; s < steps; s = (s == 1 && steps > 4) ? steps - 2 : s + 1)
        for (int z = 0; z < parts; z++) {
          const int k0 = 16 * s, k = k0 + (16 / parts) * z + per * lp, group = k / 4 * 4 - k0;
          const bool whole = k0 + 16 <= K;
          const int64_t at = (int64_t)k0 * size + off + 64 * z + (whole ? 0 : gd_end_shift(k0, group, K, size));
          const int64_t want = (r * K + k - (whole ? 0 : std::max(0, k0 + group + 4 - K))) * size;
          if (at != want || at < 0 || at + 16 > bytes) faults++;
        }
    }
  return faults;
}

extern "C" int reaches(int64_t rows, int K, int size) { return gd_reaches(rows, K, size); }
