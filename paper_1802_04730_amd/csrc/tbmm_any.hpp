// Transposed batched matmul of small matrices of any size (Section 7, "Transposed Batched Matrix Multiplication",
// listing tbmm): what tbmm_lds.hpp does, without its conditions on alignment and with room for larger matrices.
//
//     Z(b,n,m) = sum_k X(b,n,k) * Y(b,m,k)
//
// What bounds it: HBM at large batches, the launch and one chain load -> MFMAs -> store at small ones, the fp64 matrix core where the
// matrices approach 100 x 100.
// A workgroup owns a strip of rows of X_b and a strip of rows of Y_b -- all of both where they are small, several batch elements
// where they are smaller still -- and its wavefronts share the strips' 16 x 16 tiles out.  The strips are contiguous runs of
// memory.  They travel straight to LDS (no registers, no LDS writes), every wavefront requests its part, and one barrier later
// every wavefront reads what it needs.  Nothing is pipelined inside a workgroup: 24-122 registers and the LDS of one strip pair
// leave room for several workgroups per compute unit, whose loads, MFMAs and stores cover each other.
//   * 16-byte pieces from the strip's first element on (4-byte alignment is enough), its last 1 .. 3 elements one by one: nothing
//     beyond a strip is read.
//   * VEC (K a multiple of 4: rows start on pieces): an operand read is one piece, whose four elements feed four MFMA steps, and
//     piece p of a strip lies in slot p ^ (p / 16 % 16), so that 16 rows at any such stride fall into different banks.
//     Otherwise an operand read is one element per lane, and rows at odd or singly even strides spread by themselves.
//   * Results are laid out in LDS and leave as contiguous streams: 16-byte pieces of the whole block where the strip covers
//     all of M (first and last piece element by element where they are shared), else row by row.  Where there are few, or the
//     reduction is long, they leave from the registers instead: two barriers less (4.2 -> 3.6 us at (17,27,55,86)).
// Against one wavefront per strip pair with a private LDS region and the next strips on their way in registers (us):
// (B,N,M,K) = (4000,27,61,35) 21.8 -> 17.3 (4.4 TB/s), (5117,46,61,72) 87 -> 52, (904,88,89,77) 43.6 -> 34, (2097,16,28,83)
// 10.7 -> 8.0, (207,39,49,73) 8.1 -> 5.3, (14,9,68,41) 3.5 -> 3.1; over 268 random shapes 1.14 times as fast, 4 of them 6-10 %
// slower (4-8 us each: (107,44,44,95) 4.4 -> 4.9).  That one held two strips per wavefront in registers, so a SIMD had two or
// three wavefronts and little to cover a round trip with.  Taken back: 16 wavefronts per workgroup (within 2 %).
#pragma once
#include "tbmm_any_plan.hpp"
#include "tc355_device.hpp"

namespace tc355 {

struct TbmmAnyArgs {
  const float* X;  // [B][N][K]
  const float* Y;  // [B][M][K]
  float* Z;        // [B][N][M]
  int B, N, M, K;          // B * strips_n * strips_m < 2^31
  int strips_n, strips_m;  // strips of 16 TN gn rows of X, of 16 TM gm rows of Y
  int direct;              // results straight from the registers
  unsigned first;          // number of the launch's first workgroup
};
// workgroup: gm wavefronts in x, gn in y, nb batch elements in z (1 where there are several strips)

// where piece p of a strip lies: 16 pieces in another order per 256 bytes
template <bool VEC>
__device__ __forceinline__ int ta_slot(int p) { return VEC ? p ^ ((p >> 4) & 15) : p; }

// lane l's 16 (4) bytes to lds + 16 l (4 l); a uniform address
__device__ __forceinline__ void ta_load16(const char* g, unsigned lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(uintptr_t)g,
                                   (__attribute__((address_space(3))) void*)(uintptr_t)lds, 16, 0, 0);
}
__device__ __forceinline__ void ta_load4(const char* g, unsigned lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(uintptr_t)g,
                                   (__attribute__((address_space(3))) void*)(uintptr_t)lds, 4, 0, 0);
}

template <int TN, int TM, bool VEC>
__global__ __launch_bounds__(TA_MAX_WAVES * WAVE, TN * TM <= 2 ? 6 : TN * TM <= 5 ? 4 : 3) void tbmm_any_kernel(TbmmAnyArgs p) {
  extern __shared__ __attribute__((aligned(16))) char ta_lds[];
  float* ldsf = reinterpret_cast<float*>(ta_lds);
  const int lane = threadIdx.x & (WAVE - 1);
  const int gm = blockDim.x / WAVE, gn = blockDim.y, nb = blockDim.z, waves = gm * gn * nb;
  const int wm = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE), wn = __builtin_amdgcn_readfirstlane(threadIdx.y),
            e = __builtin_amdgcn_readfirstlane(threadIdx.z);
  const int wave = (e * gn + wn) * gm + wm;
  const int r16 = lane & 15, q = lane >> 4;
  const int N = p.N, M = p.M, K = p.K;

  // ---- the workgroup's strips
  int b0 = (int)(p.first + blockIdx.x), n0 = 0, m0 = 0, ne = 1;
  if (p.strips_n * p.strips_m == 1) {
    b0 *= nb;
    ne = min(nb, p.B - b0);
  } else {
    const unsigned rest = (unsigned)b0 / (unsigned)p.strips_m;
    m0 = (b0 - (int)rest * p.strips_m) * 16 * TM * gm;
    b0 = (int)(rest / (unsigned)p.strips_n);
    n0 = ((int)rest - b0 * p.strips_n) * 16 * TN * gn;
  }
  const int rows = min(16 * TN * gn, N - n0), cols = min(16 * TM * gm, M - m0);
  const int xlen = ne * rows * K, ylen = ne * cols * K;  // elements
  const int xslots = VEC ? ((xlen >> 2) + 15) & ~15 : (xlen + 3) >> 2;
  const int yslots = VEC ? ((ylen >> 2) + 15) & ~15 : ylen >> 2;
  {
    const char* x = reinterpret_cast<const char*>(p.X + ((int64_t)b0 * N + n0) * K);
    const char* y = reinterpret_cast<const char*>(p.Y + ((int64_t)b0 * M + m0) * K);
    const unsigned base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)ta_lds;
    auto copy = [&](const char* src, int slots, int pieces, unsigned at, int g) {  // 64 slots from 64 g on
      const int s = WAVE * g + lane, u = ta_slot<VEC>(s);
      if (s < slots && u < pieces) ta_load16(src + 16u * (unsigned)u, at + 1024u * (unsigned)g);
    };
    const int gx = ((VEC ? xslots : xlen >> 2) + WAVE - 1) / WAVE, gy = (yslots + WAVE - 1) / WAVE;
    for (int g = wave; g < gx; g += waves) copy(x, VEC ? xslots : xlen >> 2, xlen >> 2, base, g);
    for (int g = wave; g < gy; g += waves) copy(y, yslots, ylen >> 2, base + 16u * (unsigned)xslots, g);
    if (!VEC && wave == waves - 1) {  // what a strip holds beyond whole pieces
      if (lane < (xlen & 3)) ta_load4(x + 16u * (unsigned)(xlen >> 2) + 4 * lane, base + 16u * (unsigned)(xlen >> 2));
      if (lane < (ylen & 3)) ta_load4(y + 16u * (unsigned)(ylen >> 2) + 4 * lane, base + 16u * (unsigned)(xslots + (ylen >> 2)));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
  }

  // ---- contraction: MFMA rows = rows of X, columns = rows of Y (clamped into the strip; such results are not stored)
  d4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; i++)
#pragma unroll
    for (int j = 0; j < TM; j++) acc[i][j] = d4_zero();
  if (e < ne) {
    int arow[TN], brow[TM];  // first element of the lane's rows
#pragma unroll
    for (int i = 0; i < TN; i++) arow[i] = (e * rows + min(16 * (TN * wn + i) + r16, rows - 1)) * K;
#pragma unroll
    for (int j = 0; j < TM; j++) brow[j] = (e * cols + min(16 * (TM * wm + j) + r16, cols - 1)) * K;
    const int yword = 4 * xslots;
    auto mma = [&](const float (&a)[TN], const float (&b)[TM]) {
#pragma unroll
      for (int i = 0; i < TN; i++)
#pragma unroll
        for (int j = 0; j < TM; j++) acc[i][j] = mfma_f64((double)a[i], (double)b[j], acc[i][j]);
    };
    int k = 0;
    if constexpr (VEC) {
      for (; k + 16 <= K; k += 16) {  // lane (r16, q): k + 4 q .. + 3
        f4 a4[TN], b4[TM];
#pragma unroll
        for (int i = 0; i < TN; i++) a4[i] = *reinterpret_cast<const f4*>(ta_lds + 16 * ta_slot<true>(((arow[i] + k) >> 2) + q));
#pragma unroll
        for (int j = 0; j < TM; j++) b4[j] = *reinterpret_cast<const f4*>(ta_lds + 16 * (xslots + ta_slot<true>(((brow[j] + k) >> 2) + q)));
#pragma unroll
        for (int c = 0; c < 4; c++) {
          float a[TN], b[TM];
#pragma unroll
          for (int i = 0; i < TN; i++) a[i] = a4[i][c];
#pragma unroll
          for (int j = 0; j < TM; j++) b[j] = b4[j][c];
          mma(a, b);
        }
      }
    } else {
      for (; k + 16 <= K; k += 16) {
        float a[4][TN], b[4][TM];
#pragma unroll
        for (int c = 0; c < 4; c++) {
#pragma unroll
          for (int i = 0; i < TN; i++) a[c][i] = ldsf[arow[i] + q + k + 4 * c];
#pragma unroll
          for (int j = 0; j < TM; j++) b[c][j] = ldsf[yword + brow[j] + q + k + 4 * c];
        }
#pragma unroll
        for (int c = 0; c < 4; c++) mma(a[c], b[c]);
      }
    }
    for (; k < K; k += 4) {  // single steps; slots past K are zeroed in BOTH operands: what lies there may be an Inf
      float a[TN], b[TM];
      const bool in = VEC || k + q < K;
      const int at = in ? q : 0;  // (k itself is in)
#pragma unroll
      for (int i = 0; i < TN; i++) {
        const float v = VEC ? ldsf[4 * ta_slot<true>((arow[i] + k) >> 2) + q] : ldsf[arow[i] + k + at];
        a[i] = in ? v : 0.f;
      }
#pragma unroll
      for (int j = 0; j < TM; j++) {
        const float v = VEC ? ldsf[yword + 4 * ta_slot<true>((brow[j] + k) >> 2) + q] : ldsf[yword + brow[j] + k + at];
        b[j] = in ? v : 0.f;
      }
      mma(a, b);
    }
  }

  const int64_t z0 = ((int64_t)b0 * N + n0) * M + m0;
  if (p.direct) {
    if (e >= ne) return;
    float* z = p.Z + z0 + (int64_t)e * N * M;
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int row = 16 * (TN * wn + i) + d_row(q, v);
#pragma unroll
        for (int j = 0; j < TM; j++) {
          const int col = 16 * (TM * wm + j) + r16;
          if (row < rows && col < cols) z[(int64_t)row * M + col] = (float)acc[i][j][v];
        }
      }
    return;
  }

  // ---- results through LDS
  const bool flat = cols == M;  // one contiguous block (uniform)
  const int zoff = flat ? (int)(z0 & 3) : 0;
  __syncthreads();
  if (e < ne) {
#pragma unroll
    for (int i = 0; i < TN; i++)
#pragma unroll
      for (int v = 0; v < 4; v++) {
        const int row = 16 * (TN * wn + i) + d_row(q, v);
#pragma unroll
        for (int j = 0; j < TM; j++) {
          const int col = 16 * (TM * wm + j) + r16;
          if (row < rows && col < cols) ldsf[zoff + (e * rows + row) * cols + col] = (float)acc[i][j][v];
        }
      }
  }
  __syncthreads();
  if (flat) {
    const int end = zoff + ne * rows * M, zu = (end + 3) >> 2;
    float* zs = p.Z + (z0 - zoff);
    for (int u = WAVE * wave + lane; u < zu; u += WAVE * waves) {
      const f4 v = *reinterpret_cast<const f4*>(ta_lds + 16 * u);
      if (4 * u >= zoff && 4 * u + 4 <= end) {
        store_stream(reinterpret_cast<f4*>(zs + 4 * u), v);
      } else {
#pragma unroll
        for (int c = 0; c < 4; c++)
          if (4 * u + c >= zoff && 4 * u + c < end) zs[4 * u + c] = v[c];
      }
    }
  } else {
    float* zs = p.Z + z0;
    for (int r = wave; r < rows; r += waves)
      for (int c = lane; c < cols; c += WAVE) store_stream(zs + (int64_t)r * M + c, ldsf[r * cols + c]);
  }
}

}  // namespace tc355
