// Kronecker-factored layer for any extents whose operands fit LDS:
//   T(b,i,l) = sum_k W1(i,k) X(b,k,l)     then     Y(b,i,j) = sum_l T(b,i,l) W2(j,l).
//
// What bounds it: the fp64 matrix core at large batches, the chain launch -> operands -> MFMAs -> store at small ones.
// The wave-level kernel (kron_wave.hpp) gathers every operand from global memory again for every MFMA, with a select
// and a conversion each: it never had the matrix core busy.  Here a workgroup of 8 wavefronts stages the factors once
// and `nb` batch elements at a time, widened to fp64 (as fp32, widened at the read, where fp64 would not fit), and a
// wavefront owns 16 rows i of one of them.  As in kron_lds.hpp the first contraction is computed transposed, so that
// its result registers are the A operands of the second one: T never moves and is never rounded.
//   * Either factor may go first.  SECOND computes T(b,k,j) = sum_l X(b,k,l) W2(j,l) and Y(b,i,j) = sum_k W1(i,k) T(b,k,j): the
//     same loops with (I, W1, K) and (J, W2, L) exchanged (the host passes them so, and all names below follow), where the
//     streamed tiles are rows of X as they lie in memory, T's result registers are B operands, and the partial group's k slots
//     serve all groups.  The host takes the order whose estimate is 10 % lower; multiply-adds are I L (K + J) against K J (L + I).
//     At 400 random layers: 1.106 times faster on average, 4 of them slower by 3-7 % (5-7 us each); (1647,77,68,13,88)
//     61.5 -> 25.6 us, (454,89,96,10,100) 34.3 -> 12.6, (1828,89,26,31,87) 45.3 -> 21.6.
//   * Two tiles of 16 l advance together, so a W1 operand feeds two MFMAs.
//   * k slot q of step e of a group is k = 4q + e: the four k slots of an X read are then 4 rows apart, and a row
//     stride of 4 (mod 8) elements spreads them over all banks; the last, partial group takes k = 4s + q.
//   * A row of fewer than 8 tiles in all (few rows i, few batch elements) is split over its l tiles (`lsp` wavefronts
//     per tile, combined through LDS in a fixed order), so that a single batch element keeps 8 wavefronts busy.
// Measured, wave-level kernel -> this one: (B,I,K,J,L) = (200,48,50,75,36) 22.7 -> 7.8 us (252 MFMAs per batch element, one
// per compute unit: 1.6 us of launch, 2 of staging, 84 MFMAs in the longest wavefront), (40,79,89,29,74) 52.7 -> 7.2,
// (2000,18,98,40,48) 63 -> 26, (500,96,100,100,100) 243 -> 49 us (matrix pipe busy 56 % of it),
// (8,8,8,8,8) 4.0 -> 3.3.
// Registers decide the occupancy (two workgroups per compute unit up to four column tiles): everything that is uniform
// over a wavefront is kept scalar, and few loads are in flight while accumulators live.  A read-ahead by a whole group
// of 16 k was slower for that reason (9.9 -> 13 us at the first shape, with spills); so were five column tiles at two workgroups.
#pragma once
#include "kron_tile_plan.hpp"
#include "tc355_device.hpp"

namespace tc355 {

static_assert(KT_WAVE == WAVE, "lanes of a wavefront");
constexpr int KT_BATCH = 4;  // first loads of each operand, per thread
constexpr int KT_REST = 12;  // loads in flight per thread behind them

struct KronTileArgs {
  const float* W1;  // [I][K]
  const float* W2;  // [J][L]
  const float* X;   // [B][K][L]
  float* Y;         // [B][I][J]
  int B, I, K, J, L;
  int nb, lsp;       // batch elements staged together; wavefronts per 16-row tile
  int groups;        // ceil(B / nb)
  int itb, jblocks;  // 16-row tiles per block of rows; blocks of 16*TJ columns
  int k4;            // K rounded up to 4
  int ls, ls1, ls2;  // LDS row strides of X, W1, W2 in elements
  int xs;            // LDS elements of the X region (also large enough for the partial sums)
  unsigned l_magic, k_magic;  // ceil(2^32 / L), ceil(2^32 / K)
};

// `total` contiguous floats, rows of `len`, on their way to LDS rows of `stride` elements; `gap` elements more after
// every K rows (the zero rows between batch elements).
template <typename TS, bool GAPS>
struct KronCopy {
  const float* src;
  TS* dst;
  int total, len, stride, gap, tid;
  unsigned magic, k_magic;

  template <int U>
  __device__ __forceinline__ void load(float (&v)[U], int e0) const {
#pragma unroll
    for (int u = 0; u < U; u++)
      v[u] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(src) + (unsigned)min(e0 + u * KT_THREADS + tid, total - 1) * 4u);
  }
  template <int U>
  __device__ __forceinline__ void store(const float (&v)[U], int e0) const {
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int e = min(e0 + u * KT_THREADS + tid, total - 1);  // (beyond the end: the last element again)
      const int row = (int)__umulhi((unsigned)e, magic);
      int at = row * stride + (e - row * len);
      if (GAPS) at += (int)__umulhi((unsigned)row, k_magic) * gap;
      dst[at] = (TS)v[u];
    }
  }
  // everything behind the first KT_THREADS * KT_BATCH elements
  __device__ __forceinline__ void rest() const {
    int e0 = KT_THREADS * KT_BATCH;
#pragma unroll 1
    for (; e0 + KT_THREADS * 4 < total; e0 += KT_THREADS * KT_REST) {
      float v[KT_REST];
      load(v, e0);
      store(v, e0);
    }
    if (e0 < total) {
      float v[4];
      load(v, e0);
      store(v, e0);
    }
  }
};

template <typename TS>
struct KronTileJob {
  const TS* x;   // Xs of this batch element: + r16, row 4q of a group (SECOND: + q)
  const TS* xt;  // the same, row (column) q of the partial group
  const TS* w1;  // W1s row of this lane + 4q (SECOND: + q)
  const TS* w1t; // W1s row of this lane + first k of the partial group + q
};

// One or two tiles of 16 l from l0 on: T, then its share of all TJ column tiles.  FULL: every l of the tiles is below L.
template <typename TS, int TJ, bool SECOND, int NL, bool FULL>
__device__ __forceinline__ void kron_l_tiles(const KronTileJob<TS>& jb, const TS* w2, int cs, int l0, int L, int K, int ls, int r16, int q, d4 (&acc)[TJ]) {
  d4 T[NL];
  int xo[NL];  // first element of tile n; rows beyond the last repeat it (their T is replaced by zeros)
#pragma unroll
  for (int n = 0; n < NL; n++) {
    T[n] = d4_zero();
    xo[n] = SECOND ? (FULL ? l0 + 16 * n + r16 : min(l0 + 16 * n + r16, L - 1)) * ls : 16 * n;
  }
  const int k16 = K >> 4;
  const TS* xp = SECOND ? jb.x : jb.x + l0;
  const TS* wp = jb.w1;
#pragma unroll 1
  for (int g = 0; g < k16; g++) {
    TS a[NL][4], w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      w[e] = wp[SECOND ? 4 * e : e];
#pragma unroll
      for (int n = 0; n < NL; n++) a[n][e] = xp[xo[n] + e * (SECOND ? 4 : ls)];
    }
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int n = 0; n < NL; n++) T[n] = mfma_f64((double)a[n][e], (double)w[e], T[n]);
    xp += SECOND ? 16 : 16 * ls;
    wp += 16;
  }
  {
    const TS* xt = SECOND ? jb.xt : jb.xt + l0;
    const TS* wt = jb.w1t;
#pragma unroll 1
    for (int k = k16 * 16; k < K; k += 4) {
      const double w = (double)*wt;
#pragma unroll
      for (int n = 0; n < NL; n++) T[n] = mfma_f64((double)xt[xo[n]], w, T[n]);
      xt += SECOND ? 4 : 4 * ls;
      wt += 4;
    }
  }
  // the W2 operands of one step are read while the step before it is contracted (all steps' reads at once, as the compiler
  // would have it, cost the registers of a second workgroup per compute unit)
  const TS* wl = w2 + l0;
  TS w[TJ];
#pragma unroll
  for (int c = 0; c < TJ; c++) w[c] = wl[c * cs];
#pragma unroll
  for (int n = 0; n < NL; n++)
#pragma unroll
    for (int v = 0; v < 4; v++) {
      if (FULL || l0 + 16 * n + 4 * v < L) {
        const int s = 4 * n + v;
        double t = T[n][v];
        if (!FULL) t = l0 + 4 * s + q < L ? t : 0.0;  // an Inf in W1 makes the rows of T beyond L NaN
        TS wn[TJ];
        if (s < 4 * NL - 1) {
#pragma unroll
          for (int c = 0; c < TJ; c++) wn[c] = wl[c * cs + 4 * s + 4];
        }
#pragma unroll
        for (int c = 0; c < TJ; c++) acc[c] = SECOND ? mfma_f64((double)w[c], t, acc[c]) : mfma_f64(t, (double)w[c], acc[c]);
        __builtin_amdgcn_sched_barrier(0);
        if (s < 4 * NL - 1) {
#pragma unroll
          for (int c = 0; c < TJ; c++) w[c] = wn[c];
        }
      }
    }
}

template <typename TS, int TJ, bool SECOND>
__global__ __launch_bounds__(KT_THREADS, TJ <= 4 ? 4 : 2) void kron_tile_kernel(KronTileArgs p) {
  extern __shared__ __attribute__((aligned(16))) char kron_smem[];
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / WAVE);  // (scalar: so is all that is derived from it)
  const int r16 = lane & 15, q = lane >> 4;
  const int I = p.I, K = p.K, J = p.J, L = p.L, ls = p.ls;
  const int i0 = (int)(blockIdx.y / p.jblocks) * p.itb * 16, j0 = (int)(blockIdx.y % p.jblocks) * 16 * TJ;
  const int irows = min(p.itb * 16, I - i0), jrows = min(16 * TJ, J - j0), itiles = (irows + 15) >> 4;
  TS* Xs = reinterpret_cast<TS*>(kron_smem);
  TS* W2s = Xs + p.xs;
  TS* W1s = W2s + 16 * TJ * p.ls2;
  const int l4 = (L + 3) & ~3;

  // zeros that the partial last steps read: k in [K, k4) of X and W1, l in [L, l4) of W2
  const int zrows = p.k4 - K;
  auto zero_rows = [&] {
    if constexpr (SECOND) {  // the ends of all rows
      for (int r = tid; r < L * p.nb; r += KT_THREADS)
        for (int k = K; k < p.k4; k++) Xs[r * ls + k] = (TS)0;
    } else {
      for (int e = tid; e < zrows * ls * p.nb; e += KT_THREADS) {
        const int b = e / (zrows * ls);
        Xs[(b * p.k4 + K) * ls + e - b * zrows * ls] = (TS)0;
      }
    }
  };
  zero_rows();
  if (tid < irows)
    for (int k = K; k < p.k4; k++) W1s[tid * p.ls1 + k] = (TS)0;
  if (tid < jrows)
    for (int l = L; l < l4; l++) W2s[tid * p.ls2 + l] = (TS)0;
  // the first loads of all three operands go out together: one round trip to memory before the first MFMA
  auto x_copy = [&](int g) {
    return KronCopy<TS, !SECOND>{p.X + (int64_t)g * p.nb * K * L, Xs, min(p.nb, p.B - g * p.nb) * K * L, SECOND ? K : L, ls, zrows * ls, tid,
                                 SECOND ? p.k_magic : p.l_magic, p.k_magic};
  };
  float vx[KT_BATCH];
  {
    const KronCopy<TS, false> c1{p.W1 + (int64_t)i0 * K, W1s, irows * K, K, p.ls1, 0, tid, p.k_magic, 0};
    const KronCopy<TS, false> c2{p.W2 + (int64_t)j0 * L, W2s, jrows * L, L, p.ls2, 0, tid, p.l_magic, 0};
    float v1[KT_BATCH], v2[KT_BATCH];
    x_copy(blockIdx.x).load(vx, 0);
    c1.load(v1, 0);
    c2.load(v2, 0);
    c1.store(v1, 0);
    c2.store(v2, 0);
    c1.rest();
    c2.rest();
  }

  const TS* w2 = W2s + r16 * p.ls2 + q;  // (rows of the last tile beyond J hold anything: they feed columns that are not stored)
  const int ltiles = (L + 15) >> 4, per_part = (ltiles + p.lsp - 1) / p.lsp;

  for (int g = blockIdx.x; g < p.groups; g += gridDim.x) {
    const int b0 = g * p.nb, nb = min(p.nb, p.B - b0);
    {
      const KronCopy<TS, !SECOND> cx = x_copy(g);
      cx.store(vx, 0);
      cx.rest();
    }
    __syncthreads();
    if (g + (int)gridDim.x < p.groups) x_copy(g + gridDim.x).load(vx, 0);  // travels while this group is contracted
    const int njobs = nb * itiles * p.lsp;
    for (int job0 = 0; job0 < njobs; job0 += KT_WAVES) {  // one turn where lsp > 1
      const int job = job0 + wave;
      const int part = job % p.lsp, tile = job / p.lsp, bi = tile / itiles, it = tile - bi * itiles;
      const bool mine = job < njobs;
      d4 acc[TJ];
#pragma unroll
      for (int c = 0; c < TJ; c++) acc[c] = d4_zero();
      if (mine) {
        KronTileJob<TS> jb;
        const TS* xb = SECOND ? Xs + bi * L * ls : Xs + bi * p.k4 * ls + r16;
        const TS* wr = W1s + min(16 * it + r16, irows - 1) * p.ls1;
        jb.x = xb + (SECOND ? q : 4 * q * ls);
        jb.xt = xb + ((K & ~15) + q) * (SECOND ? 1 : ls);
        jb.w1 = wr + (SECOND ? q : 4 * q);
        jb.w1t = wr + (K & ~15) + q;
        const int lend = min(L, 16 * per_part * (part + 1));
        int l0 = 16 * per_part * part;
        for (; l0 + 32 <= lend; l0 += 32) kron_l_tiles<TS, TJ, SECOND, 2, true>(jb, w2, 16 * p.ls2, l0, L, K, ls, r16, q, acc);
        if (lend - l0 > 16) kron_l_tiles<TS, TJ, SECOND, 2, false>(jb, w2, 16 * p.ls2, l0, L, K, ls, r16, q, acc);
        else if (lend > l0) kron_l_tiles<TS, TJ, SECOND, 1, false>(jb, w2, 16 * p.ls2, l0, L, K, ls, r16, q, acc);
      }
      if (p.lsp > 1) {
        __syncthreads();  // X is no longer read: the region takes the partial sums
        double* sums = reinterpret_cast<double*>(kron_smem) + (size_t)tile * (p.lsp - 1) * TJ * 4 * WAVE + lane;
        if (mine && part > 0) {
#pragma unroll
          for (int c = 0; c < TJ; c++)
#pragma unroll
            for (int v = 0; v < 4; v++) sums[(((part - 1) * TJ + c) * 4 + v) * WAVE] = acc[c][v];
        }
        __syncthreads();
        if (mine && part == 0) {
#pragma unroll 1
          for (int o = 0; o < p.lsp - 1; o++)
#pragma unroll
            for (int c = 0; c < TJ; c++)
#pragma unroll
              for (int v = 0; v < 4; v++) {
                acc[c][v] += sums[((o * TJ + c) * 4 + v) * WAVE];
                if (v == 3 && c % 2) __builtin_amdgcn_sched_barrier(0);
              }
        }
      }
      if (mine && part == 0) {
        float* Y = p.Y + (int64_t)(b0 + bi) * I * J;
        if constexpr (SECOND) {  // (the extents are exchanged: Y's rows are J and its columns I here)
          // a scalar row pointer plus the lane's own offset: pointers per lane would cost the registers of the second
          // workgroup per compute unit
          Y += (int64_t)j0 * I + i0 + 16 * it;
          const unsigned own = (unsigned)(q * I + r16);
          const bool col = 16 * it + r16 < irows;
#pragma unroll
          for (int c = 0; c < TJ; c++) {
#pragma unroll
            for (int v = 0; v < 4; v++) {
              if (col && 16 * c + d_row(q, v) < jrows) Y[own] = (float)acc[c][v];
              Y += 4 * (int64_t)I;
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        } else {
          Y += (int64_t)(i0 + 16 * it) * J + j0 + r16;
#pragma unroll
          for (int v = 0; v < 4; v++) {
            const int i = d_row(q, v);
            if (16 * it + i < irows) {
#pragma unroll
              for (int c = 0; c < TJ; c++)
                if (16 * c + r16 < jrows) Y[(int64_t)i * J + 16 * c] = (float)acc[c][v];
            }
          }
        }
      }
    }
    __syncthreads();  // before the region is staged again
    if (p.lsp > 1) zero_rows();  // the partial sums have overwritten them
  }
}

}  // namespace tc355
