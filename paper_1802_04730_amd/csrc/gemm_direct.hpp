// One matrix pair  C[n][m] = sum_k A[n][k] * Bm[m][k]  (B = 1 of tc_tbmm, or one fcrelu layer: Section 3, listing fcrelu)
// with the reduction split over the wavefronts of a workgroup, for any extents with K >= 4.
//
// What bounds it: loads.  A 16-byte load whose neighbouring lanes hold neighbouring rows -- the MFMA operand layout -- takes a
// compute unit's address path 41-65 clocks; the same 16 rows x 64 bytes with four lanes per row take 19-27 (rows of 1716,
// 2048, 4000 and 4096 bytes), with or without LDS as the target.  So operands go straight to LDS (global_load_lds, 16 bytes
// per lane: no registers, no LDS writes by the wavefront, a swizzle in the choice of the lane's piece instead of padding) and
// are read back in operand layout.  Every wavefront has a ring of its own and waits for its own loads only; the wavefronts
// meet once, to add their partial tiles in a fixed order, starting from the bias.  The kernel needs 34-78 registers, so many
// workgroups share a compute unit and cover each other's latencies: two steps of 16 k in flight are enough.
//
// A piece = 1 KiB: 16 rows x 64 bytes.  Lane l loads row l / 4, 16-byte part (l % 4) ^ (l / 16), and the piece lies in LDS in
// lane order; reading part x of row r at 64 r + 16 (x ^ (r / 4)) touches 16 different bank groups for 16 rows.  A step of fp32
// is one piece per 16 rows; of fp64 two.  Rows past the extents repeat the last one, columns and rows past them are not
// stored.  In the last step groups of 4 k that would pass the end are moved back to end at K (4-byte alignment is enough) and
// what they share with the group before counts as zero, in both operands.
//
// Against the kernels it took over from (16 x 16 tiles staged through registers; 64 x 64 blocks; us): (N,M,K) = (64,64,64)
// 3.2 -> 2.5, (973,699,108) 9.7 -> 7.8, (128,2864,488) 15.9 -> 10.9, (128,3240,1220) 31.2 -> 25.6, (1000,1000,1000) 45.8 -> 38.4;
// on fp64 activations (300,600,1000) 14.2 -> 12.2, (128,1024,1024) 9.8 -> 8.4, (973,285,132) 9.1 -> 5.6.  Over 650 sizes
// 1.26 times as fast as the better one of them.  Taken back: operands straight from global memory to registers (the load
// pattern above), four steps in flight (fewer workgroups fit), steps of 32 k.
#pragma once
#include <type_traits>
#include <utility>

#include "gemm_direct_plan.hpp"
#include "gemm_wave.hpp"

namespace tc355 {

struct GemmDirectArgs {
  const void* A;      // [N][K], float or double
  const float* Bm;    // [M][K]
  const float* bias;  // [M], FC only
  float* C;           // [N][M], or nullptr
  double* C64;        // the same in fp64, or nullptr
  unsigned* clear;    // FC: a word that the launch sets to 0, or nullptr
  int N, M, K;
  int tiles_n, tiles_m;  // blocks of 16 RT rows, of 16 CT columns
  int rows_slow;         // order of the tiles: those of one block of rows follow each other
  unsigned first;        // number of the launch's first workgroup (a multiple of 8)
};

// RT x CT tiles of 16 x 16 per workgroup, NW wavefronts
template <typename TA, int RT, int CT, int NW>
struct GemmDirectGeom {
  static constexpr int AI = sizeof(TA) == 8 ? 2 : 1;  // pieces per 16 rows of A
  static constexpr int NP = RT * AI + CT;             // pieces per step
  static constexpr int STEP = NP * 1024;
  static constexpr int PART = RT * CT * 4 * WAVE * 8;  // a wavefront's partial tiles
  static constexpr int WAVE_BYTES = 2 * STEP > PART ? 2 * STEP : PART;
  static constexpr int LDS = NW * WAVE_BYTES;
};

template <int N>
__device__ __forceinline__ void wait_loads() {  // until at most N of the wavefront's loads are in flight
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// 16 bytes per lane to LDS: lane l's to lds + 16 l (a uniform address)
__device__ __forceinline__ void load_to_lds(const char* g, unsigned lds) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(uintptr_t)g,
                                   (__attribute__((address_space(3))) void*)(uintptr_t)lds, 16, 0, 0);
}
// Several 16-byte LDS reads and their wait in one block.  (The compiler, which knows of the loads to LDS, would wait for all
// of them before any LDS read of its own.)
template <int I0, int I1>
__device__ __forceinline__ void lds_read(f4 (&o)[2], const unsigned (&a)[2]) {
  asm volatile("ds_read_b128 %0, %2 offset:%4\n\tds_read_b128 %1, %3 offset:%5\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(o[0]), "=&v"(o[1])
               : "v"(a[0]), "v"(a[1]), "n"(I0), "n"(I1)
               : "memory");
}
template <int I0, int I1, int I2>
__device__ __forceinline__ void lds_read(f4 (&o)[3], const unsigned (&a)[3]) {
  asm volatile("ds_read_b128 %0, %3 offset:%6\n\tds_read_b128 %1, %4 offset:%7\n\tds_read_b128 %2, %5 offset:%8\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2])
               : "v"(a[0]), "v"(a[1]), "v"(a[2]), "n"(I0), "n"(I1), "n"(I2)
               : "memory");
}
template <int I0, int I1, int I2, int I3>
__device__ __forceinline__ void lds_read(f4 (&o)[4], const unsigned (&a)[4]) {
  asm volatile("ds_read_b128 %0, %4 offset:%8\n\tds_read_b128 %1, %5 offset:%9\n\tds_read_b128 %2, %6 offset:%10\n\tds_read_b128 %3, %7 offset:%11\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3])
               : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "n"(I0), "n"(I1), "n"(I2), "n"(I3)
               : "memory");
}
template <int I0, int I1, int I2, int I3, int I4, int I5>
__device__ __forceinline__ void lds_read(f4 (&o)[6], const unsigned (&a)[6]) {
  asm volatile("ds_read_b128 %0, %6 offset:%12\n\tds_read_b128 %1, %7 offset:%13\n\tds_read_b128 %2, %8 offset:%14\n\tds_read_b128 %3, %9 offset:%15\n\tds_read_b128 %4, %10 offset:%16\n\tds_read_b128 %5, %11 offset:%17\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(o[0]), "=&v"(o[1]), "=&v"(o[2]), "=&v"(o[3]), "=&v"(o[4]), "=&v"(o[5])
               : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "n"(I0), "n"(I1), "n"(I2), "n"(I3), "n"(I4), "n"(I5)
               : "memory");
}
// where piece x of a step is read: the two pieces of 16 fp64 rows are addressed from the first one
template <int NA, int AI>
constexpr int piece_offset(int x) { return (x < NA ? x / AI * AI : x) * 1024; }
template <int SO, int NA, int AI, int... I>
__device__ __forceinline__ void read_step(f4 (&o)[sizeof...(I)], const unsigned (&a)[sizeof...(I)], std::integer_sequence<int, I...>) {
  lds_read<(SO + piece_offset<NA, AI>(I))...>(o, a);
}

template <typename TA, bool FC, int RT, int CT, int NW>
__global__ __launch_bounds__(NW * WAVE, RT * CT == 4 ? 3 : 4) void gemm_nt_direct_kernel(GemmDirectArgs p) {
  using Gm = GemmDirectGeom<TA, RT, CT, NW>;
  constexpr bool A64 = sizeof(TA) == 8;
  constexpr int AI = Gm::AI, NP = Gm::NP, PE = A64 ? 2 : 4;  // PE: elements of A per 16 bytes
  extern __shared__ __attribute__((aligned(16))) char gd_lds[];
  const int tid = threadIdx.x;
  if (FC && p.clear && blockIdx.x == 0 && tid == 0) *p.clear = 0;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int r16 = lane & 15, q = lane >> 4;
  const int N = p.N, M = p.M, K = p.K;
  // every XCD (workgroups equal modulo 8) takes a run of tiles: all of the smaller operand and an eighth of the larger one
  const int jobs = p.tiles_n * p.tiles_m, share = (jobs + 7) / 8;
  const unsigned wg = p.first + blockIdx.x;
  const int job = (int)(wg % 8) * share + (int)(wg / 8);
  if (job >= jobs) return;  // (the whole workgroup)
  const int per = p.rows_slow ? p.tiles_m : p.tiles_n, slow = job / per, fast = job - slow * per;
  const int n0 = (p.rows_slow ? slow : fast) * 16 * RT, m0 = (p.rows_slow ? fast : slow) * 16 * CT;
  const int steps = (K + 15) / 16;
  const int s0 = (int)((int64_t)steps * wave / NW), n = (int)((int64_t)steps * (wave + 1) / NW) - s0;  // this wavefront's steps

  // ---- loading: byte offsets of the lane's parts from the operands (32 bits: the host asks gd_reaches)
  const int lr = lane >> 2, lp = (lane & 3) ^ (lane >> 4);
  unsigned aoff[RT], boff[CT];
#pragma unroll
  for (int i = 0; i < RT; i++) aoff[i] = gd_offset(min(n0 + 16 * i + lr, N - 1), PE * lp, K, sizeof(TA));
#pragma unroll
  for (int j = 0; j < CT; j++) boff[j] = gd_offset(min(m0 + 16 * j + lr, M - 1), 4 * lp, K, 4);
  const char* A = static_cast<const char*>(p.A);
  const char* B = reinterpret_cast<const char*>(p.Bm);
  const unsigned ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)gd_lds + (unsigned)wave * Gm::WAVE_BYTES;
  auto load = [&](int slot, int s) {
    const unsigned base = ring + slot * Gm::STEP;
    const int k0 = 16 * s;
    const char* Ak = A + (size_t)k0 * sizeof(TA);
    const char* Bk = B + (size_t)k0 * 4;
    if (k0 + 16 <= K) {
#pragma unroll
      for (int i = 0; i < RT; i++)
#pragma unroll
        for (int z = 0; z < AI; z++) load_to_lds(Ak + aoff[i] + 64 * z, base + (i * AI + z) * 1024);
#pragma unroll
      for (int j = 0; j < CT; j++) load_to_lds(Bk + boff[j], base + (RT * AI + j) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < RT; i++)
#pragma unroll
        for (int z = 0; z < AI; z++) {
          const int group = A64 ? 4 * ((4 * z + lp) >> 1) : 4 * lp;  // first k of the group that this part belongs to
          load_to_lds(Ak + aoff[i] + 64 * z + gd_end_shift(k0, group, K, sizeof(TA)), base + (i * AI + z) * 1024);
        }
#pragma unroll
      for (int j = 0; j < CT; j++) load_to_lds(Bk + boff[j] + gd_end_shift(k0, 4 * lp, K, 4), base + (RT * AI + j) * 1024);
    }
  };

  // ---- contraction: lane (r16, q) takes k = 4 q .. 4 q + 3 of a step: part q of fp32 rows, parts 2 q and 2 q + 1 of fp64 rows
  const unsigned rb = ring + 64 * r16 + 16 * (q ^ (r16 >> 2));
  const unsigned ra0 = A64 ? ring + 1024 * (q >> 1) + 64 * r16 + 16 * ((2 * (q & 1)) ^ (r16 >> 2)) : rb;
  const unsigned ra1 = A64 ? ring + 1024 * (q >> 1) + 64 * r16 + 16 * ((2 * (q & 1) + 1) ^ (r16 >> 2)) : rb;
  d4 acc[RT][CT];
#pragma unroll
  for (int i = 0; i < RT; i++)
#pragma unroll
    for (int j = 0; j < CT; j++) acc[i][j] = d4_zero();
  auto contract = [&](auto slot, int s) {
    f4 o[NP];
    unsigned ad[NP];
#pragma unroll
    for (int x = 0; x < NP; x++) ad[x] = x >= RT * AI ? rb : x % AI == 0 ? ra0 : ra1;
    read_step<decltype(slot)::value * Gm::STEP, RT * AI, AI>(o, ad, std::make_integer_sequence<int, NP>{});
    double a[RT][4];
    float b[CT][4];
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
      for (int e = 0; e < 4; e++) {
        if constexpr (A64) a[i][e] = __builtin_bit_cast(dbl2, o[2 * i + (e >> 1)])[e & 1];
        else a[i][e] = (double)o[i][e];
      }
#pragma unroll
    for (int j = 0; j < CT; j++)
#pragma unroll
      for (int e = 0; e < 4; e++) b[j][e] = o[RT * AI + j][e];
    if (16 * s + 16 > K) {  // (uniform) the last step
      const int moved = min(0, K - 4 - (16 * s + 4 * q));
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const bool in = moved + e >= 0;
#pragma unroll
        for (int i = 0; i < RT; i++) a[i][e] = in ? a[i][e] : 0.0;
#pragma unroll
        for (int j = 0; j < CT; j++) b[j][e] = in ? b[j][e] : 0.f;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; e++)
#pragma unroll
      for (int i = 0; i < RT; i++)
#pragma unroll
        for (int j = 0; j < CT; j++) acc[i][j] = mfma_f64(a[i][e], (double)b[j][e], acc[i][j]);
  };
  auto step = [&](auto slot, int t) {  // (a slot is loaded again only behind the wait for its reads)
    if (t >= n) return;
    if (t + 1 < n) wait_loads<NP>();
    else wait_loads<0>();
    contract(slot, s0 + t);
    if (t + 2 < n) load(decltype(slot)::value, s0 + t + 2);
  };
  if (n > 0) load(0, s0);
  if (n > 1) load(1, s0 + 1);
  for (int t = 0; t < n; t += 2) {
    step(std::integral_constant<int, 0>{}, t);
    step(std::integral_constant<int, 1>{}, t + 1);
  }

  // ---- partial tiles, in the wavefront's own ring: [tile][v][lane]
  auto part = [&](int w) { return reinterpret_cast<double*>(gd_lds + w * Gm::WAVE_BYTES); };
  {
    double* own = part(wave);
#pragma unroll
    for (int i = 0; i < RT; i++)
#pragma unroll
      for (int j = 0; j < CT; j++)
#pragma unroll
        for (int v = 0; v < 4; v++) own[((i * CT + j) * 4 + v) * WAVE + lane] = acc[i][j][v];
  }
  __syncthreads();
  constexpr int ROWS = RT * CT * 4;  // rows of 64 outputs, dealt to the wavefronts
#pragma unroll
  for (int x = 0; x < (ROWS + NW - 1) / NW; x++) {
    const int at = wave + x * NW;
    if (ROWS % NW != 0 && at >= ROWS) break;
    const int t = at >> 2, row = n0 + 16 * (t / CT) + d_row(q, at & 3), col = m0 + 16 * (t % CT) + r16;
    double sum = FC ? (double)p.bias[min(col, M - 1)] : 0.0;  // the listing's first statement
#pragma unroll
    for (int w = 0; w < NW; w++) sum += part(w)[at * WAVE + lane];
    if (FC) sum = relu64(sum);
    if (row < N && col < M) {
      const int64_t c = (int64_t)row * M + col;
      if (p.C) p.C[c] = (float)sum;
      if (FC && p.C64) p.C64[c] = sum;
    }
  }
}

}  // namespace tc355
