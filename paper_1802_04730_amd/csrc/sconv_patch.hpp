// Strided convolution (Section 3, listing sconv2d) on the int8 matrix core for filters of nine taps over a multiple of 32
// channels and a multiple of 32 filters:
//
//   O(n,f,h,w) = B(f) + sum_{c,kh,kw} I(n,c, sh*h + kh, sw*w + kw) * W(f,c,kh,kw)
//
// sconv_i8.hpp gathers every tap of every pixel and slices it: an element of the input as often as there are taps over it, the
// filters as often as there are workgroups.  Here a workgroup slices the rows of the input that its pixels touch ONCE, where they
// lie, and a tap is an offset into them.
//
// A workgroup of 8 wavefronts owns TF filters and a run of up to 16 NTW PG pixels of one image (PG = 8 / (TF / 16) wavefronts
// per filter tile) and walks over the channels, 32 at a time:
//   * Patch: the input rows under the run, whole rows, so that a channel's part is one contiguous run of memory.  A thread slices
//     pieces of 4 positions x 4 channels (four 16-byte loads, requested a stage ahead); LDS holds [16 channels][digit][position][16
//     bytes].  One scale for the patch of a stage.
//   * Filters: a wavefront slices the 16 filters of its own tile, in registers, in operand order; nobody else has them.  Their taps
//     lie channel by channel in memory; pieces of 4 channels x 2 travel to a private LDS ring (global_load_lds) and are read back
//     tap by tap.  Scale per filter and stage.
//   * Contraction: an MFMA step is 2 taps x 32 channels (lane (r16, q): tap 2 s + q / 2, channels 16 (q % 2) ..), rows =
//     pixels, columns = filters.  An operand read touches 16 positions sw apart.  The hardware serves lanes 0-3, 12-15 and 20-27
//     together (then 4-11, 16-19, 28-31; the same 32 lanes on): half of them are of the other 16 channels.  At stride 1 their
//     pieces of 16 bytes fill the banks where both halves of the channels start on the same one; at even strides both would take
//     the even pieces, so there the second half starts one piece later: 10.2 -> 6.2 clocks per read at stride 2 and 56 columns
//     (counted from that order, which explains every stride measured), bank-conflict cycles of the launch 5.9 -> 3.4
//     million, 35.9 -> 34.9 us.  The 13 digit products of a tile are summed over all taps of the stage before they are
//     scaled: 9 taps x 32 channels instead of 128 taps.
// The arithmetic is that of sconv_i8.hpp (32-bit fixed point, four signed 8-bit digits, the products with k + l >= 2 summed
// exactly in int32, fp64 over the stages, one rounding).  An element is off by at most 2^-31 of the binade that its scale is taken
// for, by nothing where it is above 2^-7 of it.  That the scale is shared is only sound while no output suffers from what it does
// not read, so a run is done by patches only if, in every stage and in either half of its channels (16 channels x 9 taps, about a
// block of sconv_i8.hpp), the patch's scale is taken for at most 2^SP_SPREAD times the binade of the largest element of EVERY pixel's own window,
// and each filter's for at most that of its own half (halves of zeros alone are exact and do not count).  A run that fails is
// done by the workgroup from its first channel on as sconv_i8.hpp does it, with a scale per pixel and 128 taps.  The check (every
// position's largest magnitude, which the patch's is made of as well, the maximum of nine of them per pixel, the minimum over the
// pixels) takes 0 .. 6 % of a launch, 2 % on average.  Where runs fail, the launch takes (us, all Gaussian / one element of 1e4 / log-normal, sigma 1.5 /
// sconv_i8.hpp): (N,C,F,H,W) = (32,64,128,56,56) at stride 2 35.3 / 52 / 63 / 46.6, (32,64,64,56,56) at 1 68 / 88 / 112 / 109,
// (12,96,96,45,46) at 1 42.5 / 84 / 85 / 95.  SP_SPREAD = 3: of patches of 11 rows of 56, emulated, fail at 1, 2, 3, 4: Gaussian 22 %,
// none, none, none; rectified channels of different mean and size 83 %, 16 %, none, none; Student-t(3) all, 99 %, 67 %, 14 %; log-normal, sigma
// 1.5, all, all, all, 90 %.  Where a window of Gaussian data just passes, the roundings are a quarter of the one to fp32, 3 % more error in all.
// Errors on the metric: 1.1e-7 .. 1.8e-7 on Gaussian data, 2e-7 .. 4.5e-7 on heavy-tailed.
// Inf and NaN reach what they reach there: a position that holds one is left out of the patch (and of its scale) and marked, and
// pixels whose window touches a mark become NaN; a filter that holds one gives NaN everywhere.
// (N,C,F,H,W) at stride s, sconv_i8.hpp -> this, us: (32,64,128,56,56) at 2 46.6 -> 35.3, (32,64,64,56,56) at 1 109 -> 68,
// (3,128,256,58,58) at 1 71 -> 51, (15,128,192,13,72) at 1 79 -> 54.5.  What bounds it: a stage of 6 tiles is 8 us, 5.2 of them MFMAs at
// their rate; the 4 to 5 us in front of it are vector instructions (the filters' slicing above all) and LDS round trips that
// nothing covers, so layers with few pixels per compute unit stay with sconv_i8.hpp.  Filters straight from memory in
// operand order would touch 32 lines per load; scratch registers (one 64-bit address per load kept over the loop) cost 9 us.
#pragma once
#include "sconv_i8.hpp"
#include "sconv_patch_plan.hpp"

namespace tc355 {

struct SconvPatchArgs {
  SconvI8Args e;
  int px, blocks;     // pixels per workgroup, runs of them per image (blockIdx.x = image * blocks + run)
  unsigned ow_magic, kw_magic;  // sp_magic of OW, KW
};

constexpr int SP_THREADS = SP_WAVES * WAVE;
constexpr int SP_PLANE = SP_POSITIONS * 16;    // one digit of 16 channels
constexpr int SP_GROUP = 4 * SP_PLANE;
constexpr int SP_UNITS = (2 * SP_POSITIONS + SP_THREADS - 1) / SP_THREADS;  // (4 positions, 4 channels) per thread
constexpr int SP_RAW = 32 * SP_TAPS * 16;  // 16 filters x 4 channels x 2, all taps
constexpr int SP_RING = 2 * SP_GROUP + 256;    // 8 wavefronts x 2 of them (behind a second group that may start 16 bytes later)
constexpr int SP_MAXIMA = SP_RING + SP_WAVES * 2 * SP_RAW;  // [2] largest magnitude of a stage's patch; [1] without Inf and NaN
constexpr int SP_LEAST = 4;                    // (words behind those) [2] smallest window maximum of a stage; [1] some filter asks for taps
constexpr int SP_UNEVEN = 6;
constexpr int SP_MARKS = SP_MAXIMA + 32;       // [position] holds Inf or NaN in some channel
constexpr int SP_TOPS = SP_MARKS + SP_POSITIONS;  // [position][half of the channels] largest magnitude, 16 bits of it, rounded up
constexpr int SP_LDS_BYTES = SP_TOPS + SP_POSITIONS * 4;
constexpr int SP_SPREAD = 3;                   // binades between a scale and what it is taken for, at most
static_assert(SP_LDS_BYTES <= 160 * 1024, "one workgroup per compute unit");

// Exponent of the binade that a scale is made for, from the bits of the largest magnitude.  (Significands above 0xFEFEFE count as
// the next binade's.)
__device__ __forceinline__ int sp_binade(unsigned mbits) { return (int)max((mbits + 0x10101u) >> 23, 1u); }
// The power of two that takes the largest magnitude just below the largest number of four signed digits, 0x7F7F7F7F, and its
// inverse: elements above 2^-7 of the maximum become integers without rounding.
__device__ __forceinline__ void sp_scales(unsigned mbits, double& scale, double& inverse) {
  const int e = sp_binade(mbits);
  scale = __hiloint2double((1023 + 157 - e) << 20, 0);
  inverse = i8_nonfinite(mbits) ? __longlong_as_double(0x7ff8000000000000ll) : __hiloint2double((1023 - 157 + e) << 20, 0);
}

// n / d for n and d below 2^11 and magic = sp_magic(d)
static_assert(SP_MAX_TILES * 16 * SP_WAVES / 2 + SP_POSITIONS <= 1 << 11, "a run of pixels from the last column on (KH * W, so OW too, is at most SP_POSITIONS)");
__device__ __forceinline__ int sp_div(int n, unsigned magic) { return (int)(((unsigned)n * magic) >> SP_MAGIC_SHIFT); }

// Largest magnitude of four elements, as bits; NaN is the largest.
__device__ __forceinline__ int sp_max4(float a, float b, float c, float d) {
  float m;
  asm("v_maximum3_f32 %0, |%1|, |%2|, |%3|" : "=v"(m) : "v"(a), "v"(b), "v"(c));
  asm("v_maximum3_f32 %0, %0, |%1|, |%1|" : "+v"(m) : "v"(d));
  return __float_as_int(m);
}
// v, where what is made of it shall not be kept in registers over the loop around
__device__ __forceinline__ int sp_here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// 16 bytes per lane to LDS: lane l's to lds + 16 l.  In assembly: the compiler would wait for such loads before any LDS read.
__device__ __forceinline__ void sp_load_to_lds(const char* base, unsigned off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory", "m0");
}

template <int TF, int NTW>
__global__ __launch_bounds__(SP_THREADS, 1) void sconv_patch_kernel(SconvPatchArgs args) {
  const SconvI8Args& p = args.e;
  constexpr int FT = TF / 16, PG = SP_WAVES / FT;
  constexpr int STEPS = (SP_TAPS + 1) / 2;
  extern __shared__ __attribute__((aligned(16))) char sp_lds[];
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int r16 = lane & 15, q = lane >> 4;
  const int W = p.W, HW = p.H * W, OW = p.OW, OHW = p.OH * OW, C = p.C;
  constexpr int KHW = SP_TAPS;
  const int grp = blockIdx.z, f0 = blockIdx.y * TF;
  const int img = blockIdx.x / args.blocks, p0 = ((int)blockIdx.x - img * args.blocks) * args.px;
  const int npx = min(args.px, OHW - p0);
  const int row0 = p0 / OW, col0 = p0 - row0 * OW;                       // the first pixel
  const int rows = sp_div(col0 + npx - 1, args.ow_magic) * p.sh + p.KH;      // input rows
  const int npos = rows * W;                                             // at most SP_POSITIONS (the host asks)
  const int ft = wave % FT, pg = wave / FT;
  const int group = SP_GROUP + (p.sw % 2 == 0 ? 16 : 0);  // from the first 16 channels' records to the others' (see Contraction above)
  unsigned* maxima = reinterpret_cast<unsigned*>(sp_lds + SP_MAXIMA);
  unsigned char* marks = reinterpret_cast<unsigned char*>(sp_lds + SP_MARKS);
  if (tid < 8) maxima[tid] = (tid & ~1) == SP_LEAST ? 0x7fffffffu : 0u;
  for (int i = tid; i < SP_POSITIONS / 4; i += SP_THREADS) reinterpret_cast<int*>(marks)[i] = 0;

  // ---- patch: unit j of this thread is 4 positions (the last ones moved back to end with the run) x 4 channels: quad cq of 8
  const int quads = (npos + 3) >> 2, rounds = (8 * quads + SP_THREADS - 1) / SP_THREADS;  // (uniform)
  unsigned goff[SP_UNITS];
  int loff[SP_UNITS];
#pragma unroll
  for (int j = 0; j < SP_UNITS; j++) {
    const int u = min(j * SP_THREADS + tid, 8 * quads - 1), cq = u & 7, pos = min(4 * (u >> 3), npos - 4);
    goff[j] = 4u * (unsigned)(4 * cq * HW + pos);
    loff[j] = (cq >> 2) * group + pos * 16 + 4 * (cq & 3);
  }
  const float* in = p.I + ((int64_t)img * p.G + grp) * C * HW + (int64_t)row0 * p.sh * W;
  f4 pre[SP_UNITS][4];  // [channel][position]
  auto fetch = [&](int c0) {  // (every register gets a value on every way: a kept one would stay live all along)
    const char* at = reinterpret_cast<const char*>(in + (int64_t)c0 * HW);
#pragma unroll
    for (int c = 0; c < 4; c++) {
      const char* plane = at + 4 * (int64_t)c * HW;
      asm volatile("" : "+s"(plane));  // (a scalar base and a 32-bit offset: not 64-bit addresses kept over the loop)
#pragma unroll
      for (int j = 0; j < SP_UNITS; j++) {
        pre[j][c] = f4{0.f, 0.f, 0.f, 0.f};
        if (j < rounds && c0 < C) pre[j][c] = *reinterpret_cast<const f4_any*>(plane + goff[j]);
      }
    }
  };
  auto patch_max = [&]() {
    int sm = 0;
    unsigned um = 0;
#pragma unroll
    for (int j = 0; j < SP_UNITS; j++)
      if (j < rounds) {
#pragma unroll
        for (int c = 0; c < 4; c++) gi8_absmax4(pre[j][c], sm, um);
      }
    return i8_wave_max((unsigned)gi8_magnitude(sm, um));
  };
  auto post = [&](unsigned* to) {
    const unsigned m = patch_max();
    if (lane == 0) __hip_atomic_fetch_max(to, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };

  // what the pixels' windows hold: every position's largest magnitude in either half of the channels ..
  auto post_tops = [&](unsigned* to) {
    const int t0 = sp_here(tid);
    int all = 0;
#pragma unroll
    for (int j = 0; j < SP_UNITS; j++)
      if (j < rounds) {
        int top = 0;  // of position t0 % 4 of the piece: four neighbouring lanes have the 16 channels
#pragma unroll
        for (int e = 0; e < 4; e++) {
          int v = sp_max4(pre[j][0][e], pre[j][1][e], pre[j][2][e], pre[j][3][e]);
          v = max(v, __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xF, 0xF, false));  // quad_perm [1,0,3,2]
          v = max(v, __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xF, 0xF, false));  // quad_perm [2,3,0,1]
          top = (t0 & 3) == e ? v : top;
        }
        const int at = min(16 * ((j * SP_THREADS + t0) >> 3), 4 * npos - 16) + 4 * (t0 & 3) + 2 * ((t0 >> 2) & 1);
        if (j * SP_THREADS + t0 < 8 * quads) *reinterpret_cast<unsigned short*>(sp_lds + SP_TOPS + at) = (unsigned short)((unsigned)(top + 0xffff) >> 16);
        all = max(all, top);
      }
    const unsigned m = i8_wave_max((unsigned)all);
    if (lane == 0) __hip_atomic_fetch_max(to, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  // .. and the smallest of the pixels' own, a thread per pixel; windows of zeros alone are exact and do not count
  const int astep = 4 * (p.KW == 3 ? W : p.KW == 1 ? 3 * W : 3), bstep = 4 * (p.KW == 1 ? W : 1);  // tap 3 a + b of 3 x 3, 9 x 1, 1 x 9
  auto post_least = [&](unsigned* to) {
    typedef unsigned short us2 __attribute__((ext_vector_type(2)));
    if (WAVE * wave >= npx) return;  // (uniform)
    const int px = min(sp_here(tid), npx - 1) + col0, oh = sp_div(px, args.ow_magic), at = SP_TOPS + 4 * (oh * p.sh * W + (px - oh * OW) * p.sw);
    us2 v = {0, 0};
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
      for (int b = 0; b < 3; b++) v = __builtin_elementwise_max(v, *reinterpret_cast<const us2*>(sp_lds + (at + a * astep + b * bstep)));
    // less one, which is below the maximum whatever its rounding and makes nothing the largest
    const unsigned least = i8_wave_min(min((unsigned)v[0] - 1u, (unsigned)v[1] - 1u) & 0x7fffffffu);
    if (lane == 0) __hip_atomic_fetch_min(to, least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };

  // ---- filters of this wavefront's tile: pieces of quarter j of a stage (channels 4 j .. + 3 of both groups), filter by filter
  const unsigned ring = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)sp_lds + SP_RING + (unsigned)wave * (2 * SP_RAW);
  const char* wt = reinterpret_cast<const char*>(p.Wt + ((int64_t)grp * p.F + f0 + 16 * ft) * C * KHW);
  unsigned woff[STEPS];  // byte offset of the lane's pieces from the quarter's first one
#pragma unroll
  for (int i = 0; i < STEPS; i++) {
    const int u = min(WAVE * i + lane, 32 * KHW - 1), fg = u / KHW;
    woff[i] = 4u * (unsigned)((fg >> 1) * C * KHW + (fg & 1) * 16 * KHW) + 16u * (unsigned)(u - fg * KHW);
  }
  auto load_raw = [&](int c0, int j) {
    const char* at = wt + (int64_t)(c0 + 4 * j) * KHW * 4;
#pragma unroll
    for (int i = 0; i < STEPS; i++)
      if (WAVE * i + lane < 32 * KHW) sp_load_to_lds(at, woff[i], ring + (unsigned)(j & 1) * SP_RAW + 1024u * i);
  };
  f4 raw[STEPS][4];
  auto read_raw = [&](int j) {
    const float* src = reinterpret_cast<const float*>(sp_lds + SP_RING + wave * (2 * SP_RAW) + (j & 1) * SP_RAW) + (2 * r16 + (q & 1)) * 4 * KHW + (q >> 1);
#pragma unroll
    for (int s = 0; s < STEPS; s++) {
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const float v = src[2 * s + e * KHW];
        raw[s][j][e] = 2 * s + 1 < KHW || q < 2 ? v : 0.f;  // (the last step has one tap)
      }
    }
  };

  // ---- contraction: pixel tiles pg, pg + PG, .. against the wavefront's filter tile
  unsigned base[NTW], toff[STEPS];
#pragma unroll
  for (int i = 0; i < NTW; i++) {
    const int px = min(16 * (pg + PG * i) + r16, npx - 1) + col0, oh = sp_div(px, args.ow_magic), ow = px - oh * OW;
    base[i] = 16u * (unsigned)(oh * p.sh * W + ow * p.sw);
  }
#pragma unroll
  for (int s = 0; s < STEPS; s++) {
    const int tap = min(2 * s + (q >> 1), KHW - 1), kh = sp_div(tap, args.kw_magic), kw = tap - kh * p.KW;
    toff[s] = 16u * (unsigned)(kh * W + kw) + (unsigned)((q & 1) * group);
  }
  double acc[NTW][4];
#pragma unroll
  for (int i = 0; i < NTW; i++)
#pragma unroll
    for (int v = 0; v < 4; v++) acc[i][v] = 0.0;
  bool marked = false;  // (uniform) some position is
  bool redo = false;

  fetch(0);
  load_raw(0, 0);
  load_raw(0, 1);
  __syncthreads();  // the cleared words
  for (int c0 = 0, t = 0; c0 < C; c0 += 32, t ^= 1) {
    post_tops(maxima + t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    read_raw(0);
    read_raw(1);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    load_raw(c0, 2);
    load_raw(c0, 3);
    __syncthreads();  // (also: everybody has contracted the stage before)
    unsigned m = __builtin_amdgcn_readfirstlane(maxima[t]);
    if (i8_nonfinite(m)) {  // (uniform) leave such elements out, mark their positions
      marked = true;
#pragma unroll
      for (int j = 0; j < SP_UNITS; j++)
        if (j < rounds) {
#pragma unroll
          for (int c = 0; c < 4; c++)
#pragma unroll
            for (int e = 0; e < 4; e++)
              if (i8_nonfinite(__float_as_uint(pre[j][c][e]) & 0x7fffffffu)) {
                pre[j][c][e] = 0.f;
                marks[((loff[j] >= SP_GROUP ? loff[j] - group : loff[j]) >> 4) + e] = 1;
              }
        }
      post(maxima + 2);
      __syncthreads();
      m = __builtin_amdgcn_readfirstlane(maxima[2]);
      __syncthreads();
      if (tid == 0) maxima[2] = 0;
    }
    if (tid == 0) {  // read a stage ago, written behind the next barrier
      maxima[t ^ 1] = 0;
      maxima[SP_LEAST + (t ^ 1)] = 0x7fffffffu;
    }
    double pscale, pinverse;
    sp_scales(m, pscale, pinverse);
#pragma unroll
    for (int j = 0; j < SP_UNITS; j++)
      if (j < rounds) {
#pragma unroll
        for (int e = 0; e < 4; e++) {
          int y[4];
          gi8_digits4(f4{pre[j][0][e], pre[j][1][e], pre[j][2][e], pre[j][3][e]}, pscale, y);
#pragma unroll
          for (int k = 0; k < 4; k++) *reinterpret_cast<int*>(sp_lds + loff[j] + 16 * e + k * SP_PLANE) = y[k];
        }
      }
    post_least(maxima + SP_LEAST + t);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    read_raw(2);
    read_raw(3);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (c0 + 32 < C) {
      load_raw(c0 + 32, 0);
      load_raw(c0 + 32, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    // the filters' scale and digits, in operand order
    i4 wd[STEPS][4];
    double factor;
    {
      int sm = 0;
      unsigned um = 0;
#pragma unroll
      for (int s = 0; s < STEPS; s++)
#pragma unroll
        for (int j = 0; j < 4; j++) gi8_absmax4(raw[s][j], sm, um);
      int v = gi8_magnitude(sm, um);
      v = max(v, __shfl_xor(v, 32));
      const int half = v;  // channels 16 (q % 2) ..
      v = max(v, __shfl_xor(v, 16));
      if (__any(half != 0 && sp_binade((unsigned)v) > sp_binade((unsigned)half) + SP_SPREAD)) maxima[SP_UNEVEN] = 1;
      double scale, inverse;
      sp_scales((unsigned)v, scale, inverse);
      factor = inverse * pinverse * 16777216.0;  // 2^24: the weight of the lowest kept diagonal
#pragma unroll
      for (int s = 0; s < STEPS; s++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          int y[4];
          gi8_digits4(raw[s][j], scale, y);
#pragma unroll
          for (int k = 0; k < 4; k++) wd[s][k][j] = y[k];
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    fetch(c0 + 32);  // (registers: not before the filters are digits)
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();  // the patch's digits
    // a scale too coarse for some window or some half of a filter: the run by taps
    redo = sp_binade(m) > (int)(__builtin_amdgcn_readfirstlane(maxima[SP_LEAST + t]) >> 7) + SP_SPREAD ||
           __builtin_amdgcn_readfirstlane(maxima[SP_UNEVEN]) != 0;
    if (redo) break;  // (uniform in the workgroup)
#pragma unroll
    for (int i = 0; i < NTW; i++) {
      __builtin_amdgcn_sched_barrier(0);
      // order: no two consecutive products on one diagonal
      constexpr int PK[13] = {3, 2, 3, 3, 2, 1, 2, 1, 0, 3, 2, 1, 0};
      constexpr int PL[13] = {0, 1, 1, 2, 2, 2, 3, 3, 3, 3, 0, 1, 2};
      i4 d[5];  // d[x]: diagonal k + l = 2 + x
      bool begun[5] = {};  // (compile-time after unrolling)
#pragma unroll
      for (int s = 0; s < STEPS; s++) {
        const char* at = sp_lds + (base[i] + toff[s]);
        i4 ya[4];
#pragma unroll
        for (int k = 0; k < 4; k++) ya[k] = *reinterpret_cast<const i4*>(at + k * SP_PLANE);
#pragma unroll
        for (int pr = 0; pr < 13; pr++) {
          const int dg = PK[pr] + PL[pr] - 2;
          d[dg] = mfma_i8(ya[PK[pr]], wd[s][PL[pr]], begun[dg] ? d[dg] : i4{0, 0, 0, 0});
          begun[dg] = true;
        }
      }
#pragma unroll
      for (int v = 0; v < 4; v++) {
        // 288 terms of at most 2^14 per digit pair: 288 x 2^14 x 256 + 2 x 288 x 2^14 stays below 2^31, the next pair of
        // diagonals (three and four digit pairs) would not
        const int hi = d[4][v] * 256 + d[3][v];
        double rr = __builtin_fma((double)d[2][v], 256.0, (double)d[1][v]);
        rr = __builtin_fma((double)hi, 65536.0, rr);
        rr = __builtin_fma((double)d[0][v], 0.00390625, rr);
        acc[i][v] = __builtin_fma(rr, factor, acc[i][v]);
      }
    }
  }

  if (redo) {  // (nothing of the above is kept)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // loads on their way to LDS
    constexpr int NT = sp_redo_tiles(TF);
    for (int at = 0; at < npx; at += 16 * NT) {
      __syncthreads();  // LDS is free
      const int first = img * OHW + p0 + at;
      sconv_i8_block<TF, NT, 2>(p, sp_lds, first, min(first + 16 * NT, img * OHW + p0 + npx), f0, grp);
    }
    return;
  }

  if (marked) {  // (uniform) pixels whose window touches a mark
#pragma unroll 1
    for (int i = 0; i < NTW; i++)
#pragma unroll 1
      for (int v = 0; v < 4; v++) {
        const int px = min(16 * (pg + PG * i) + 4 * q + v, npx - 1) + col0, oh = sp_div(px, args.ow_magic), ow = px - oh * OW;
        const unsigned char* at = marks + (oh * p.sh * W + ow * p.sw);
        bool hit = false;
        for (int kh = 0; kh < p.KH; kh++)
          for (int kw = 0; kw < p.KW; kw++) hit |= at[kh * W + kw] != 0;
#pragma unroll
        for (int a = 0; a < NTW; a++)
#pragma unroll
          for (int b = 0; b < 4; b++)
            if (hit && a == i && b == v) acc[a][b] = __longlong_as_double(0x7ff8000000000000ll);
      }
  }

  // ---- outputs: staged in the patch's LDS as [filter][pixel], written as runs of consecutive pixels of one filter
  constexpr int TP = 16 * NTW * PG, OS = TP + 1;  // odd: the 16 filters of a wavefront's write fall into 16 banks
  static_assert(TF * OS * 4 <= SP_RING, "the output stage fits the patch");
  float* ostage = reinterpret_cast<float*>(sp_lds);
  __syncthreads();
  {
    const double bz = p.bias ? (double)p.bias[grp * p.F + f0 + 16 * ft + r16] : 0.0;
#pragma unroll
    for (int i = 0; i < NTW; i++)
#pragma unroll
      for (int v = 0; v < 4; v++) ostage[(16 * ft + r16) * OS + 16 * (pg + PG * i) + 4 * q + v] = (float)(acc[i][v] + bz);
  }
  __syncthreads();
  float* out = p.O + (((int64_t)img * p.G + grp) * p.F + f0) * OHW + p0;
  for (int idx = tid; idx < TF * TP; idx += SP_THREADS) {
    const int fl = idx / TP, px = idx - fl * TP;
    if (px < npx) store_stream(out + (int64_t)fl * OHW + px, ostage[fl * OS + px]);
  }
}

}  // namespace tc355
