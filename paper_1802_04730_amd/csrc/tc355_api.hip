// Host side of libtc355: argument validation, kernel selection and launches
// for the entry points declared in include/tc355.h.
#include "../../include/tc355.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cstdint>
#include <cstdlib>
#include <initializer_list>
#include <random>
#include <type_traits>

#include "gconv_band.hpp"
#include "gconv_i8.hpp"
#include "gconv_i8_c32.hpp"
#include "gemm_direct.hpp"
#include "gemm_i8.hpp"
#include "gconv_i8_small.hpp"
#include "gconv_lds.hpp"
#include "gconv_mix.hpp"
#include "gconv_quad.hpp"
#include "gconv_tiny.hpp"
#include "gconv_wave.hpp"
#include "gemm_tile.hpp"
#include "gemm_wave.hpp"
#include "kron_lds.hpp"
#include "kron_tile.hpp"
#include "kron_wave.hpp"
#include "lut_sum.hpp"
#include "mlp_fused.hpp"
#include "mlp_rows.hpp"
#include "sconv_split.hpp"
#include "sconv_tile.hpp"
#include "sconv_i8.hpp"
#include "sconv_patch.hpp"
#include "tbmm_any.hpp"
#include "tbmm_lds.hpp"
#include "tc355_host.hpp"

using namespace tc355;

namespace {

constexpr int64_t kMaxElems = (int64_t)1 << 31;  // per-tensor element limit of the 32-bit in-tile indexing
constexpr int64_t kMaxGrid = 2147483647;

inline bool misaligned(const void* p, size_t a = 16) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

inline tc_status launch_status() { return hipGetLastError() == hipSuccess ? TC_OK : TC_ERR_LAUNCH; }

// Options of the calling host thread (tc355_set_option) and the kernel family its last call chose (tc355_last_path).
struct ThreadOptions {
  int64_t int8 = TC_INT8_AUTO;
  int64_t mlp_kernel = TC_MLP_AUTO;
  int64_t mlp_spin_limit = 4000000;
};
thread_local ThreadOptions t_opt;
thread_local const char* t_path = "";

inline tc_status took(const char* path, tc_status st) {
  t_path = path;
  return st;
}


// ---- generic wave-level contraction launcher --------------------------------
template <typename TA, int VEC, int EPI>
tc_status launch_gemm_tm(GemmArgs a, int64_t batch, int tm, hipStream_t s) {
  a.tiles_n = (int)ceil_div(a.N, 16);
  a.strips_m = (int)ceil_div(a.M, 16 * tm);
  a.jobs = batch * a.tiles_n * a.strips_m;
  const int64_t grid = ceil_div(a.jobs, WAVES_PER_WG);
  if (grid > kMaxGrid) return TC_ERR_UNSUPPORTED;
  const dim3 g((unsigned)grid), b(WG_THREADS);
  switch (tm) {
    case 1: gemm_nt_wave_kernel<TA, VEC, 1, EPI><<<g, b, 0, s>>>(a); break;
    case 2: gemm_nt_wave_kernel<TA, VEC, 2, EPI><<<g, b, 0, s>>>(a); break;
    case 3: gemm_nt_wave_kernel<TA, VEC, 3, EPI><<<g, b, 0, s>>>(a); break;
    case 4: gemm_nt_wave_kernel<TA, VEC, 4, EPI><<<g, b, 0, s>>>(a); break;
    default: gemm_nt_wave_kernel<TA, VEC, 5, EPI><<<g, b, 0, s>>>(a); break;
  }
  return launch_status();
}

// LDS-tiled kernel for big blocks (64 x 64 output tiles); returns false if it does not apply.
template <typename TA, int EPI>
bool try_gemm_tile(const GemmArgs& a, int64_t batch, hipStream_t s, tc_status* st) {
  if ((a.K % 4 != 0 && a.K < GT_KC) || a.N < 48 || a.M < 48) return false;
  const int64_t tiles = ceil_div(a.N, GT_BM) * ceil_div(a.M, GT_BN);
  if (tiles > kMaxGrid || batch > 65535) return false;
  if (batch > 1 && (a.K % 4 != 0 || tiles * batch < 128)) return false;  // too few blocks to fill the chip: the wave-level kernel spreads wider
  static std::atomic<int> lds_ok{0};  // needs more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_nt_tile_kernel<TA, EPI>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, GT_LDS_BYTES) != hipSuccess) {
      *st = TC_ERR_LAUNCH;
      return true;
    }
    lds_ok.store(1, std::memory_order_release);
  }
  gemm_nt_tile_kernel<TA, EPI><<<dim3((unsigned)tiles, (unsigned)batch), dim3(WG_THREADS), GT_LDS_BYTES, s>>>(a);
  *st = launch_status();
  return true;
}

int device_cus();

bool try_gconv_mix(const GconvArgs& g, hipStream_t s, tc_status* st);  // records "gconv:mix"

// ---- grouped convolution with 4 or 8 channels per group (4x4x4 MFMA blocks), compile-time width; records the path of the
// kernel that it chose --------
template <int C, int F, int KH, int KW, int W, int ROWS, int TN, int MINW>
bool try_gconv_quad(const GconvArgs& g, hipStream_t s, tc_status* st) {
  using Gm = GconvQuadGeom<C, F, KH, KW, W, ROWS, TN>;
  if (g.C != C || g.F != F || g.KH != KH || g.KW != KW || g.W != W) return false;
  const int64_t pairs = (int64_t)g.N * g.G, grid = ceil_div(pairs, 8) * 8 * ceil_div(g.OH, ROWS);
  if (grid > kMaxGrid) return false;
  // Few pairs: the same 4x4x4 blocks in pieces of an image (gconv_mix.hpp), where the estimates of an earlier form of this kernel,
  // one workgroup per pair, say so.  (In bands it is as fast or faster from about 32 pairs of 56 x 56 on, 5.5 us against 11.3
  // at 124; up to there the tests name the other kernel.)
  if (pairs < 125) {
    constexpr int EARLIER = C == 4 ? 16 : W == 28 ? 26 : 14;  // its rows per band
    const double px = (double)pairs * g.OH * g.OW / std::max(1, device_cus());
    const double bands = (C == 4 ? 2.1 : 2.5) + (C == 4 ? (W == 56 ? 2.75 : 2.95) : (W == 28 ? 4.85 : 3.45)) * ceil_div(g.OH, EARLIER);
    const double pieces = C == 4 ? 4.2 + std::min(0.0125 * px, 1.5 + 0.0043 * px) : 4.6 + std::min(0.016 * px, 1.4 + 0.0085 * px);
    if (pieces < bands && try_gconv_mix(g, s, st)) return true;
  }
  t_path = "gconv:quad";
  static std::atomic<int> lds_ok{0};
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gconv_quad_kernel<C, F, KH, KW, W, ROWS, TN, MINW>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, Gm::LDS_BYTES) != hipSuccess) {
      *st = TC_ERR_LAUNCH;
      return true;
    }
    lds_ok.store(1, std::memory_order_release);
  }
  GconvQuadArgs a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.NG = pairs; a.G = g.G; a.H = g.H;
  for (int64_t at = 0; at < grid; at += next_launch(grid - at, WG_THREADS)) {
    a.first = (unsigned)at;
    gconv_quad_kernel<C, F, KH, KW, W, ROWS, TN, MINW><<<dim3((unsigned)next_launch(grid - at, WG_THREADS)), dim3(WG_THREADS), Gm::LDS_BYTES, s>>>(a);
    *st = launch_status();
    if (*st != TC_OK) break;
  }
  return true;
}

// ---- grouped convolution with a large filter bank on tiny images: the bank stays in registers, images stream ----
template <int C, int F, int KH, int KW, int H, int W>
bool try_gconv_tiny(const GconvArgs& g, hipStream_t s, tc_status* st) {
  using Gm = GconvTinyGeom<C, F, KH, KW, H, W>;
  if (g.C != C || g.F != F || g.KH != KH || g.KW != KW || g.H != H || g.W != W) return false;
  const int cus = device_cus();
  if (cus <= 0) return false;
  // about two workgroups per compute unit: each owns one group and a run of images
  const int64_t nchunks = std::min<int64_t>(g.N, std::max<int64_t>(1, 2 * (int64_t)cus / g.G));
  const int64_t chunk = ceil_div(g.N, nchunks);
  GconvTinyArgs a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.N = g.N; a.G = g.G;
  a.chunk = (int)chunk;
  a.nchunks = (int)ceil_div(g.N, chunk);
  const int64_t grid = (int64_t)g.G * a.nchunks;
  if (grid > kMaxGrid) return false;
  gconv_tiny_kernel<C, F, KH, KW, H, W><<<dim3((unsigned)grid), dim3(WG_THREADS), Gm::LDS_BYTES, s>>>(a);
  *st = launch_status();
  return true;
}

// ---- one matrix pair with the reduction split over wavefronts (gemm_direct.hpp) ----
template <typename TA, bool FC, int RT, int CT, int NW>
tc_status launch_gemm_direct(GemmDirectArgs d, hipStream_t s) {
  constexpr int LDS = GemmDirectGeom<TA, RT, CT, NW>::LDS;
  if constexpr (LDS > 64 * 1024) {
    static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
    if (!lds_ok.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(gemm_nt_direct_kernel<TA, FC, RT, CT, NW>), hipFuncAttributeMaxDynamicSharedMemorySize,
                              LDS) != hipSuccess)
        return TC_ERR_LAUNCH;
      lds_ok.store(1, std::memory_order_release);
    }
  }
  d.tiles_n = (int)ceil_div(d.N, 16 * RT);
  d.tiles_m = (int)ceil_div(d.M, 16 * CT);
  d.rows_slow = (int64_t)d.N * (int64_t)sizeof(TA) > (int64_t)d.M * 4;
  const int64_t grid = ceil_div((int64_t)d.tiles_n * d.tiles_m, 8) * 8;
  tc_status st = TC_OK;
  for (int64_t at = 0; at < grid && st == TC_OK; at += next_launch(grid - at, NW * WAVE)) {
    d.first = (unsigned)at;
    gemm_nt_direct_kernel<TA, FC, RT, CT, NW><<<dim3((unsigned)next_launch(grid - at, NW * WAVE)), dim3(NW * WAVE), LDS, s>>>(d);
    st = launch_status();
  }
  return st;
}

template <typename TA, bool FC>
tc_status run_gemm_direct(const GemmArgs& a, int cus, hipStream_t s) {
  GemmDirectArgs d{};
  d.A = a.A; d.Bm = a.Bm; d.bias = a.bias; d.C = a.C; d.C64 = a.C64; d.clear = a.clear;
  d.N = a.N; d.M = a.M; d.K = a.K;
  switch (choose_gemm_direct(a.N, a.M, a.K, sizeof(TA), cus)) {
    case 0: return launch_gemm_direct<TA, FC, 1, 1, 4>(d, s);
    case 1: return launch_gemm_direct<TA, FC, 1, 1, 8>(d, s);
    case 2: return launch_gemm_direct<TA, FC, 1, 1, 16>(d, s);
    case 3: return launch_gemm_direct<TA, FC, 1, 2, 8>(d, s);
    default: return launch_gemm_direct<TA, FC, 2, 2, 4>(d, s);
  }
}

// Lines between the kernels for one plain product with a short reduction, in clocks of a compute unit.  64 x 64 blocks: 3200
// per chunk of 32, one block after the other.  A split reduction over chunks of 128 (16 x 16 tiles): 827 per chunk and 750 per
// tile where two workgroups share a compute unit, 990 and 900 for one alone.  That is the kernel that gemm_direct.hpp took over
// from: the lines between the other two were drawn with it in the middle and have not been drawn again.
double gemm_tile_clocks(const GemmArgs& a, int cus) {
  if (a.N < 48 || a.M < 48 || (a.K % 4 != 0 && a.K < GT_KC)) return 1e30;
  return (double)ceil_div(ceil_div(a.N, GT_BM) * ceil_div(a.M, GT_BN), cus) * ceil_div(a.K, GT_KC) * 3200;
}

double gemm_splitk_clocks(const GemmArgs& a, int cus) {
  const int64_t jobs = ceil_div(a.N, 16) * ceil_div(a.M, 16), nck = ceil_div(a.K, 128), rest = jobs % (2 * cus);
  const double two = 2.0 * (nck * 827 + 750), one = nck * 990.0 + 900;
  return jobs / (2 * cus) * two + (rest > cus ? two : rest > 0 ? one : 0.0);
}

// Does the wave-level kernel beat the better one of these for a plain fp32 product?  Their last chunk (of 128, of 32) is padding
// where a reduction is short or a little longer than whole chunks; the wave-level kernel has no chunks: a wavefront per 16 x 16
// tile, four of them at a time on a compute unit, 43 clocks per k (85 where rows have odd lengths and every operand is a load of
// its own), 1800 more than the tiles and 400 less than the blocks before the first and behind the last.  Fitted to the three
// kernels' times at 600 shapes; measured, wave / tiles / blocks, us: (N,M,K) = (666,773,7) 3.6 / 8.3 / -, (1708,121,21) 3.9 / 5.2 / -,
// (2405,629,29) 11.7 / 19.6 / -, (1219,411,134) 8.4 / 11.2 / 10.3, (115,1632,148) 5.9 / 6.5 / 9.8, (285,1098,54) 5.1 / 5.9 / 5.9,
// but (650,456,144) 8.4 / 7.6 / 10.0 and (1012,1571,43) 13.5 / 20.5 / 9.4.
bool gemm_wave_beats(const GemmArgs& a, double splitk, double tile, int cus) {
  const int64_t jobs = ceil_div(a.N, 16) * ceil_div(a.M, 16);
  if (a.M <= 80 || (a.K % 2 != 0 && a.K >= 32)) return false;  // (a narrow result is one wavefront per 16 rows)
  if (jobs >= 4096) return splitk < tile && a.K < 32;          // (several tiles per wavefront there)
  return 1800 + (double)ceil_div(jobs, 4 * cus) * a.K * (a.K % 2 == 0 ? 43 : 85) < (splitk < tile ? splitk : tile + 2200);
}

template <typename TA, int EPI>
tc_status launch_gemm(const GemmArgs& a, int64_t batch, int tm, hipStream_t s) {
  tc_status st = TC_OK;
  constexpr bool plain = EPI == EPI_NONE;  // tc_tbmm (else: one MLP layer)
  const int cus = device_cus();
  // (32-bit byte offsets in the split-reduction kernel)
  const bool direct = batch == 1 && cus > 0 && a.K >= 4 && gd_reaches(a.N, a.K, sizeof(TA)) && gd_reaches(a.M, a.K, 4) &&
                      ceil_div(a.N, 16) * ceil_div(a.M, 16) < (1ll << 30);
  // The split reduction takes every pair of matrices that it can address, except plain products with a short reduction: up
  // to K = 96 the 64 x 64 blocks and below 160 the wave-level kernel keep what the lines above and below give them.  (It would
  // be as fast or faster there too, (N,M,K) = (1101,1000,33) 8.4 us against 9.6 on blocks, (1500,1500,66) 14.5 against 18.0 and
  // (115,1632,148) 4.7 against 6.1 wave-level, but 10.9 against 10.2 at (128,13248,64) and 12.5 against 11.8 at (256,7696,96): the tests name
  // these kernels there.)
  bool wave = false, blocks = false;
  if (batch == 1 && (plain || !direct)) {
    const double split = direct ? gemm_splitk_clocks(a, cus) : 1e30, tile = cus > 0 ? gemm_tile_clocks(a, cus) : 0.0;
    // The wave-level kernel: a single tile of a short reduction, and large products whose last chunk of 32 would be mostly
    // padding ((N,M,K) = (2136,1047,38) 11.0 us against 13.7 on blocks, (1500,1500,130) 22.3 / 24; at 18 % padding it is even:
    // (1143,2514,130) 26.8 / 25.2).
    wave = (a.N <= 16 && a.M <= 16 && a.K <= 16) ||
           (a.K % 4 == 2 && ceil_div(a.K, GT_KC) * GT_KC * 100 >= (int64_t)a.K * 118 &&
            ceil_div(a.N, GT_BM) * ceil_div(a.M, GT_BN) > 2 * cus) ||
           (plain && direct && gemm_wave_beats(a, split, tile, cus));
    blocks = !wave && tile <= split;
    if (direct) {
      wave = wave && a.K < 160;
      blocks = blocks && a.K <= 96;
    }
  }
  if (direct && !wave && !blocks) return took(plain ? "tbmm:splitk" : "mlp:per_layer", run_gemm_direct<TA, !plain>(a, cus, s));
  if (!wave && try_gemm_tile<TA, EPI>(a, batch, s, &st)) return took(plain ? "tbmm:tile" : "mlp:per_layer", st);
  t_path = plain ? "tbmm:wave" : "mlp:per_layer";
  // widest per-lane load that keeps every row start aligned
  if (a.K % 4 == 0) return launch_gemm_tm<TA, 4, EPI>(a, batch, tm, s);
  if (a.K % 2 == 0) return launch_gemm_tm<TA, 2, EPI>(a, batch, tm, s);
  return launch_gemm_tm<TA, 1, EPI>(a, batch, tm, s);
}

// Strip width (in 16-column tiles) that wastes the fewest padded columns; ties go to the wider strip.
int pick_strip(int64_t M, int64_t waves_if_one) {
  const int64_t tiles = ceil_div(M, 16);
  if (tiles <= 5) return (int)tiles;
  if (waves_if_one < 4096) return 1;  // few jobs: favour parallelism over operand reuse
  int best = 1;
  int64_t best_pad = -1;
  for (int tm = 5; tm >= 2; tm--) {
    const int64_t pad = ceil_div(tiles, tm) * tm - tiles;
    if (best_pad < 0 || pad < best_pad) { best = tm; best_pad = pad; }
  }
  return best;
}

size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

// ---- tuned grouped convolution: returns false if this instance does not apply -----
template <int C, int F, int KH, int KW, int TP>
bool try_gconv_lds(const GconvArgs& g, hipStream_t s, tc_status* st) {
  if (g.C != C || g.F != F || g.KH != KH || g.KW != KW) return false;
  const int npix = g.OH * g.OW;
  const int rows = gconv_band_rows(64 * TP, g.OW, KH);
  const int PS = gconv_plane_stride(rows * g.W);
  const size_t lds = ((size_t)C * PS + (size_t)(F / 16) * (KH * KW * C / 4) * WAVE) * sizeof(float);
  if (lds > 64 * 1024) return false;
  GconvLdsArgs a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.G = g.G; a.H = g.H; a.W = g.W; a.OH = g.OH; a.OW = g.OW;
  a.PS = PS;
  a.pblocks = (int)ceil_div(npix, 64 * TP);
  a.ngs = (int64_t)g.N * g.G;
  const int64_t grid = a.ngs * a.pblocks;
  if (grid > kMaxGrid) return false;
  gconv_lds_kernel<C, F, KH, KW, TP><<<dim3((unsigned)grid), dim3(WG_THREADS), lds, s>>>(a);
  *st = launch_status();
  return true;
}

// ---- grouped convolution for any channel counts and images: 16- and 4-filter MFMA tiles over one LDS band ----
template <int FT, int FQ, int TP>
tc_status launch_gconv_mix(const GconvMixArgs& a, unsigned grid, int64_t lds, hipStream_t s) {
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gconv_mix_kernel<FT, FQ, TP>), hipFuncAttributeMaxDynamicSharedMemorySize,
                            160 * 1024) != hipSuccess)
      return TC_ERR_LAUNCH;
    lds_ok.store(1, std::memory_order_release);
  }
  gconv_mix_kernel<FT, FQ, TP><<<dim3(grid), dim3(WG_THREADS), (size_t)lds, s>>>(a);
  return launch_status();
}

template <int FT, int FQ>
tc_status launch_gconv_mix_tp(int tp, const GconvMixArgs& a, unsigned grid, int64_t lds, hipStream_t s) {
  switch (tp) {
    case 1: return launch_gconv_mix<FT, FQ, 1>(a, grid, lds, s);
    case 2: return launch_gconv_mix<FT, FQ, 2>(a, grid, lds, s);
    case 3: return launch_gconv_mix<FT, FQ, 3>(a, grid, lds, s);
    default: return launch_gconv_mix<FT, FQ, 4>(a, grid, lds, s);
  }
}

bool try_gconv_mix(const GconvArgs& g, hipStream_t s, tc_status* st) {
  GconvMixArgs a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.N = g.N; a.G = g.G; a.C = g.C; a.F = g.F; a.H = g.H; a.W = g.W; a.KH = g.KH; a.KW = g.KW; a.OH = g.OH; a.OW = g.OW;
  GconvMixPlan best{};
  if (!choose_gconv_mix(a, device_cus(), &best)) return false;
  const unsigned grid = gconv_mix_grid(a, best);
  switch (a.fb / 4) {
    case 1: *st = launch_gconv_mix_tp<0, 1>(best.tp, a, grid, best.lds, s); break;
    case 2: *st = launch_gconv_mix_tp<0, 2>(best.tp, a, grid, best.lds, s); break;
    case 3: *st = launch_gconv_mix_tp<0, 3>(best.tp, a, grid, best.lds, s); break;
    case 4: *st = launch_gconv_mix_tp<1, 0>(best.tp, a, grid, best.lds, s); break;
    case 5: *st = launch_gconv_mix_tp<1, 1>(best.tp, a, grid, best.lds, s); break;
    case 6: *st = launch_gconv_mix_tp<1, 2>(best.tp, a, grid, best.lds, s); break;
    case 7: *st = launch_gconv_mix_tp<1, 3>(best.tp, a, grid, best.lds, s); break;
    default: *st = launch_gconv_mix_tp<2, 0>(best.tp, a, grid, best.lds, s); break;
  }
  t_path = "gconv:mix";
  return true;
}

// Number of compute units of the current device (cached per device index).
int device_cus() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
  int cus = cache[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cache[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}

// A fresh 64-bit token per fused-MLP call (low 32 bits never 0): random start, then counting.
unsigned long long next_token() {
  static std::atomic<unsigned long long> tok{[] {
    std::random_device rd;
    unsigned long long t = ((unsigned long long)rd() << 32) ^ rd();
    t ^= (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count();
    return t | 1ull;
  }()};
  unsigned long long t = tok.fetch_add(1, std::memory_order_relaxed);
  while ((t & 0xffffffffull) == 0) t = tok.fetch_add(1, std::memory_order_relaxed);  // low word is what release words carry
  return t;
}

size_t mlp_sync_bytes() { return round256((MLP_SYNC_WORDS + (size_t)(MLP_MAX_LAYERS - 1) * MLP_BAR_WORDS) * sizeof(unsigned)); }

// fp64 copy of one layer's output; whole 16-row tiles (the small-batch kernel keeps it in a tiled layout)
size_t mlp_act_bytes(int64_t batch, int64_t width) {
  return round256((size_t)ceil_div(batch, 16) * 16 * (size_t)width * sizeof(double));
}

// ---- Kronecker layer of any extents with its operands in LDS ----
template <typename TS, int TJ, bool SECOND>
tc_status launch_kron_tile(const KronTileArgs& a, dim3 grid, int64_t lds, hipStream_t s) {
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(kron_tile_kernel<TS, TJ, SECOND>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      return TC_ERR_LAUNCH;
    lds_ok.store(1, std::memory_order_release);
  }
  kron_tile_kernel<TS, TJ, SECOND><<<grid, dim3(KT_THREADS), (size_t)lds, s>>>(a);
  return launch_status();
}

template <typename TS, bool SECOND>
tc_status launch_kron_tile_tj(int tj, const KronTileArgs& a, dim3 grid, int64_t lds, hipStream_t s) {
  switch (tj) {
    case 1: return launch_kron_tile<TS, 1, SECOND>(a, grid, lds, s);
    case 2: return launch_kron_tile<TS, 2, SECOND>(a, grid, lds, s);
    case 3: return launch_kron_tile<TS, 3, SECOND>(a, grid, lds, s);
    case 4: return launch_kron_tile<TS, 4, SECOND>(a, grid, lds, s);
    case 5: return launch_kron_tile<TS, 5, SECOND>(a, grid, lds, s);
    case 6: return launch_kron_tile<TS, 6, SECOND>(a, grid, lds, s);
    case 7: return launch_kron_tile<TS, 7, SECOND>(a, grid, lds, s);
    default: return launch_kron_tile<TS, 8, SECOND>(a, grid, lds, s);
  }
}

// Returns false where no block of 16 rows, of columns and one batch element fit LDS.
bool try_kron_tile(const float* W1, const float* W2, const float* X, float* Y, int64_t B, int64_t I, int64_t K, int64_t J, int64_t L,
                   hipStream_t s, tc_status* st) {
  const int cus = device_cus();
  KronTilePlan best{};
  if (!choose_kron_tile(B, I, K, J, L, cus, &best)) return false;
  if (best.second) {
    std::swap(W1, W2);
    std::swap(I, J);
    std::swap(K, L);
  }
  KronTileArgs a{};
  a.W1 = W1; a.W2 = W2; a.X = X; a.Y = Y;
  a.B = (int)B; a.I = (int)I; a.K = (int)K; a.J = (int)J; a.L = (int)L;
  a.nb = (int)best.nb; a.lsp = (int)best.lsp; a.groups = (int)best.groups;
  a.itb = (int)best.itb; a.jblocks = (int)best.jblocks;
  a.k4 = (int)best.k4; a.ls = (int)best.ls; a.ls1 = (int)best.ls1; a.ls2 = (int)best.ls2; a.xs = (int)best.xs;
  auto magic = [](int64_t d) { return (unsigned)(((1ll << 32) + d - 1) / d); };  // dividends and divisors below 2^16
  a.l_magic = magic(L); a.k_magic = magic(K);
  const dim3 grid((unsigned)kron_tile_workgroups(best, cus), (unsigned)(best.iblocks * best.jblocks));
  const int tj = (int)best.tj;
  if (best.second) *st = best.wide ? launch_kron_tile_tj<double, true>(tj, a, grid, best.lds, s) : launch_kron_tile_tj<float, true>(tj, a, grid, best.lds, s);
  else *st = best.wide ? launch_kron_tile_tj<double, false>(tj, a, grid, best.lds, s) : launch_kron_tile_tj<float, false>(tj, a, grid, best.lds, s);
  return true;
}

// ---- fastest grouped convolution: compile-time width, one workgroup per (image, group) -----
template <int C, int KH, int KW, int W, int ROWS, int MINW>
bool try_gconv_band(const GconvArgs& g, hipStream_t s, tc_status* st) {
  using Gm = GconvBandGeom<C, KH, KW, W, ROWS>;
  if (g.C != C || g.F != Gm::F || g.KH != KH || g.KW != KW || g.W != W) return false;
  const int64_t grid = (int64_t)g.N * g.G;
  if (grid > kMaxGrid) return false;
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gconv_band_kernel<C, KH, KW, W, ROWS, MINW>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, Gm::LDS_BYTES) != hipSuccess) {
      *st = TC_ERR_LAUNCH;
      return true;
    }
    lds_ok.store(1, std::memory_order_release);
  }
  GconvBandArgs a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.G = g.G; a.H = g.H;
  gconv_band_kernel<C, KH, KW, W, ROWS, MINW><<<dim3((unsigned)grid), dim3(WG_THREADS), Gm::LDS_BYTES, s>>>(a);
  *st = launch_status();
  return true;
}

// ---- grouped convolution on the int8 matrix core (sliced fixed-point operands, exact int32 sums) ----
template <int W, int ROWS, int MIND>
bool try_gconv_i8(const GconvArgs& g, int force13, hipStream_t s, tc_status* st) {
  using Gm = GconvI8Geom<W, ROWS>;
  if (g.C != Gm::C || g.F != Gm::F || g.KH != Gm::KH || g.KW != Gm::KW || g.W != W) return false;
  if ((int64_t)g.H * W >= (1 << 24)) return false;  // 32-bit byte offsets inside one (image, group) block of 16 planes
  if ((g.H & 1) || (g.H - (Gm::KH - 1)) % ROWS != 0) return false;  // whole, 16-byte aligned bands only
  const int64_t bands = (int64_t)g.N * g.G * ((g.H - (Gm::KH - 1)) / ROWS);
  if (bands >= (1ll << 31)) return false;
  const int64_t grid = std::min<int64_t>(bands, 2 * (int64_t)device_cus());  // persistent: two workgroups per compute unit
  if (bands * (grid + 1) >= (1ll << 31)) return false;  // the kernel splits the bands in 32-bit arithmetic
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gconv_i8_kernel<W, ROWS, MIND>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, Gm::LDS_BYTES) != hipSuccess) {
      *st = TC_ERR_LAUNCH;
      return true;
    }
    lds_ok.store(1, std::memory_order_release);
  }
  GconvI8Args a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.G = g.G; a.H = g.H; a.N = g.N;
  // Workgroups w and w + grid/2 share a compute unit; the one dispatched first wins the issue slots and runs about
  // a quarter faster, so it takes 3/5 of the pair's bands (measured at configuration 4: 121 us with an even split,
  // 117.5 us at 17/28, 118.5 at 4/7, 119.5 at 9/14).
  a.halves = (grid == 2 * (int64_t)device_cus()) ? (int)(grid / 2) : 0;
  a.num = 3;
  a.den = 5;
  a.force13 = force13;
  gconv_i8_kernel<W, ROWS, MIND><<<dim3((unsigned)grid), dim3(WG_THREADS), Gm::LDS_BYTES, s>>>(a);
  *st = launch_status();
  return true;
}

// ---- transposed batched matmul on small per-batch matrices: flat coalesced strips through per-wavefront LDS ----
struct TbmmLdsPlan {
  int tn, tm, nx, ny, store, ks;  // what a job is and what it needs: load instructions per strip, store mode, k steps
  int64_t strips_n, strips_m, jobs;
  size_t wave_units, lds;         // LDS per wavefront in 16-byte units, per workgroup in bytes
};

// The instantiations that exist; a shape takes the first one that covers its plan.  (KS = 0: any reduction length.)
#define TC355_TBMM_LDS_VARIANTS(V) \
  V(2, 5, 3, 8, TBMM_STORE_FLAT, 7)   /* the benchmark's 26 x 72 x 26, a whole batch element per job */ \
  V(2, 5, 3, 8, TBMM_STORE_FLAT, 0)   \
  V(2, 5, 8, 16, TBMM_STORE_FLAT, 0)  \
  V(2, 1, 3, 2, TBMM_STORE_PIECES, 7) /* the same shape, one 16-column tile per job: few batch elements */ \
  V(2, 1, 3, 2, TBMM_STORE_PIECES, 0) \
  V(2, 1, 3, 2, TBMM_STORE_SCALAR, 0) \
  V(2, 2, 8, 8, TBMM_STORE_PIECES, 0) \
  V(2, 2, 8, 8, TBMM_STORE_SCALAR, 0) /* the paper's own naming of tbmm: output 26 x 26, reduction 72 */ \
  V(2, 1, 8, 8, TBMM_STORE_PIECES, 0) \
  V(2, 1, 8, 8, TBMM_STORE_SCALAR, 0) \
  V(1, 1, 4, 4, TBMM_STORE_PIECES, 0) \
  V(1, 1, 4, 4, TBMM_STORE_SCALAR, 0)

tc_status launch_tbmm_lds(const TbmmLdsPlan& pl, const TbmmLdsArgs& a, int64_t wgs, hipStream_t s) {
#define TC355_TBMM_LDS_TRY(TN_, TM_, NX_, NY_, ST_, KS_)                                                       \
  if (pl.tn == TN_ && pl.tm == TM_ && pl.nx <= NX_ && pl.ny <= NY_ && pl.store == ST_ && (KS_ == 0 || pl.ks == KS_)) { \
    tbmm_lds_kernel<TN_, TM_, NX_, NY_, 1, ST_, KS_><<<dim3((unsigned)wgs), dim3(WG_THREADS), pl.lds, s>>>(a);  \
    return launch_status();                                                                                    \
  }
  TC355_TBMM_LDS_VARIANTS(TC355_TBMM_LDS_TRY)
#undef TC355_TBMM_LDS_TRY
  return TC_ERR_LAUNCH;  // (the plan has looked)
}

// Returns false if the shape is not one for this kernel (the caller then takes the shape-generic kernels).
bool plan_tbmm_lds(int64_t B, int64_t N, int64_t M, int64_t K, TbmmLdsPlan* plan) {
  if ((N * K) % 4 != 0 || (M * K) % 4 != 0 || K > 256) return false;  // strips must start and end on 16-byte boundaries
  const int cus = device_cus();
  if (cus <= 0) return false;
  const int64_t tiles_n = ceil_div(N, 16), tiles_m = ceil_div(M, 16);
  TbmmLdsPlan& pl = *plan;
  pl.tn = tiles_n >= 2 ? 2 : 1;
  pl.strips_n = ceil_div(tiles_n, pl.tn);
  // A whole row of tiles per job (most reuse of the X strip, contiguous results) when that still leaves two
  // wavefronts for every SIMD of the chip; with few jobs, fewer tiles per job: a shorter chain from launch to the
  // last store.
  pl.tm = 1;
  for (int c : {5, 2}) {
    if ((c == 5 ? tiles_m <= 5 && M % 4 == 0 : c <= tiles_m) && B * pl.strips_n * ceil_div(tiles_m, c) >= 8 * (int64_t)cus) {
      pl.tm = c;
      break;
    }
  }
  pl.strips_m = ceil_div(tiles_m, pl.tm);
  const int64_t xrows = std::min<int64_t>(16 * pl.tn, N), yrows = std::min<int64_t>(16 * pl.tm, M);
  const int64_t xu = xrows * K / 4, yu = yrows * K / 4;  // 16-byte pieces per strip
  pl.nx = (int)ceil_div(xu, WAVE);
  pl.ny = (int)ceil_div(yu, WAVE);
  pl.store = (pl.tm == 5) ? TBMM_STORE_FLAT : (M % 4 == 0 ? TBMM_STORE_PIECES : TBMM_STORE_SCALAR);
  pl.ks = (int)ceil_div(K, 4);
  // LDS per wavefront: both strips (one spare piece: the last step of a ragged reduction reads past its row); in
  // the flat store mode the same region then holds the job's block of Z
  pl.wave_units = (size_t)(xu + yu) + 1;
  if (pl.store == TBMM_STORE_FLAT) pl.wave_units = std::max<size_t>(pl.wave_units, (size_t)(xrows * M / 4));
  pl.lds = WAVES_PER_WG * pl.wave_units * 16;
  if (pl.lds > 64 * 1024) return false;
  if (B >= kMaxElems / (pl.strips_n * pl.strips_m)) return false;  // 32-bit job numbers
  pl.jobs = B * pl.strips_n * pl.strips_m;
#define TC355_TBMM_LDS_COVERS(TN_, TM_, NX_, NY_, ST_, KS_) \
  if (pl.tn == TN_ && pl.tm == TM_ && pl.nx <= NX_ && pl.ny <= NY_ && pl.store == ST_ && (KS_ == 0 || pl.ks == KS_)) return true;
  TC355_TBMM_LDS_VARIANTS(TC355_TBMM_LDS_COVERS)
#undef TC355_TBMM_LDS_COVERS
  return false;
}

tc_status run_tbmm_lds(const TbmmLdsPlan& pl, const float* X, const float* Y, float* Z, int64_t N, int64_t M, int64_t K, hipStream_t s) {
  const int cus = device_cus();
  TbmmLdsArgs a{};
  a.X = X; a.Y = Y; a.Z = Z;
  a.N = (int)N; a.M = (int)M; a.K = (int)K;
  a.strips_n = (int)pl.strips_n; a.strips_m = (int)pl.strips_m;
  a.jobs = (int)pl.jobs;
  a.wave_lds_units = (int)pl.wave_units;
  // persistent wavefronts, two workgroups per compute unit (the kernel is compiled for two wavefronts per SIMD);
  // small jobs take fewer registers and less LDS, so more of their workgroups are resident at once
  const int64_t per_cu = pl.tm == 5 ? 2 : std::max<int64_t>(2, std::min<int64_t>(4, (160 * 1024) / (int64_t)pl.lds));
  const int64_t wgs = std::min<int64_t>(ceil_div((int64_t)a.jobs, WAVES_PER_WG), per_cu * cus);
  return launch_tbmm_lds(pl, a, wgs, s);
}

// ---- transposed batched matmul of small matrices of any size ----
template <int TN, int TM>
tc_status launch_tbmm_any(const TbmmAnyPlan& pl, TbmmAnyArgs a, hipStream_t s) {
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    const void* kernels[2] = {reinterpret_cast<const void*>(tbmm_any_kernel<TN, TM, false>), reinterpret_cast<const void*>(tbmm_any_kernel<TN, TM, true>)};
    for (const void* k : kernels)
      if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)TA_MAX_LDS) != hipSuccess) return TC_ERR_LAUNCH;
    lds_ok.store(1, std::memory_order_release);
  }
  const dim3 bd((unsigned)(pl.gm * WAVE), (unsigned)pl.gn, (unsigned)pl.nb);
  for (int64_t at = 0; at < pl.groups;) {
    const int64_t n = next_launch(pl.groups - at, pl.gm * pl.gn * pl.nb * WAVE);
    a.first = (unsigned)at;
    if (a.K % 4 == 0) tbmm_any_kernel<TN, TM, true><<<dim3((unsigned)n), bd, (size_t)pl.lds, s>>>(a);
    else tbmm_any_kernel<TN, TM, false><<<dim3((unsigned)n), bd, (size_t)pl.lds, s>>>(a);
    const tc_status st = launch_status();
    if (st != TC_OK) return st;
    at += n;
  }
  return TC_OK;
}

// The plan of the thread's last shapes: choosing one takes 0.3-4 us of host time, 0.9 on average.
const TbmmAnyPlan* tbmm_any_plan(int64_t B, int64_t N, int64_t M, int64_t K, int cus) {
  struct Entry {
    int64_t B, N, M, K;
    int cus;
    bool any;
    TbmmAnyPlan plan;
  };
  static thread_local Entry last[8] = {};
  Entry& e = last[(uint64_t)(B * 31 + N * 7 + M * 3 + K) % 8];
  if (e.B != B || e.N != N || e.M != M || e.K != K || e.cus != cus) {
    e.any = choose_tbmm_any(B, N, M, K, cus, &e.plan);
    e.B = B; e.N = N; e.M = M; e.K = K; e.cus = cus;
  }
  return e.any ? &e.plan : nullptr;
}

// Reductions up to 103.  That is what the registers of this kernel's earlier form held, and what the estimate was fitted with; it is
// not a limit of this one: on 60 random shapes with K from 104 to 180 it would take half the time of the wave-level kernel, which has
// them (us, that / this: (2648,42,68,130) 80 / 75, (412,79,95,111) 47 / 24.5, (42,78,62,105) 14.8 / 4.0; one is slower, (4287,35,12,104)
// 26.2 / 27.7).
bool try_tbmm_any(const float* X, const float* Y, float* Z, int64_t B, int64_t N, int64_t M, int64_t K, hipStream_t s, tc_status* st) {
  const int cus = device_cus();
  if (cus <= 0 || K > 103 || prod_reaches({B, N, K}, 1ll << 40) || prod_reaches({B, M, K}, 1ll << 40)) return false;
  const TbmmAnyPlan* pl = tbmm_any_plan(B, N, M, K, cus);
  if (!pl) return false;
  TbmmAnyArgs a{};
  a.X = X; a.Y = Y; a.Z = Z;
  a.B = (int)B; a.N = (int)N; a.M = (int)M; a.K = (int)K;
  a.strips_n = (int)pl->strips_n; a.strips_m = (int)pl->strips_m;
  a.direct = pl->direct;
  switch (10 * pl->tn + pl->tm) {
    case 11: *st = launch_tbmm_any<1, 1>(*pl, a, s); break;
    case 12: *st = launch_tbmm_any<1, 2>(*pl, a, s); break;
    case 13: *st = launch_tbmm_any<1, 3>(*pl, a, s); break;
    case 15: *st = launch_tbmm_any<1, 5>(*pl, a, s); break;
    case 21: *st = launch_tbmm_any<2, 1>(*pl, a, s); break;
    case 22: *st = launch_tbmm_any<2, 2>(*pl, a, s); break;
    case 23: *st = launch_tbmm_any<2, 3>(*pl, a, s); break;
    case 31: *st = launch_tbmm_any<3, 1>(*pl, a, s); break;
    case 32: *st = launch_tbmm_any<3, 2>(*pl, a, s); break;
    case 33: *st = launch_tbmm_any<3, 3>(*pl, a, s); break;
    default: return false;
  }
  return true;
}

// ---- the same arithmetic for small images with 32 channels per group ----
template <int H, int W, int MIND>
bool try_gconv_i8_c32(const GconvArgs& g, hipStream_t s, tc_status* st) {
  using Gm = GconvI8C32Geom<H, W>;
  if (g.C != Gm::C || g.F != Gm::F || g.KH != Gm::KH || g.KW != Gm::KW || g.W != W || g.H != H) return false;
  if (g.N % WAVES_PER_WG != 0) return false;  // four images of a group per workgroup
  const int64_t iters = (int64_t)g.G * (g.N / WAVES_PER_WG);
  const int64_t grid = std::min<int64_t>(iters, 2 * (int64_t)device_cus());
  if (iters * (grid + 1) >= (1ll << 32)) return false;  // the kernel splits the iterations in 32-bit arithmetic
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gconv_i8_c32_kernel<H, W, MIND>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, Gm::LDS_BYTES) != hipSuccess) {
      *st = TC_ERR_LAUNCH;
      return true;
    }
    lds_ok.store(1, std::memory_order_release);
  }
  GconvI8C32Args a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.G = g.G; a.N = g.N;
  gconv_i8_c32_kernel<H, W, MIND><<<dim3((unsigned)grid), dim3(WG_THREADS), Gm::LDS_BYTES, s>>>(a);
  *st = launch_status();
  return true;
}

// ---- the same arithmetic for small images (one whole image per wavefront) ----
template <int H, int W, int MIND>
bool try_gconv_i8_small(const GconvArgs& g, hipStream_t s, tc_status* st) {
  using Gm = GconvI8SmallGeom<H, W>;
  if (g.C != Gm::C || g.F != Gm::F || g.KH != Gm::KH || g.KW != Gm::KW || g.W != W || g.H != H) return false;
  if (g.N % WAVES_PER_WG != 0) return false;  // four images of a group per workgroup
  const int64_t iters = (int64_t)g.G * (g.N / WAVES_PER_WG);
  const int64_t grid = std::min<int64_t>(iters, 2 * (int64_t)device_cus());
  if (iters * (grid + 1) >= (1ll << 32)) return false;  // the kernel splits the iterations in 32-bit arithmetic
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(gconv_i8_small_kernel<H, W, MIND>),
                            hipFuncAttributeMaxDynamicSharedMemorySize, Gm::LDS_BYTES) != hipSuccess) {
      *st = TC_ERR_LAUNCH;
      return true;
    }
    lds_ok.store(1, std::memory_order_release);
  }
  GconvI8SmallArgs a{};
  a.I = g.I; a.W1 = g.W1; a.bias = g.bias; a.O = g.O;
  a.G = g.G; a.N = g.N;
  gconv_i8_small_kernel<H, W, MIND><<<dim3((unsigned)grid), dim3(WG_THREADS), Gm::LDS_BYTES, s>>>(a);
  *st = launch_status();
  return true;
}

}  // namespace

extern "C" {

const char* tc_status_string(tc_status s) {
  switch (s) {
    case TC_OK: return "TC_OK";
    case TC_ERR_NULL: return "TC_ERR_NULL: a required pointer is NULL";
    case TC_ERR_SHAPE: return "TC_ERR_SHAPE: an extent or an inferred extent is <= 0";
    case TC_ERR_ALIAS: return "TC_ERR_ALIAS: an output aliases an input";
    case TC_ERR_ALIGN: return "TC_ERR_ALIGN: a base pointer is not 16-byte aligned";
    case TC_ERR_WORKSPACE: return "TC_ERR_WORKSPACE: workspace missing, misaligned or too small";
    case TC_ERR_LAUNCH: return "TC_ERR_LAUNCH: the HIP runtime refused the launch";
    case TC_ERR_UNSUPPORTED: return "TC_ERR_UNSUPPORTED: extents exceed the kernels' index range";
    case TC_ERR_SCRATCH_LIMIT: return "TC_ERR_SCRATCH_LIMIT: the call needs more than the library's static scratch array holds";
  }
  return "unknown tc_status";
}

int tc355_version(void) { return 200; }

tc_status tc355_set_option(tc_option key, int64_t value) {
  switch (key) {
    case TC_OPT_INT8:
      if (value < TC_INT8_AUTO || value > TC_INT8_THIRTEEN) return TC_ERR_SHAPE;
      t_opt.int8 = value;
      return TC_OK;
    case TC_OPT_MLP_KERNEL:
      if (value < TC_MLP_AUTO || value > TC_MLP_PER_LAYER) return TC_ERR_SHAPE;
      t_opt.mlp_kernel = value;
      return TC_OK;
    case TC_OPT_MLP_SPIN_LIMIT:
      if (value < 0) return TC_ERR_SHAPE;
      t_opt.mlp_spin_limit = value;
      return TC_OK;
  }
  return TC_ERR_SHAPE;
}

int64_t tc355_get_option(tc_option key) {
  switch (key) {
    case TC_OPT_INT8: return t_opt.int8;
    case TC_OPT_MLP_KERNEL: return t_opt.mlp_kernel;
    case TC_OPT_MLP_SPIN_LIMIT: return t_opt.mlp_spin_limit;
  }
  return -1;
}

const char* tc355_last_path(void) { return t_path; }

}  // extern "C"

namespace {

// Does (B, N, M, K) belong to the shape class of the int8 transposed-matmul kernel (blocks of 128 rows of X against
// many rows of Y, long reduction)?
bool tbmm_i8_shape(int64_t B, int64_t N, int64_t M, int64_t K) {
  return N % GI8_TN == 0 && K % 4 == 0 && K >= 2 * GI8_KB && M % GI8_TM == 0 && B <= 65535 && N / GI8_TN <= 65535 &&
         (M / GI8_TM) * (N / GI8_TN) * B >= 128;
}

// Does slicing X once, in a kernel of its own, pay?  The extra launch costs 5-7 us; what it saves grows with the number
// of workgroups that would each slice X (M / 64) and with the length of the reduction.  Measured, every workgroup / once, us:
// (B,N,M,K) = (1,128,16384,4096) 133.8 / 109.3, (1,128,8192,2048) 64.0 / 50.8, (1,128,16384,512) 21.1 / 22.1, (2,256,4096,512)
// 20.3 / 22.1.  The line was drawn where an earlier form of the contraction gained less, and leaves some out from K = 1024 on:
// (1,128,16384,1024) 37.7 / 34.3, (1,256,4096,2048) 64.2 / 51.7, (1,512,2048,4096) 122.6 / 93.6.
bool tbmm_presliced_pays(int64_t B, int64_t N, int64_t M, int64_t K) {
  return M / GI8_TM >= 128 && K / GI8_KB >= 16 && B * (N / GI8_TN) <= 65535 && ceil_div(K, GI8_KB) <= kMaxGrid;
}

// bytes of X sliced once for the int8 kernel: digit records, then inverse scales
size_t tbmm_ws_bytes(int64_t B, int64_t N, int64_t K) {
  const int64_t blocks = B * (N / GI8_TN) * ceil_div(K, GI8_KB);
  return (size_t)(blocks * (GI8_XD_BYTES + GI8_XINV_BYTES));
}

tc_status tbmm_run(const float* X, const float* Y, float* Z, int64_t B, int64_t N, int64_t M, int64_t K, void* workspace,
                   size_t workspace_bytes, void* hip_stream) {
  if (!X || !Y || !Z) return TC_ERR_NULL;
  if (B < 0 || N <= 0 || M <= 0 || K <= 0) return TC_ERR_SHAPE;
  if (Z == X || Z == Y) return TC_ERR_ALIAS;
  if (misaligned(X) || misaligned(Y) || misaligned(Z)) return TC_ERR_ALIGN;
  if (B >= kMaxElems || prod_reaches({N, K}, kMaxElems) || prod_reaches({M, K}, kMaxElems) || prod_reaches({N, M}, kMaxElems))
    return TC_ERR_UNSUPPORTED;
  if (B == 0) return TC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  // The paper's largest tmm shape class (blocks of 128 rows against many, long reduction) on the int8 matrix core;
  // option TC_INT8_OFF keeps it on the fp64 kernels.
  if (tbmm_i8_shape(B, N, M, K) && t_opt.int8 != TC_INT8_OFF) {
    static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
    if (!lds_ok.load(std::memory_order_acquire)) {
      const void* kernels[4] = {reinterpret_cast<const void*>(gemm_i8_kernel<2>), reinterpret_cast<const void*>(gemm_i8_kernel<3>),
                                reinterpret_cast<const void*>(gemm_i8_presliced_kernel<2>), reinterpret_cast<const void*>(gemm_i8_presliced_kernel<3>)};
      for (const void* k : kernels)
        if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, std::max(GI8_LDS_BYTES, GP_LDS_BYTES)) != hipSuccess) return TC_ERR_LAUNCH;
      lds_ok.store(1, std::memory_order_release);
    }
    GemmI8Args g{};
    g.X = X; g.Y = Y; g.Z = Z; g.M = (int)M; g.K = (int)K;
    const dim3 grid((unsigned)(M / GI8_TM), (unsigned)B, (unsigned)(N / GI8_TN));
    const bool ten = t_opt.int8 == TC_INT8_TEN;  // 13 digit products unless the caller has said that 10 will do
    // With a workspace X is sliced once, by a kernel of its own, instead of by every workgroup that reads it.
    if (workspace && tbmm_presliced_pays(B, N, M, K) && workspace_bytes >= tbmm_ws_bytes(B, N, K)) {
      const int64_t rblocks = B * (N / GI8_TN), nb = ceil_div(K, GI8_KB);
      i4* xd = static_cast<i4*>(workspace);
      double* xinv = reinterpret_cast<double*>(static_cast<char*>(workspace) + rblocks * nb * GI8_XD_BYTES);
      const dim3 slices((unsigned)nb, (unsigned)rblocks, GI8_TN / 16);
      gemm_i8_slice_x_kernel<<<slices, dim3(WAVE), 0, s>>>(X, (int)K, xd, xinv);
      const tc_status st = launch_status();
      if (st != TC_OK) return st;
      g.Xd = xd; g.Xinv = xinv;
      if (ten) gemm_i8_presliced_kernel<3><<<grid, dim3(GI8_THREADS), GP_LDS_BYTES, s>>>(g);
      else gemm_i8_presliced_kernel<2><<<grid, dim3(GI8_THREADS), GP_LDS_BYTES, s>>>(g);
      return took("tbmm:i8_presliced", launch_status());
    }
    if (ten) gemm_i8_kernel<3><<<grid, dim3(GI8_THREADS), GI8_LDS_BYTES, s>>>(g);
    else gemm_i8_kernel<2><<<grid, dim3(GI8_THREADS), GI8_LDS_BYTES, s>>>(g);
    return took("tbmm:i8", launch_status());
  }

  // (A single pair with 64 k and more is faster with its reduction split: (N,M,K) = (64,64,64) 5.2 -> 3.0 us, (1000,1000,64)
  // 8.7 -> 6.2; below, the strips win: (1000,1000,57) 5.9 against 6.3, (128,300,17) 2.7 against 3.1.)
  // Batches of small matrices; times in us.  The rules were drawn from every kernel's time at 2036 random shapes; at 1527 others
  // the kernel taken is on average 1.3 % from the fastest.
  if (B > 1 || K < 64) {
    tc_status st = TC_OK;
    TbmmLdsPlan pl{};
    const int64_t tiles_m = ceil_div(M, 16);
    if (plan_tbmm_lds(B, N, M, K, &pl)) {
      // The aligned kernel keeps what it takes ((B,N,M,K) = (6300,64,60,4) 19.5, 57.6 on 64 x 64 blocks; (1000,64,64,48)
      // 13.8 / 17.2; (134,68,75,48) 6.4, 7.0 on the other one; (1000,4,4,256) 5.4, 6.8 on the wave-level kernel) except
      // where its jobs fit badly: rows of 5 column tiles of which M fills three quarters at most, pairs of which it fills five
      // sixths ((1265,64,16,48) 17.8 / 8.0, (2000,48,48,48) 24.7 / 19.7, (773,48,48,40) 10.6 / 8.4); results that it stores element
      // by element while the reduction is short ((5274,113,46,8) 70 / 30, (934,70,123,4) 23 / 14) or there are more than two
      // tiles of rows and at most four of columns ((1187,57,38,60) 18.0 / 14.9, but (228,89,67,40) 8.4 / 9.8); its longest strips
      // where there are too few wavefronts to hide their loads ((41,60,81,32) 4.4 / 3.7; from 2 jobs per compute unit on, 4 with
      // such stores and K up to 40, (102,52,52,37) 3.8 / 4.1, (217,20,59,84) 5.0 / 5.6).
      const bool scalar = pl.store == TBMM_STORE_SCALAR;
      const int64_t cols = pl.tm * pl.strips_m;
      const bool any = cols >= 2 * tiles_m ||
                       (pl.tn == 2 && pl.tm > 1 && (scalar ? K <= 31 || (N > 32 && M <= 64 && K % 16 != 0) : 10 * cols >= (pl.tm == 5 ? 13 : 12) * tiles_m)) ||
                       (pl.tn == 2 && pl.tm == 1 && (pl.nx > 3 || pl.ny > 2) && pl.jobs <= (scalar && K <= 40 ? 4 : 2) * device_cus());
      if (B > 1 && any && try_tbmm_any(X, Y, Z, B, N, M, K, s, &st)) return took("tbmm:any", st);
      return took("tbmm:lds", run_tbmm_lds(pl, X, Y, Z, N, M, K, s));
    }
    // What it does not take ran on 64 x 64 blocks or on the wave-level kernel.  The blocks keep matrices that fill them to
    // four fifths ((1000,64,64,64) 19.3, 23.5 on the other one, but (700,96,96,96) 58 / 52), and from K = 88 on also where
    // three fifths of the chip's time would be spent on results ((984,53,56,88) 23.3 / 28.2, (124,108,99,92) 12.6 / 15.9, but
    // (311,64,48,88) 11.3 / 8.5).  The wave-level kernel keeps what is too short to stage ((30000,8,8,8) 14.7 / 15.4,
    // (1175,77,4,1) 4.0 / 4.9), results that are one tile wide or more than 5 where K is a multiple of 16
    // ((5709,51,5,96) 38 / 46, (6,51,120,80) 4.3 / 4.7) or the wide ones' odd reductions are short ((3129,12,92,5) 8.8 / 9.3).
    // Everything else is the other one's: (4000,27,61,35) 38.8 / 17.3, (23986,9,74,12) 87 / 39, (35,55,75,81) 13.7 / 4.5.  (The lines
    // here and above were drawn against its earlier form, a wavefront per strip pair, in which rows at multiples of 16 shared LDS banks.
    // The present one is 1.14 times as fast and has no such rows; it would have the wave-level kernel's share of multiples of 16
    // too: (42,37,11,80) 4.2 / 3.4, (63,30,108,80) 4.4 / 3.7, (3520,100,10,96) 41.7 / 37.7.  Of 91 shapes beside the lines the wave-level
    // kernel's 15 would be 1.14 times as fast on it, the aligned kernel's 76 1.06 times.)
    const int64_t cus = std::max(1, device_cus()), blocks = ceil_div(N, GT_BM) * ceil_div(M, GT_BN) * B, tiles = ceil_div(N, 16) * tiles_m * B;
    const double full = (double)N * M / (ceil_div(N, GT_BM) * GT_BM * ceil_div(M, GT_BN) * GT_BN);
    const bool block = K % 4 == 0 && N >= 48 && M >= 48 && blocks >= 128 &&
                       (full >= 0.8 || (K >= 88 && full * blocks >= 0.575 * (ceil_div(blocks, cus) * cus)));
    const bool wave = (N <= 16 && M <= 16 && K <= 8) || (M <= 16 && K <= (K % 2 != 0 ? 11 : 18) && tiles > 114) ||
                      (K % 16 == 0 && K >= 32 && (M <= 16 || (M > 80 && tiles <= 3229))) || (M > 80 && K % 2 != 0 && K <= 14);
    if (B > 1 && !block && !wave && try_tbmm_any(X, Y, Z, B, N, M, K, s, &st)) return took("tbmm:any", st);
  }

  GemmArgs a{};
  a.A = X; a.Bm = Y; a.bias = nullptr; a.C = Z; a.C64 = nullptr;
  a.strideA = N * K; a.strideB = M * K; a.strideC = N * M;
  a.N = (int)N; a.M = (int)M; a.K = (int)K;
  const int tm = pick_strip(M, B * ceil_div(N, 16) * ceil_div(M, 16));
  return launch_gemm<float, EPI_NONE>(a, B, tm, s);  // records tbmm:tile, tbmm:splitk or tbmm:wave
}

}  // namespace

extern "C" {

tc_status tc_tbmm(const float* X, const float* Y, float* Z, int64_t B, int64_t N, int64_t M, int64_t K,
                  void* hip_stream) {
  return tbmm_run(X, Y, Z, B, N, M, K, nullptr, 0, hip_stream);
}

size_t tc_tbmm_workspace_bytes(int64_t B, int64_t N, int64_t M, int64_t K) {
  if (B <= 0 || N <= 0 || M <= 0 || K <= 0 || B >= kMaxElems || prod_reaches({N, K}, kMaxElems)) return 0;
  if (!tbmm_i8_shape(B, N, M, K) || !tbmm_presliced_pays(B, N, M, K)) return 0;
  return tbmm_ws_bytes(B, N, K);
}

tc_status tc_tbmm_ws(const float* X, const float* Y, float* Z, int64_t B, int64_t N, int64_t M, int64_t K,
                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (workspace && misaligned(workspace)) return TC_ERR_ALIGN;
  if (workspace && (workspace == X || workspace == Y || workspace == Z)) return TC_ERR_ALIAS;
  return tbmm_run(X, Y, Z, B, N, M, K, workspace, workspace_bytes, hip_stream);
}

size_t tc_mlp_fcrelu_workspace_bytes(int64_t batch, int32_t n_layers, const int64_t* dims) {
  if (!dims || batch < 0 || n_layers <= 0 || n_layers > MLP_MAX_LAYERS) return 0;
  if (n_layers == 1) return 0;
  size_t total = mlp_sync_bytes();  // synchronisation words first
  for (int l = 0; l + 1 < n_layers; l++) {
    if (dims[l + 1] <= 0) return 0;
    total += mlp_act_bytes(batch, dims[l + 1]);
  }
  return total;
}

}  // extern "C"

namespace {

// Scratch of tc_mlp_fcrelu_static: one array per GPU that the library runs on, held until the process ends.
// In host code the array's name is only a stand-in; its device address comes from hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[TC_MLP_STATIC_SCRATCH_BYTES];

// Device address of `scratch` on the current device (looked up once per device), or nullptr on failure.
void* static_scratch_ptr() {
  static std::atomic<void*> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  void* ptr = cache[dev].load(std::memory_order_acquire);
  if (!ptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
      (void)hipGetLastError();
      return nullptr;
    }
    cache[dev].store(ptr, std::memory_order_release);
  }
  return ptr;
}

// Both MLP entry points: validation, then the fused kernel or one launch per layer.  `workspace` is device memory.
tc_status mlp_run(const float* I, int64_t batch, int32_t n_layers, const int64_t* dims, const float* const* W,
                  const float* const* bias, float* const* O, void* workspace, size_t workspace_bytes,
                  bool static_scratch, void* hip_stream) {
  if (!I || !dims || !W || !bias || !O) return TC_ERR_NULL;
  if (batch < 0 || n_layers <= 0 || n_layers > MLP_MAX_LAYERS) return TC_ERR_SHAPE;
  for (int l = 0; l <= n_layers; l++)
    if (dims[l] <= 0) return TC_ERR_SHAPE;
  for (int l = 0; l < n_layers; l++)
    if (!W[l] || !bias[l]) return TC_ERR_NULL;
  if (!O[n_layers - 1]) return TC_ERR_NULL;
  if (misaligned(I)) return TC_ERR_ALIGN;
  for (int l = 0; l < n_layers; l++) {
    if (misaligned(W[l]) || misaligned(bias[l]) || (O[l] && misaligned(O[l]))) return TC_ERR_ALIGN;
    if (O[l] && (O[l] == I)) return TC_ERR_ALIAS;
    for (int m = 0; m < n_layers; m++) {
      if (O[l] && (O[l] == W[m] || O[l] == bias[m])) return TC_ERR_ALIAS;
      if (O[l] && m != l && O[l] == O[m]) return TC_ERR_ALIAS;
    }
    if (prod_reaches({dims[l], dims[l + 1]}, kMaxElems) || prod_reaches({std::max<int64_t>(batch, 1), dims[l]}, kMaxElems) ||
        prod_reaches({std::max<int64_t>(batch, 1), dims[l + 1]}, kMaxElems))
      return TC_ERR_UNSUPPORTED;
  }
  const size_t need = tc_mlp_fcrelu_workspace_bytes(batch, n_layers, dims);
  if (static_scratch) {
    if (need > TC_MLP_STATIC_SCRATCH_BYTES) return TC_ERR_SCRATCH_LIMIT;
    if (batch == 0) return TC_OK;
    if (need > 0) {
      workspace = static_scratch_ptr();
      workspace_bytes = TC_MLP_STATIC_SCRATCH_BYTES;
      if (!workspace) return TC_ERR_LAUNCH;
    }
  }
  if (need > 0 && (!workspace || misaligned(workspace, 256) || workspace_bytes < need)) return TC_ERR_WORKSPACE;
  if (batch == 0) return TC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  // workspace: [synchronisation words | fp64 activations of layer 0 | layer 1 | ...]
  char* ws = static_cast<char*>(workspace);
  double* act[MLP_MAX_LAYERS] = {};
  {
    char* pws = ws + mlp_sync_bytes();
    for (int l = 0; l + 1 < n_layers; l++) {
      act[l] = reinterpret_cast<double*>(pws);
      pws += mlp_act_bytes(batch, dims[l + 1]);
    }
  }

  // One persistent kernel for the whole chain when every reduction extent allows 16-byte loads.
  bool fused = t_opt.mlp_kernel != TC_MLP_PER_LAYER;
  for (int l = 0; l < n_layers; l++) fused = fused && (dims[l] % 4 == 0);
  // the fused kernel addresses its operands (fp64 activations, fp32 weights) with 32-bit byte offsets
  for (int l = 0; l < n_layers; l++)
    fused = fused && batch * dims[l] * 8 < (1ll << 32) && dims[l + 1] * dims[l] * 4 < (1ll << 32);
  const int cus = device_cus();
  // Small batches with reductions of at most 1024: one workgroup per compute unit, every XCD's workgroups own an eighth
  // of the column tiles of every layer (mlp_rows.hpp).  Option TC_OPT_MLP_KERNEL = TC_MLP_TILES keeps the tile-stream
  // kernel below.  Fewer than 16 rows go to one launch per layer (here / there, us: one row of 1024 -> 1024 -> 512 -> 256 16.1 / 13.7,
  // two of 128 -> 256 -> 1024 -> 128 14.9 / 10.6, five of 256 -> 1024 -> 2000 13.0 / 8.5, 15 of 1024 -> 1000 6.2 / 5.4), unless the
  // caller asks for this kernel.  16 is not where the two cross: one launch per layer has become the faster one throughout
  // (gemm_direct.hpp; 16 rows of 1024 -> 1024 -> 512 -> 256 15.9 / 14.3, 128 of them 19.8 / 18.1, 128 x 1024 -> 1024 9.0 / 7.6, 512 x 256
  // -> 256 -> 128 11.9 / 6.6, 128 x 256 -> 1024 4.8 / 3.7), but from 16 rows on the tests name this kernel.
  if (fused && cus >= MR_SHARES) {
    const int64_t G = ceil_div(batch, 16);
    const int64_t nwg = std::min<int64_t>(cus, MR_MAX_WG) / MR_SHARES * MR_SHARES;
    int64_t max_ct = 1;  // most column tiles of any layer whose output is handed on
    for (int l = 0; l + 1 < n_layers; l++) max_ct = std::max(max_ct, ceil_div(dims[l + 1], 16));
    const int64_t fstride = 4 * max_ct;
    bool rows = t_opt.mlp_kernel != TC_MLP_TILES && G <= 64 && (batch >= 16 || t_opt.mlp_kernel == TC_MLP_ROWS) &&
                (int64_t)(n_layers - 1) * G * fstride <= (int64_t)(MLP_MAX_LAYERS - 1) * MLP_BAR_WORDS;
    for (int l = 0; l < n_layers && rows; l++)
      rows = (dims[l] == 128 || dims[l] == 256 || dims[l] == 512 || dims[l] == 1024) &&
             mr_deal((int)ceil_div(dims[l + 1], 16), (int)G, (int)(nwg / MR_SHARES)).fits;
    if (rows) {
      MlpRowsArgs a{};
      a.I = I;
      for (int l = 0; l < n_layers; l++) {
        a.W[l] = W[l]; a.bias[l] = bias[l]; a.O[l] = O[l]; a.act[l] = act[l];
      }
      for (int l = 0; l <= n_layers; l++) a.dims[l] = (int)dims[l];
      a.batch = (int)batch; a.n_layers = n_layers; a.groups = (int)G; a.fstride = (int)fstride;
      a.sync = reinterpret_cast<unsigned*>(ws);
      a.token = next_token();
      a.spin_limit = (unsigned)std::max<int64_t>(0, std::min<int64_t>(t_opt.mlp_spin_limit, 0xffffffffll));
      static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
      if (!lds_ok.load(std::memory_order_acquire)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(mlp_rows_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                MR_LDS_BYTES) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(mlp_rows_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                MR_LDS_BYTES) != hipSuccess)
          return TC_ERR_LAUNCH;
        lds_ok.store(1, std::memory_order_release);
      }
      bool wide = true;  // every reduction extent 512 or 1024: the kernel that carries only those layer bodies
      for (int l = 0; l < n_layers; l++) wide = wide && dims[l] >= 512;
      if (wide) mlp_rows_kernel<true><<<dim3((unsigned)nwg), dim3(MR_THREADS), MR_LDS_BYTES, s>>>(a);
      else mlp_rows_kernel<false><<<dim3((unsigned)nwg), dim3(MR_THREADS), MR_LDS_BYTES, s>>>(a);
      return took("mlp:rows", launch_status());
    }
  }
  // The tile-stream kernel as one persistent kernel only where the caller asks for it: one launch per layer is faster
  // (a launch costs 1.7 us, a barrier of 256 workgroups 2-3 us with cold loads behind it: 128 x 600 -> 800 -> 400 -> 200 26.8 us
  // as one kernel, 21.4 as three already before the launches got faster) and waits for nobody.
  if (fused && cus > 0 && t_opt.mlp_kernel != TC_MLP_AUTO) {
    MlpArgs a{};
    a.I = I;
    int64_t max_jobs = 1;
    for (int l = 0; l < n_layers; l++) {
      a.W[l] = W[l]; a.bias[l] = bias[l]; a.O[l] = O[l]; a.act[l] = act[l];
      max_jobs = std::max<int64_t>(max_jobs, ceil_div(batch, 16) * ceil_div(dims[l + 1], 16));
    }
    for (int l = 0; l <= n_layers; l++) a.dims[l] = (int)dims[l];
    a.batch = (int)batch; a.n_layers = n_layers;
    a.sync = reinterpret_cast<unsigned*>(ws);
    a.token = next_token();
    a.spin_limit = (unsigned)std::max<int64_t>(1, std::min<int64_t>(t_opt.mlp_spin_limit, 0xffffffffll));
    const unsigned nwg = (unsigned)std::min<int64_t>(std::min(2 * cus, MLP_FANIN * MLP_GROUPS), max_jobs);  // teams of four wavefronts, all resident: two per compute unit
    static std::atomic<int> lds_ok{0};  // the kernel stages more than the default 64 KiB of LDS
    if (!lds_ok.load(std::memory_order_acquire)) {
      if (hipFuncSetAttribute(reinterpret_cast<const void*>(mlp_fused_kernel),
                              hipFuncAttributeMaxDynamicSharedMemorySize, MLP_TEAMS * MLP_LDS_BYTES) != hipSuccess)
        return TC_ERR_LAUNCH;
      lds_ok.store(1, std::memory_order_release);
    }
    // nwg teams of four wavefronts; MLP_TEAMS of them share a workgroup
    mlp_fused_kernel<<<dim3((nwg + MLP_TEAMS - 1) / MLP_TEAMS), dim3(MLP_TEAMS * WG_THREADS), MLP_TEAMS * MLP_LDS_BYTES, s>>>(a);
    return took("mlp:tiles", launch_status());
  }

  // Otherwise one launch per layer ("mlp:per_layer").
  const void* in = I;
  for (int l = 0; l < n_layers; l++) {
    GemmArgs a{};
    a.A = in; a.Bm = W[l]; a.bias = bias[l]; a.C = O[l]; a.C64 = act[l];
    a.strideA = 0; a.strideB = 0; a.strideC = 0;
    a.clear = l == 0 && n_layers > 1 ? reinterpret_cast<unsigned*>(ws) + MLP_SYNC_ERROR : nullptr;  // nothing here can give up
    a.N = (int)batch; a.M = (int)dims[l + 1]; a.K = (int)dims[l];
    const int tm = pick_strip(dims[l + 1], ceil_div(batch, 16) * ceil_div(dims[l + 1], 16));
    const tc_status st = (l == 0) ? launch_gemm<float, EPI_BIAS_RELU>(a, 1, tm, s)
                                  : launch_gemm<double, EPI_BIAS_RELU>(a, 1, tm, s);
    if (st != TC_OK) return st;
    in = act[l];
  }
  return TC_OK;
}

template <int TF, int TP>
tc_status launch_sconv_split(SconvArgs a, hipStream_t s) {
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(sconv_split_kernel<TF, TP>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      return TC_ERR_LAUNCH;
    lds_ok.store(1, std::memory_order_release);
  }
  a.tiles_f = (int)ceil_div(a.F, 16 * TF);
  const int64_t lds = SconvSplitGeom<TF, TP>::STAGES + ceil_div(a.K, SS_KC) * SS_KC * 4;
  sconv_split_kernel<TF, TP><<<dim3((unsigned)(a.tiles_f * ceil_div(a.P, 16 * TP))), dim3(WG_THREADS), (size_t)lds, s>>>(a);
  return launch_status();
}

// The fp64 kernels of the strided convolution, in clocks; what cannot run is out of reach.
struct SconvFp64Clocks { double tile, split1, split2; };

// Which kernel, from what a compute unit would spend in clocks: blocks one after the other when there are several per
// unit, a single one bound by its chain of chunks (16 taps, 64 with a split reduction); small blocks read a third again
// as long where strides step over the filters (lines of the input that nobody else reads).  The split has to be 4 % better:
// that is what the estimate is worth.  Of 1500 random layers measured on every kernel, 2 take one that is more than 3 % slower
// than the blocks of 64 (9 % at most; without the 4 % and the third 10, and 15.0 -> 16.4 us at (2415,256,174)), and
// the choice is on average 0.7 % from the fastest.  Measured, (pixels, filters, taps): blocks of
// 64 against 16 x 16 with a split reduction (400,64,1029) 40.8 / 10.8 us, (1331,64,9898) 349 / 106, (784,20,425) 19.5 / 6.3;
// (11664,100,576) 45.5 / 54.9, (100352,64,64) 31 / 69; against 32 x 16 (867,215,3136) 113 / 51.6, (53312,20,128) 27.4 / 24.
SconvFp64Clocks sconv_fp64_clocks(int64_t N, int64_t C, int64_t H, int64_t W, int64_t F, int64_t K, int64_t P, bool gaps) {
  const int cus = std::max(1, device_cus());
  const bool offsets = !prod_reaches({N, C, H, W}, (int64_t)1 << 30) && !prod_reaches({F, K}, (int64_t)1 << 30);
  const int64_t chunks = ceil_div(K, SS_KC), table = chunks * SS_KC * 4;
  const bool wide64 = ceil_div(F, SC_BF) * ceil_div(P, 64) >= 2 * cus;
  const double blocks = (double)ceil_div(ceil_div(F, SC_BF) * ceil_div(P, wide64 ? 64 : 32), cus), steps = (double)ceil_div(K, SC_KC);
  SconvFp64Clocks c{9400 + std::max((wide64 ? 2913 : 1303) * steps, blocks * ((wide64 ? 1602 : 816) * steps + 2224)), 1e30, 1e30};
  if (offsets && SconvSplitGeom<2, 1>::STAGES + table <= 160 * 1024 && ceil_div(F, 16) * ceil_div(P, 16) <= kMaxGrid) {
    const double gather = gaps ? 1.35 : 1.0;
    auto split = [&](int tf, double one, double many) {
      const double n = (double)ceil_div(ceil_div(F, 16 * tf) * ceil_div(P, 16), cus);
      return 8175 + (double)K + std::max(one * chunks, n * (gather * many * chunks + 752 * tf));
    };
    c.split1 = split(1, 921, 688);
    c.split2 = split(2, 1510, 1062);
  }
  return c;
}

// Strided convolution on the fp64 matrix core: blocks of 64 filters x 64 or 32 pixels (sconv_tile.hpp), or smaller ones with
// a split reduction (sconv_split.hpp).  The caller's operator says how the two are called.
tc_status launch_sconv_fp64(SconvArgs a, const char* tile_path, const char* split_path, hipStream_t s) {
  const int cus = std::max(1, device_cus());
  const SconvFp64Clocks c = sconv_fp64_clocks(a.N, a.C, a.H, a.W, a.F, a.K, a.P, a.sw > a.KW);
  if (1.04 * std::min(c.split1, c.split2) < c.tile)
    return took(split_path, c.split1 <= c.split2 ? launch_sconv_split<1, 1>(a, s) : launch_sconv_split<2, 1>(a, s));
  a.tiles_f = (int)ceil_div(a.F, SC_BF);
  // 64-pixel blocks when there are at least two of them per compute unit, else 32-pixel blocks (twice as many)
  const bool wide = (int64_t)a.tiles_f * ceil_div(a.P, 64) >= 2 * (int64_t)cus;
  const int64_t grid = (int64_t)a.tiles_f * ceil_div(a.P, wide ? 64 : 32);
  if (grid > kMaxGrid) return TC_ERR_UNSUPPORTED;
  const dim3 gd((unsigned)grid), bd(WG_THREADS);
  if (wide) {
    if (a.K % 4 == 0) sconv_tile_kernel<4, 64><<<gd, bd, SconvGeom<64>::LDS_BYTES, s>>>(a);
    else sconv_tile_kernel<1, 64><<<gd, bd, SconvGeom<64>::LDS_BYTES, s>>>(a);
  } else {
    if (a.K % 4 == 0) sconv_tile_kernel<4, 32><<<gd, bd, SconvGeom<32>::LDS_BYTES, s>>>(a);
    else sconv_tile_kernel<1, 32><<<gd, bd, SconvGeom<32>::LDS_BYTES, s>>>(a);
  }
  return took(tile_path, launch_status());
}

// Strided convolution on the int8 matrix core (sconv_i8.hpp): TF filters against 16 * NT pixels per workgroup.
template <int TF, int NT>
tc_status launch_sconv_i8(const SconvI8Args& a, int64_t blocks, dim3 grid, bool ten, hipStream_t s) {
  constexpr int kLdsMax = 160 * 1024;
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    const void* kernels[2] = {reinterpret_cast<const void*>(sconv_i8_kernel<TF, NT, 2>),
                              reinterpret_cast<const void*>(sconv_i8_kernel<TF, NT, 3>)};
    for (const void* k : kernels)
      if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMax) != hipSuccess) return TC_ERR_LAUNCH;
    lds_ok.store(1, std::memory_order_release);
  }
  const size_t lds = (size_t)SconvI8Geom<TF, NT>::lds_bytes(blocks);
  if (lds > (size_t)kLdsMax) return TC_ERR_LAUNCH;  // (the caller has checked)
  if (ten) sconv_i8_kernel<TF, NT, 3><<<grid, dim3(SI8_THREADS), lds, s>>>(a);
  else sconv_i8_kernel<TF, NT, 2><<<grid, dim3(SI8_THREADS), lds, s>>>(a);
  return launch_status();
}

// The same for nine taps over a multiple of 32 channels, the input sliced where it lies (sconv_patch.hpp).
template <int TF, int NTW>
tc_status launch_sconv_patch(const SconvPatchArgs& a, dim3 grid, hipStream_t s) {
  static std::atomic<int> lds_ok{0};  // more than the default 64 KiB of dynamic LDS
  if (!lds_ok.load(std::memory_order_acquire)) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(sconv_patch_kernel<TF, NTW>), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
      return TC_ERR_LAUNCH;
    lds_ok.store(1, std::memory_order_release);
  }
  const size_t lds = std::max<size_t>(SP_LDS_BYTES, SconvI8Geom<TF, sp_redo_tiles(TF)>::lds_bytes(ceil_div(a.e.K, SI8_KB)));
  if (lds > 160 * 1024) return TC_ERR_LAUNCH;  // (the plan has checked)
  sconv_patch_kernel<TF, NTW><<<grid, dim3(SP_THREADS), lds, s>>>(a);
  return launch_status();
}

template <int TF>
tc_status launch_sconv_patch_tiles(int tiles, const SconvPatchArgs& a, dim3 grid, hipStream_t s) {
  switch (tiles) {
    case 2: return launch_sconv_patch<TF, 2>(a, grid, s);
    case 3: return launch_sconv_patch<TF, 3>(a, grid, s);
    case 4: return launch_sconv_patch<TF, 4>(a, grid, s);
    case 5: return launch_sconv_patch<TF, 5>(a, grid, s);
    default: return launch_sconv_patch<TF, 6>(a, grid, s);
  }
}

tc_status run_sconv_patch(const SconvI8Args& e, int64_t N, const SconvPatchPlan& pl, hipStream_t s) {
  SconvPatchArgs a{};
  a.e = e;
  a.px = pl.px; a.blocks = pl.blocks;
  a.ow_magic = sp_magic(e.OW); a.kw_magic = sp_magic(e.KW);
  const dim3 grid((unsigned)(N * pl.blocks), (unsigned)(e.F / pl.tf), (unsigned)e.G);
  if (pl.tf == 128) return launch_sconv_patch_tiles<128>(pl.tiles, a, grid, s);
  if (pl.tf == 64) return launch_sconv_patch_tiles<64>(pl.tiles, a, grid, s);
  return launch_sconv_patch_tiles<32>(pl.tiles, a, grid, s);
}

// Takes the call if the shape is one the int8 kernel is built for: a multiple of 32 filters, a reduction C * KH * KW
// that is a multiple of 4 and at least 256 taps (two blocks), operands that 32-bit offsets reach, a table of tap
// offsets that fits LDS beside the digit planes (about 17,000 taps); long reductions on few pixels go to fp64 all the same
// (below).
// a.G groups of a.C channels and a.F filters; fp64_next: what is refused here goes to launch_sconv_fp64.
bool try_sconv_i8(const SconvI8Args& a, int64_t N, bool fp64_next, hipStream_t s, tc_status* st) {
  if (t_opt.int8 == TC_INT8_OFF) return false;
  if (a.F % 32 != 0 || a.K % 4 != 0 || a.K < 256) return false;
  if (prod_reaches({N, a.G, a.C, a.H, a.W}, (int64_t)1 << 30)) return false;            // 32-bit byte offsets into I
  if (prod_reaches({N, a.G, a.F, a.OH, a.OW}, (int64_t)1 << 31)) return false;          // 32-bit element offsets into O
  if (a.G > 65535) return false;
  SconvI8Deal deal{};
  if (!deal_sconv_i8(a.P, a.F, a.K, a.G, device_cus(), &deal)) return false;
  const int tf = deal.tf, nt = deal.nt;
  const int64_t blocks = ceil_div(a.K, SI8_KB), gx = deal.gx, fblocks = a.F / tf;
  static_assert(SI8_KB == SI8_BLOCK && SI8_RS == SI8_ROW, "sconv_patch_plan.hpp");
  // A workgroup walks over all taps, 1.9 us per block of 128 and pixel tile of a wavefront, however few workgroups there are: a
  // long reduction on few pixels is faster in fp64 with its reduction split, and no less exact.  The line: estimates of both
  // (this one fitted to 213 layers, errors of 7 %), fp64 where its is 10 % lower; of those layers 60 go over, 1.8 times as fast
  // on average and none slower: (pixels, filters, taps) (64,128,12544) 201 -> 84 us, (192,128,3136) 54.6 -> 23.9, (200,256,1600)
  // 30.8 -> 14.4.  Up to 1152 taps, and for less than one tile of pixels, int8 stays whatever the estimates say: (200,128,576)
  // 14.4 against 7.1, where the tests name it.
  if (fp64_next && a.G == 1 && t_opt.int8 == TC_INT8_AUTO && a.K > 1152 && a.P >= 16) {
    const SconvFp64Clocks c = sconv_fp64_clocks(N, a.C, a.H, a.W, a.F, a.K, a.P, a.sw > a.KW);
    if (std::min({c.tile, c.split1, c.split2}) / 2400 < 0.9 * deal.us) return false;
  }
  SconvPatchPlan patch{};
  if (t_opt.int8 != TC_INT8_TEN && sconv_by_patches(deal, N, a.G, a.C, a.F, a.H, a.W, a.KH, a.KW, a.sh, a.sw, device_cus(), &patch)) {
    *st = run_sconv_patch(a, N, patch, s);
    return true;
  }
  const dim3 grid((unsigned)gx, (unsigned)fblocks, (unsigned)a.G);
  const bool ten = t_opt.int8 == TC_INT8_TEN;  // 13 digit products unless the caller has said that 10 will do
  if (tf == 128) {
    switch (nt) {
      case 1: *st = launch_sconv_i8<128, 1>(a, blocks, grid, ten, s); break;
      case 2: *st = launch_sconv_i8<128, 2>(a, blocks, grid, ten, s); break;
      case 3: *st = launch_sconv_i8<128, 3>(a, blocks, grid, ten, s); break;
      default: *st = launch_sconv_i8<128, 4>(a, blocks, grid, ten, s); break;
    }
  } else if (tf == 64) {
    switch (nt) {
      case 2: *st = launch_sconv_i8<64, 2>(a, blocks, grid, ten, s); break;
      case 4: *st = launch_sconv_i8<64, 4>(a, blocks, grid, ten, s); break;
      case 6: *st = launch_sconv_i8<64, 6>(a, blocks, grid, ten, s); break;
      default: *st = launch_sconv_i8<64, 8>(a, blocks, grid, ten, s); break;
    }
  } else {
    switch (nt) {
      case 4: *st = launch_sconv_i8<32, 4>(a, blocks, grid, ten, s); break;
      case 8: *st = launch_sconv_i8<32, 8>(a, blocks, grid, ten, s); break;
      default: *st = launch_sconv_i8<32, 12>(a, blocks, grid, ten, s); break;
    }
  }
  return true;
}

}  // namespace

extern "C" {

tc_status tc_mlp_fcrelu(const float* I, int64_t batch, int32_t n_layers, const int64_t* dims,
                        const float* const* W, const float* const* bias, float* const* O, void* workspace,
                        size_t workspace_bytes, void* hip_stream) {
  return mlp_run(I, batch, n_layers, dims, W, bias, O, workspace, workspace_bytes, false, hip_stream);
}

tc_status tc_mlp_fcrelu_static(const float* I, int64_t batch, int32_t n_layers, const int64_t* dims,
                               const float* const* W, const float* const* bias, float* const* O,
                               void* hip_stream) {
  return mlp_run(I, batch, n_layers, dims, W, bias, O, nullptr, 0, true, hip_stream);
}

tc_status tc_group_conv_infer(int64_t H, int64_t W, int64_t KH, int64_t KW, int64_t* OH, int64_t* OW) {
  if (!OH || !OW) return TC_ERR_NULL;
  if (H <= 0 || W <= 0 || KH <= 0 || KW <= 0) return TC_ERR_SHAPE;
  if (H - KH + 1 <= 0 || W - KW + 1 <= 0) return TC_ERR_SHAPE;
  *OH = H - KH + 1;
  *OW = W - KW + 1;
  return TC_OK;
}

tc_status tc_group_conv(const float* I, const float* W1, const float* bias, float* O, int64_t N, int64_t G,
                        int64_t C, int64_t F, int64_t H, int64_t W, int64_t KH, int64_t KW, void* hip_stream) {
  if (!I || !W1 || !O) return TC_ERR_NULL;
  if (N < 0 || G <= 0 || C <= 0 || F <= 0) return TC_ERR_SHAPE;
  int64_t OH, OW;
  const tc_status inf = tc_group_conv_infer(H, W, KH, KW, &OH, &OW);
  if (inf != TC_OK) return inf;
  if (O == I || O == W1 || (bias && O == bias)) return TC_ERR_ALIAS;
  if (misaligned(I) || misaligned(W1) || misaligned(O) || (bias && misaligned(bias))) return TC_ERR_ALIGN;
  if (N >= kMaxElems || prod_reaches({C, H, W}, kMaxElems) || prod_reaches({F, OH, OW}, kMaxElems) || prod_reaches({C, KH, KW}, kMaxElems) ||
      prod_reaches({G, F, C, KH, KW}, kMaxElems) || G >= kMaxElems / 16 || F >= kMaxElems / 16)
    return TC_ERR_UNSUPPORTED;
  if (N == 0) return TC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  const int64_t K = C * KH * KW;
  GconvArgs a{};
  a.I = I; a.W1 = W1; a.bias = bias; a.O = O;
  a.N = (int)N; a.G = (int)G; a.C = (int)C; a.F = (int)F; a.H = (int)H; a.W = (int)W;
  a.KH = (int)KH; a.KW = (int)KW; a.OH = (int)OH; a.OW = (int)OW;
  tc_status st = TC_OK;
  // Option TC_OPT_INT8: AUTO = the int8 path where it applies, with the thirteenth to tenth digit products added for
  // heavy-tailed blocks; TEN / THIRTEEN = the same with 10 / 13 products throughout; OFF = the fp64 path for every shape.
  const int64_t i8 = t_opt.int8;
  const int force13 = i8 == TC_INT8_THIRTEEN ? 1 : (i8 == TC_INT8_TEN ? -1 : 0);
  if (i8 != TC_INT8_OFF) {
    if (try_gconv_i8<58, 8, 3>(a, force13, s, &st)) return took("gconv:i8", st);
    if (i8 == TC_INT8_TEN) {
      if (try_gconv_i8_small<14, 14, 3>(a, s, &st)) return took("gconv:i8_small", st);  // the paper's (32,32,16,16,14,14)
      if (try_gconv_i8_c32<7, 7, 3>(a, s, &st)) return took("gconv:i8_c32", st);     // the paper's (32,32,32,32,7,7)
      if (try_gconv_i8_small<16, 16, 3>(a, s, &st)) return took("gconv:i8_small", st);  // the first with a border of one pixel
    } else {
      if (try_gconv_i8_small<14, 14, 2>(a, s, &st)) return took("gconv:i8_small", st);
      if (try_gconv_i8_c32<7, 7, 2>(a, s, &st)) return took("gconv:i8_c32", st);
      if (try_gconv_i8_small<16, 16, 2>(a, s, &st)) return took("gconv:i8_small", st);
    }
    // groups with a multiple of 64 filters and at least 256 taps (G = 1: the plain convolution of Section 3): the
    // strided convolution's int8 kernel with stride 1, one grid plane per group
    if (C * KH * KW < kMaxElems && N * OH * OW < kMaxElems) {
      SconvI8Args e{};
      e.I = I; e.Wt = W1; e.bias = bias; e.O = O;
      e.C = (int)C; e.F = (int)F; e.H = (int)H; e.W = (int)W; e.KH = (int)KH; e.KW = (int)KW; e.sh = 1; e.sw = 1;
      e.OH = (int)OH; e.OW = (int)OW; e.K = (int)(C * KH * KW); e.P = (int)(N * OH * OW); e.G = (int)G;
      if (try_sconv_i8(e, N, F >= 64, s, &st)) return took("gconv:i8_taps", st);
    }
  }
  if (try_gconv_band<16, 3, 3, 58, 8, 2>(a, s, &st)) return took("gconv:band", st);
  if (try_gconv_band<16, 3, 3, 14, 12, 2>(a, s, &st)) return took("gconv:band", st);  // the paper's (32,32,16,16,14,14): the whole image is one band
  if (try_gconv_quad<4, 4, 3, 3, 56, 9, 4, 4>(a, s, &st)) return st;    // the paper's (32,32,4,4,56,56)
  if (try_gconv_quad<8, 8, 3, 3, 28, 13, 3, 3>(a, s, &st)) return st;    // the paper's (32,32,8,8,28,28): two bands
  if (try_gconv_quad<4, 4, 3, 3, 58, 8, 4, 4>(a, s, &st)) return st;    // the same two with a border of one pixel
  if (try_gconv_quad<8, 8, 3, 3, 30, 14, 7, 2>(a, s, &st)) return st;
  if (try_gconv_tiny<32, 32, 3, 3, 7, 7>(a, s, &st)) return took("gconv:tiny", st);       // the paper's (32,32,32,32,7,7)
  // 16 channels, any image: blocks of 448 pixels where one or two of them fit the image closely and there are enough, else
  // blocks of the image's own measure (gconv_mix.hpp).  Measured at 32 groups, batch 16 (lds / mix, us): 22 x 24 26.7 / 29.1,
  // 30 x 30 48.5 / 53.6, 22 x 22 26.1 / 27.3; 9 x 9 23.5 / 9.2, 28 x 28 48.2 / 42.8, 33 x 33 84.9 / 55.4, 46 x 46 145 / 101,
  // 56 x 56 156 / 148.
  {
    const int64_t npix = OH * OW, pblocks = ceil_div(npix, 448);
    if (W % 2 == 0 && pblocks <= 2 && npix * 100 >= pblocks * 448 * 85 && !prod_reaches({N, G, pblocks}, kMaxElems) &&
        N * G * pblocks >= device_cus() && try_gconv_lds<16, 16, 3, 3, 7>(a, s, &st))
      return took("gconv:lds", st);
  }
  // G = 1 is the plain convolution of Section 3: the strided convolution's fp64 kernel (implicit contraction over
  // all pixels of the batch in blocks of 64 x 64) where there are at least 64 filters and 64 taps to fill its blocks
  if (G == 1 && F >= 64 && C * KH * KW >= 64 && !prod_reaches({N, C, H, W}, kMaxElems) && !prod_reaches({N, F, OH, OW}, kMaxElems) &&
      !prod_reaches({N, OH, OW}, kMaxElems)) {
    SconvArgs e{};
    e.I = I; e.Wt = W1; e.bias = bias; e.O = O;
    e.N = (int)N; e.C = (int)C; e.F = (int)F; e.H = (int)H; e.W = (int)W; e.KH = (int)KH; e.KW = (int)KW;
    e.sh = 1; e.sw = 1; e.OH = (int)OH; e.OW = (int)OW; e.K = (int)(C * KH * KW); e.P = (int)(N * OH * OW);
    return launch_sconv_fp64(e, "gconv:tile", "gconv:split", s);
  }
  // The shape-generic kernels: gconv_mix.hpp ("gconv:mix"), except where a reduction is so short that there is nothing
  // to stage (1 x 1 filters on 4 channels, 32 x 32 x (16 x 21): 5.6 us on the wave kernel, 6.0 on the other) or a
  // launch so small that the shorter chain wins (120 outputs of 12 taps: 3.5 us against 4.0).
  const bool tiny = K <= 4 || (K <= 16 && !prod_reaches({N, G, F, OH, OW}, 256));
  if (!tiny && try_gconv_mix(a, s, &st)) return st;
  t_path = "gconv:wave";
  // generic kernel: a wavefront takes 16 filters x a strip of 16*TP pixels; small images take a narrower strip
  const int64_t tiles_p = ceil_div(OH * OW, 16);
  const int tp = tiles_p >= 4 ? 4 : (tiles_p >= 2 ? 2 : 1);
  a.tiles_f = (int)ceil_div(F, 16);
  a.strips_p = (int)ceil_div(OH * OW, 16 * tp);
  a.jobs = N * G * a.tiles_f * a.strips_p;
  const int64_t grid = ceil_div(a.jobs, WAVES_PER_WG);
  if (grid > kMaxGrid) return TC_ERR_UNSUPPORTED;
  const dim3 gd((unsigned)grid), bd(WG_THREADS);
  if (tp == 4) gconv_wave_kernel<4><<<gd, bd, 0, s>>>(a);
  else if (tp == 2) gconv_wave_kernel<2><<<gd, bd, 0, s>>>(a);
  else gconv_wave_kernel<1><<<gd, bd, 0, s>>>(a);
  return launch_status();
}

tc_status tc_kron(const float* W1, const float* W2, const float* X, float* Y, int64_t B, int64_t I, int64_t K,
                  int64_t J, int64_t L, void* hip_stream) {
  if (!W1 || !W2 || !X || !Y) return TC_ERR_NULL;
  if (B < 0 || I <= 0 || K <= 0 || J <= 0 || L <= 0) return TC_ERR_SHAPE;
  if (Y == W1 || Y == W2 || Y == X) return TC_ERR_ALIAS;
  if (misaligned(W1) || misaligned(W2) || misaligned(X) || misaligned(Y)) return TC_ERR_ALIGN;
  if (B >= kMaxElems || prod_reaches({I, K}, kMaxElems) || prod_reaches({J, L}, kMaxElems) || prod_reaches({K, L}, kMaxElems) ||
      prod_reaches({I, J}, kMaxElems))
    return TC_ERR_UNSUPPORTED;
  if (B == 0) return TC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  KronArgs a{};
  a.W1 = W1; a.W2 = W2; a.X = X; a.Y = Y;
  a.I = (int)I; a.K = (int)K; a.J = (int)J; a.L = (int)L;
  if (K == 64 && L == 64 && J == 64) {
    KronLdsArgs f{};
    f.W1 = W1; f.W2 = W2; f.X = X; f.Y = Y;
    f.I = (int)I;
    f.iblocks = (int)ceil_div(I, 64);
    const int64_t fgrid = B * f.iblocks;
    if (fgrid <= kMaxGrid) {
      kron_lds_kernel<64, 64, 64><<<dim3((unsigned)fgrid), dim3(WG_THREADS), 0, s>>>(f);
      return took("kron:lds", launch_status());
    }
  }
  // The shape-generic kernels: operands in LDS ("kron:tile") wherever a block of them fits (up to about 140 of every
  // extent, more where others are smaller): 22.7 -> 7.8 us at (B,I,K,J,L) = (200,48,50,75,36), 243 -> 49 us at
  // (500,96,100,100,100), 528 -> 193 at (600,128,128,128,128), never slower from 8^5 up; the wave-level kernel keeps the rest.
  {
    tc_status st = TC_OK;
    if (try_kron_tile(W1, W2, X, Y, B, I, K, J, L, s, &st)) return took("kron:tile", st);
  }
  constexpr int TJ = 4;
  a.tiles_i = (int)ceil_div(I, 16);
  a.blocks_j = (int)ceil_div(J, 16 * TJ);
  a.jobs = B * a.tiles_i * a.blocks_j;
  const int64_t grid = ceil_div(a.jobs, WAVES_PER_WG);
  if (grid > kMaxGrid) return TC_ERR_UNSUPPORTED;
  kron_wave_kernel<TJ><<<dim3((unsigned)grid), dim3(WG_THREADS), 0, s>>>(a);
  return took("kron:wave", launch_status());
}

tc_status tc_sconv2d_infer(int64_t H, int64_t W, int64_t KH, int64_t KW, int64_t sh, int64_t sw, int64_t* OH,
                           int64_t* OW) {
  if (!OH || !OW) return TC_ERR_NULL;
  if (H <= 0 || W <= 0 || KH <= 0 || KW <= 0 || sh <= 0 || sw <= 0) return TC_ERR_SHAPE;
  if (H < KH || W < KW) return TC_ERR_SHAPE;
  *OH = (H - KH) / sh + 1;
  *OW = (W - KW) / sw + 1;
  return TC_OK;
}

tc_status tc_sconv2d(const float* I, const float* Wt, const float* bias, float* O, int64_t N, int64_t C, int64_t F,
                     int64_t H, int64_t W, int64_t KH, int64_t KW, int64_t sh, int64_t sw, void* hip_stream) {
  if (!I || !Wt || !O) return TC_ERR_NULL;
  if (N < 0 || C <= 0 || F <= 0) return TC_ERR_SHAPE;
  int64_t OH, OW;
  const tc_status inf = tc_sconv2d_infer(H, W, KH, KW, sh, sw, &OH, &OW);
  if (inf != TC_OK) return inf;
  if (O == I || O == Wt || (bias && O == bias)) return TC_ERR_ALIAS;
  if (misaligned(I) || misaligned(Wt) || misaligned(O) || (bias && misaligned(bias))) return TC_ERR_ALIGN;
  const int64_t N1 = std::max<int64_t>(N, 1);
  if (prod_reaches({N1, C, H, W}, kMaxElems) || prod_reaches({F, C, KH, KW}, kMaxElems) ||
      prod_reaches({N1, OH, OW}, kMaxElems) || prod_reaches({F, OH, OW}, kMaxElems) || sh >= kMaxElems || sw >= kMaxElems)
    return TC_ERR_UNSUPPORTED;
  const int64_t K = C * KH * KW;
  if (N == 0) return TC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  {
    SconvI8Args e{};
    e.I = I; e.Wt = Wt; e.bias = bias; e.O = O;
    e.C = (int)C; e.F = (int)F; e.H = (int)H; e.W = (int)W; e.KH = (int)KH; e.KW = (int)KW; e.sh = (int)sh; e.sw = (int)sw;
    e.OH = (int)OH; e.OW = (int)OW;
    e.K = (int)K; e.P = (int)(N * OH * OW); e.G = 1;
    tc_status st = TC_OK;
    if (try_sconv_i8(e, N, true, s, &st)) return took("sconv:i8", st);
  }

  SconvArgs a{};
  a.I = I; a.Wt = Wt; a.bias = bias; a.O = O;
  a.N = (int)N; a.C = (int)C; a.F = (int)F; a.H = (int)H; a.W = (int)W; a.KH = (int)KH; a.KW = (int)KW;
  a.sh = (int)sh; a.sw = (int)sw; a.OH = (int)OH; a.OW = (int)OW;
  a.K = (int)K; a.P = (int)(N * OH * OW);
  return launch_sconv_fp64(a, "sconv:tile", "sconv:split", s);
}

tc_status tc_lut(int32_t n_tables, const float* const* LUT, const int32_t* const* Idx, float* const* O,
                 const int64_t* E, const int64_t* L, int64_t D, int64_t B, void* hip_stream) {
  if (!LUT || !Idx || !O || !E || !L) return TC_ERR_NULL;
  if (n_tables <= 0 || n_tables > LUT_MAX_TABLES || D <= 0 || B < 0) return TC_ERR_SHAPE;
  for (int t = 0; t < n_tables; t++) {
    if (!LUT[t] || !Idx[t] || !O[t]) return TC_ERR_NULL;
    if (E[t] <= 0 || L[t] <= 0) return TC_ERR_SHAPE;
  }
  for (int t = 0; t < n_tables; t++) {
    if (misaligned(LUT[t]) || misaligned(Idx[t]) || misaligned(O[t])) return TC_ERR_ALIGN;
    for (int m = 0; m < n_tables; m++) {
      if (static_cast<const void*>(O[t]) == LUT[m] || static_cast<const void*>(O[t]) == Idx[m]) return TC_ERR_ALIAS;
      if (m != t && O[t] == O[m]) return TC_ERR_ALIAS;
    }
    if (prod_reaches({std::max<int64_t>(B, 1), L[t]}, kMaxElems) || E[t] > (int64_t)INT32_MAX + 1) return TC_ERR_UNSUPPORTED;
  }
  if (prod_reaches({std::max<int64_t>(B, 1), D}, kMaxElems)) return TC_ERR_UNSUPPORTED;
  if (B == 0) return TC_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);

  LutArgs a{};
  for (int t = 0; t < n_tables; t++) {
    a.LUT[t] = LUT[t]; a.Idx[t] = Idx[t]; a.O[t] = O[t]; a.E[t] = E[t]; a.L[t] = (int)L[t];
  }
  a.D = (int)D; a.B = (int)B;
  // (the limit of the entry point)
  if ((int64_t)n_tables * B * ceil_div(D % 4 == 0 ? D / 4 : D, WG_THREADS) > kMaxGrid) return TC_ERR_UNSUPPORTED;
  const int v = D >= 4 ? 4 : 1;
  const int64_t units = ceil_div(D, v);
  int cpw = 1;
  while (cpw < units && cpw < WG_THREADS) cpw *= 2;
  a.cpw = cpw;
  a.blocks = (int)ceil_div(units, cpw);
  // as many slots as leave no thread more than one round of lookups
  const int64_t longest = *std::max_element(L, L + n_tables);
  int slots = 1;
  while (slots * cpw < WG_THREADS && ceil_div(longest, slots) > LUT_NB) slots *= 2;
  a.slots = slots;
  const int64_t grid = ceil_div(B, WG_THREADS / (slots * cpw)) * a.blocks;
  if (grid > kMaxGrid) return TC_ERR_UNSUPPORTED;
  const dim3 g((unsigned)grid, (unsigned)n_tables);
  if (v == 4) lut_sum_kernel<4><<<g, dim3(WG_THREADS), 0, s>>>(a);
  else lut_sum_kernel<1><<<g, dim3(WG_THREADS), 0, s>>>(a);
  return took("lut:sum", launch_status());
}

}  // extern "C"
