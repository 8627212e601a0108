// Which launch of sconv_i8.hpp and of sconv_patch.hpp a strided convolution takes, and what each would need.  Plain C++: a test
// compiles it for the host and asks.
#pragma once
#include <algorithm>
#include <cstdint>

#include "tc355_host.hpp"

namespace tc355 {

constexpr int SP_WAVES = 8;
constexpr int SP_TAPS = 9;
constexpr int SP_POSITIONS = 640;  // input positions of a patch: with the filters' rings all of a compute unit's LDS
constexpr int SP_MAX_TILES = 6;    // pixel tiles per wavefront

// n / d = n * sp_magic(d) >> SP_MAGIC_SHIFT for n, d < 2^11 (a run of pixels and the column of its first one; taps)
constexpr int SP_MAGIC_SHIFT = 21;
inline unsigned sp_magic(int d) { return ((1u << SP_MAGIC_SHIFT) + (unsigned)d - 1) / (unsigned)d; }

constexpr int SI8_BLOCK = 128, SI8_ROW = SI8_BLOCK + 32;  // taps per block of sconv_i8.hpp, bytes of their digits in LDS
// LDS that tf filters, so many tiles of 16 pixels and the table of so many blocks of taps take there
inline int64_t sconv_i8_lds(int64_t tf, int64_t tiles, int64_t blocks) {
  return (tf + 16 * tiles) * (4 * SI8_ROW + 8) + 2 * 16 * tiles * 4 + blocks * SI8_BLOCK * 4;
}
// tiles at a time of a workgroup of sconv_patch.hpp that does its run by taps
constexpr int sp_redo_tiles(int tf) { return tf == 128 ? 3 : tf == 64 ? 4 : 8; }

struct SconvI8Deal {
  int tf, nt;  // filters, tiles of 16 pixels per workgroup
  int64_t gx;  // workgroups per block of filters
  double us;   // estimate of the launch, fitted to 213 layers (errors of 7 %)
};

// sconv_i8.hpp: 128 filters per workgroup and 1 .. 4 pixel tiles, or (a multiple of 64 filters only) 64 filters and 2, 4, 6, 8,
// or (a multiple of 32 only) 32 filters and 4, 8, 12.  As few rounds of workgroups as the largest tile allows, then the smallest
// tile that still makes that number of rounds.
inline bool deal_sconv_i8(int64_t P, int64_t F, int64_t K, int64_t G, int cus, SconvI8Deal* d) {
  const int tf = F % 128 == 0 ? 128 : F % 64 == 0 ? 64 : 32, step = 128 / tf, most = tf == 32 ? 12 : 4 * step;
  const int64_t blocks = ceil_div(K, SI8_BLOCK), units = ceil_div(P, 16), fblocks = F / tf;
  const int64_t per_round = std::max<int64_t>(1, cus / (fblocks * G));
  const int64_t rounds = ceil_div(units, most * per_round);
  int nt = (int)ceil_div(ceil_div(units, rounds * per_round), step) * step;
  nt = std::min(most, std::max(step, nt));
  while (nt > step && sconv_i8_lds(tf, nt, blocks) > 160 * 1024) nt -= step;
  if (sconv_i8_lds(tf, nt, blocks) > 160 * 1024) return false;
  d->tf = tf; d->nt = nt;
  d->gx = ceil_div(units, nt);
  if (d->gx > 2147483647 || fblocks > 65535) return false;
  d->us = (double)ceil_div(d->gx * fblocks * G, std::max(1, cus)) * (4.64 + (double)blocks * (0.82 + 1.12 * (nt / step)));
  return true;
}

struct SconvPatchPlan {
  int tf, tiles;   // filters per workgroup, pixel tiles per wavefront
  int px, blocks;  // pixels per workgroup, runs of them per image
  double us;       // estimate of the launch
};

// The best run of pixels, and an estimate in us; false where the kernel does not take the layer.
//   t = 3.55 + turns * (1.88 + stages * (4.69 + 1.38 * tiles + 0.49 * units * full)), with stages of 32 channels, `units` pieces of
// 4 positions x 4 channels that a thread slices per stage, and `full` the share of the chip that a turn occupies: fitted to 220
// layers at every run (4.4 % rms, 16 % at worst; without the check of the scales, 2 % of a launch).
inline bool plan_sconv_patch(int64_t N, int64_t G, int64_t C, int64_t F, int64_t H, int64_t W, int64_t KH, int64_t KW, int64_t sh, int64_t sw, int cus,
                             SconvPatchPlan* best) {
  if (KH * KW != SP_TAPS || C % 32 != 0 || F % 32 != 0 || KH * W > SP_POSITIONS || H * W >= (1 << 24) || cus <= 0) return false;
  const int64_t OH = (H - KH) / sh + 1, OW = (W - KW) / sw + 1, OHW = OH * OW, tf = F % 128 == 0 ? 128 : F % 64 == 0 ? 64 : 32, pg = 128 / tf;
  if (F / tf > 65535 || G > 65535) return false;
  const int64_t taps_lds = sconv_i8_lds(tf, sp_redo_tiles((int)tf), ceil_div(SP_TAPS * C, SI8_BLOCK));
  if (taps_lds > 160 * 1024) return false;  // (from 1376 channels on at 128 filters, 2240 at 64, 1664 at 32)
  bool any = false;
  for (int64_t tiles = 2; tiles <= SP_MAX_TILES; tiles++) {  // (with one tile the estimate never wins)
    const int64_t most = 16 * tiles * pg;
    const int64_t even = ceil_div(OHW, ceil_div(OHW, most));  // as many runs as that allows, of one length
    for (int64_t px : {even, std::min(most / OW * OW, OHW)}) {  // or whole rows
      if (px <= most - 16 * pg) continue;  // (fewer tiles would do)
      const int64_t rows = px % OW == 0 ? px / OW : std::min(OH, (px + OW - 2) / OW + 1), positions = ((rows - 1) * sh + KH) * W;
      const int64_t blocks = ceil_div(OHW, px), groups = N * blocks * (F / tf) * G;
      if (positions > SP_POSITIONS || N * blocks >= (1ll << 31)) continue;
      const double turns = (double)ceil_div(groups, cus), full = (double)std::min<int64_t>(groups, cus) / cus;
      const double units = (double)ceil_div(8 * ceil_div(positions, 4), 64 * SP_WAVES);
      const double us = 3.55 + turns * (1.88 + (double)(C / 32) * (4.69 + 1.38 * (double)tiles + 0.49 * units * full));
      if (!any || us < best->us) {
        *best = SconvPatchPlan{(int)tf, (int)tiles, (int)px, (int)blocks, us};
        any = true;
      }
    }
  }
  return any;
}

// Whether a layer that `deal` describes goes to sconv_patch.hpp, and how: filters of nine taps over a multiple of 32 channels, the
// input sliced once instead of once per tap, where the estimate of that is 5 % lower (large layers; a small one has too little to do
// between its filters).  Of 220 random layers 25 went over, 1.27 times as fast, none of them slower.  The check of the scales came
// later and takes 2 % on average: of 45 layers just beyond the line 44 are faster than by taps, one is 1 % slower.  (N,C,F,H,W) at stride s:
// (32,64,128,56,56) at 2 46.6 -> 35.3 us, (32,64,64,56,56) at 1 109 -> 68, (15,128,192,13,72) at 1 79 -> 54.5, but (10,64,128,28,28) at 2
// 14.9 / 17.4.
inline bool sconv_by_patches(const SconvI8Deal& deal, int64_t N, int64_t G, int64_t C, int64_t F, int64_t H, int64_t W, int64_t KH, int64_t KW, int64_t sh,
                             int64_t sw, int cus, SconvPatchPlan* best) {
  return plan_sconv_patch(N, G, C, F, H, W, KH, KW, sh, sw, cus, best) && best->us < 0.95 * deal.us;
}

}  // namespace tc355
