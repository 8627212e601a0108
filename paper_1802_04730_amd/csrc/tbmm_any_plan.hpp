// Which launch of tbmm_any.hpp a batch takes: tiles per wavefront, wavefronts per strip pair, batch elements per workgroup, where
// results are laid out.  Plain C++: a test compiles it for the host and asks what its shapes take.
#pragma once
#include <algorithm>
#include <cstdint>

#include "tc355_host.hpp"

namespace tc355 {

constexpr int TA_MAX_WAVES = 8;
constexpr int64_t TA_MAX_LDS = 160 * 1024;

struct TbmmAnyTile {
  int tn, tm;
  int waves;  // per SIMD, as the registers allow
};
constexpr TbmmAnyTile TA_TILES[] = {{1, 1, 8}, {1, 2, 8}, {1, 3, 8}, {1, 5, 5}, {2, 1, 8}, {2, 2, 8}, {2, 3, 5}, {3, 1, 8}, {3, 2, 5}, {3, 3, 4}};

// The constants of the estimate below, in clocks (per 64 bytes and wavefront: TA_LOAD; bytes a clock and compute unit: TA_BW):
// fitted to 500 shapes (K up to 103) measured in every plan, with most weight on what the chosen plan loses (1.6 % on average, a quarter at
// worst) and on plans slower than what the wave-level strips that this kernel took over from needed.
constexpr double TA_CVT = 1.63, TA_WAVE = 390, TA_OUT_DIRECT = 18.8, TA_OUT_LDS = 26.2, TA_LATENCY = 2680, TA_LOAD = 2.29, TA_LAYOUT = 462, TA_BW = 9.73,
                 TA_BW_DIRECT = 0.952, TA_MFMA_CHAIN = 13.4, TA_UNEVEN = 0.984, TA_LAST = 1.252;

struct TbmmAnyPlan {
  int tn, tm, gn, gm, nb;      // tiles per wavefront, wavefronts per strip pair, batch elements per workgroup
  bool direct;                 // results leave from the registers
  int64_t strips_n, strips_m;  // per batch element
  int64_t groups, lds;         // workgroups, bytes of LDS
  double cost;
};

// A plan from its free choices, and an estimate of the launch; false where it does not fit.
inline bool plan_tbmm_any(int64_t B, int64_t N, int64_t M, int64_t K, const TbmmAnyTile& t, int gn, int gm, int nb, bool direct, int cus, TbmmAnyPlan* p) {
  p->tn = t.tn; p->tm = t.tm; p->gn = gn; p->gm = gm; p->nb = nb; p->direct = direct;
  const int64_t sn = 16 * t.tn * gn, sm = 16 * t.tm * gm;
  p->strips_n = ceil_div(N, sn);
  p->strips_m = ceil_div(M, sm);
  const int64_t strips = p->strips_n * p->strips_m, rows = std::min(sn, N), cols = std::min(sm, M);
  if (strips >= ((int64_t)1 << 31) / B) return false;  // 32-bit numbers of workgroups
  const int64_t x = nb * rows * K, y = nb * cols * K, z = nb * rows * cols;
  // a multiple of 4: rows of 16 pieces that the kernel permutes
  const int64_t stage = K % 4 == 0 ? (ceil_div(x, 64) + ceil_div(y, 64)) * 256 : (ceil_div(x, 4) + ceil_div(y, 4)) * 16;
  p->lds = std::max<int64_t>(stage, direct ? 0 : (z + 6) / 4 * 16);
  if (p->lds > TA_MAX_LDS) return false;
  p->groups = strips == 1 ? ceil_div(B, nb) : B * strips;

  // Clocks: what the wavefronts of the fullest compute unit issue (MFMAs, conversions, results), its rounds of workgroups
  // as chains (launch, loads, MFMAs, results), and the bytes; the largest of the three counts most.
  const int steps = (int)ceil_div(K, 4), w = gn * gm * nb, mfma = t.tn * t.tm * steps, reads = (t.tn + t.tm) * steps;
  const double per_cu = (double)p->groups / cus, fullest = (double)ceil_div(p->groups, cus);
  const double resident = (double)std::max<int64_t>(1, std::min<int64_t>({TA_MAX_LDS / p->lds, (int64_t)(4 * t.waves / w), 16}));
  const double issue = (64.0 * mfma + TA_CVT * reads + TA_WAVE + 4 * t.tn * t.tm * (direct ? TA_OUT_DIRECT : TA_OUT_LDS)) * (w / 4.0 + TA_UNEVEN * ((w + 3) / 4 - w / 4.0));
  const double chain = TA_LATENCY + 4.0 * (x + y) / w / 64 * TA_LOAD + (direct ? 0 : TA_LAYOUT) + (64 + TA_MFMA_CHAIN) * mfma + TA_CVT * reads;
  const double turns = fullest / resident;
  const double lat = chain * (turns <= 1 ? 1 : turns + TA_LAST * (ceil_div((int64_t)fullest, (int64_t)resident) - turns));
  const double thr = issue * (fullest <= 1 ? 1 : per_cu + TA_LAST * (fullest - per_cu));
  const double mem = per_cu * 4 * (x + y + z) / TA_BW * (direct ? TA_BW_DIRECT : 1);
  p->cost = lat * lat * lat + thr * thr * thr + mem * mem * mem;
  return true;
}

// The plan of a batch; false where nothing fits LDS.
//   * Results go through LDS where there are many of them (more than 1.5 million) and the reduction is short (K < 64): full
//     lines for stores that matter, against two more barriers.
//   * Several batch elements per workgroup only up to 4 wavefronts; a single wavefront only where it does a whole element.
//   * Strips of equal numbers of wavefronts, but for one in the last.
inline bool choose_tbmm_any(int64_t B, int64_t N, int64_t M, int64_t K, int cus, TbmmAnyPlan* best) {
  const bool direct = !(B * N * M > 1500000 && K < 64);
  const int rn = (int)std::min<int64_t>(1 << 20, ceil_div(N, 16)), rm = (int)std::min<int64_t>(1 << 20, ceil_div(M, 16));
  TbmmAnyPlan pl{};
  bool any = false;
  auto consider = [&](const TbmmAnyTile& t, int gn, int gm, int nb) {
    if (plan_tbmm_any(B, N, M, K, t, gn, gm, nb, direct, cus, &pl) && (!any || pl.cost < best->cost)) {
      *best = pl;
      any = true;
    }
  };
  auto even = [](int tiles, int g) { return (tiles + g - 1) / g * g - tiles <= 1; };
  for (const TbmmAnyTile& t : TA_TILES) {
    if (t.tn > rn || t.tm > rm) continue;
    const int un = (rn + t.tn - 1) / t.tn, um = (rm + t.tm - 1) / t.tm;  // wavefronts for the whole element
    for (int gn = 1; gn <= std::min(un, TA_MAX_WAVES); gn++) {
      if (!even(un, gn)) continue;
      for (int gm = 1; gm <= std::min(um, TA_MAX_WAVES / gn); gm++) {
        if (!even(um, gm)) continue;
        const bool whole = gn == un && gm == um;
        if (gn * gm == 1 && !whole) continue;
        consider(t, gn, gm, 1);
        if (whole)
          for (int nb = 2; nb * gn * gm <= 4 && nb <= B; nb++) consider(t, gn, gm, nb);
      }
    }
  }
  return any;
}

}  // namespace tc355
