// Which launch of kron_tile.hpp a layer takes: the order of the two contractions, blocks of rows, batch elements per stage,
// wavefronts per tile, what is widened in LDS.  Plain C++: a test compiles it for the host and asks what its shapes take.
#pragma once
#include <algorithm>
#include <cstdint>

#include "tc355_host.hpp"

namespace tc355 {

constexpr int KT_WAVES = 8;
constexpr int KT_WAVE = 64;  // lanes
constexpr int KT_THREADS = KT_WAVES * KT_WAVE;

struct KronTilePlan {  // (the extents of a plan with `second` are exchanged: I and J, K and L)
  int64_t nb, lsp, itb, iblocks, jblocks, tj, k4, ls, ls1, ls2, xs, lds, groups, occ;
  bool wide, second;
  double cost;
};

// A plan from its free choices, and an estimate of the launch in clocks; false where it does not fit LDS.
inline bool plan_kron_tile(int64_t B, int64_t I, int64_t K, int64_t J, int64_t L, int64_t iblocks, int64_t nb, int64_t lsp, bool wide, bool second, int cus,
                           KronTilePlan* p) {
  const int64_t size = wide ? 8 : 4, ltiles = ceil_div(L, 16);
  p->nb = nb; p->lsp = lsp; p->wide = wide; p->second = second;
  p->itb = ceil_div(ceil_div(I, 16), iblocks);
  p->iblocks = ceil_div(ceil_div(I, 16), p->itb);
  p->jblocks = ceil_div(ceil_div(J, 16), 8);
  p->tj = ceil_div(ceil_div(J, 16), p->jblocks);
  if (p->iblocks * p->jblocks > 65535 || p->itb > 8) return false;
  p->k4 = ceil_div(K, 4) * 4;
  // Bank spread of the operand reads: 4 k rows (columns l in the second order) and 16 neighbours of the other index at a time.
  auto up = [](int64_t n, int64_t rem, int64_t mod) { return n + ((rem - n) % mod + mod) % mod; };
  p->ls = !second ? up(L, 4, 8) : wide ? up(p->k4, 2, 4) : up(p->k4, 4, 8);
  p->ls1 = second && wide ? up(p->k4, 2, 4) : up(p->k4, 4, 8);
  p->ls2 = wide ? up(ceil_div(L, 4) * 4, 2, 4) : up(ceil_div(L, 4) * 4, 4, 8);
  const int64_t xrows = second ? L : p->k4;
  if (prod_reaches({nb, xrows, p->ls}, 1 << 16)) return false;
  const int64_t x = nb * xrows * p->ls + 16;  // (the last row is read up to 15 elements past its end)
  const int64_t sums = nb * p->itb * (lsp - 1) * p->tj * 4 * KT_WAVE * 8 / size;
  p->xs = ceil_div(std::max(x, sums), 16) * 16;
  p->lds = (p->xs + 16 * p->tj * p->ls2 + std::min<int64_t>(16 * p->itb, I) * p->ls1 + 16) * size;  // (operands are read up to 7 elements ahead)
  if (p->lds > 160 * 1024) return false;
  p->groups = ceil_div(B, nb);
  p->occ = std::max<int64_t>(1, std::min<int64_t>(p->tj <= 4 ? 2 : 1, 160 * 1024 / (p->lds + 512)));
  // What a launch costs in clocks, as far as the choices change it: MFMAs (74 clocks each with what surrounds them, 79 where
  // operands are widened at the read), staging, the exchange of partial sums.  A wavefront's chain is two tiles' time
  // while the other half of the workgroup shares its SIMD; `occ` workgroups cover part of each other's staging.  The
  // constants are fitted to the measured times of 45 shapes at every choice of (iblocks, nb, lsp, wide): the plan taken
  // is on average 0.3 % from the best one, 2.4 % at worst.
  const int64_t blocks = p->iblocks * p->jblocks, jobs = nb * p->itb * lsp, per_cu = ceil_div(p->groups * blocks, cus);
  const double tile = (double)ceil_div(ltiles, lsp) * (p->k4 / 4 + 4 * p->tj) * (wide ? 74.0 : 79.0) + 355;
  const double stage = 2500 + (double)nb * K * L / KT_THREADS * 130 + (lsp > 1 ? 107.0 * lsp * p->tj : 0.0);
  const int64_t share = std::min(p->occ, per_cu), rest = jobs % KT_WAVES;
  const double chain = (jobs / KT_WAVES * 2 + (rest > 4 ? 2 : rest > 0 ? 1 : 0)) * tile + stage;
  p->cost = (double)(std::min<int64_t>(16 * p->itb, I) * K + 16 * p->tj * L) / KT_THREADS * 145 +
            (double)ceil_div(per_cu, share) * std::max(chain, share * (std::max(jobs / 4.0, 1.0) * tile + 0.72 * stage));
  return true;
}

// The best plan for one order of the two contractions (`second`: the extents come exchanged).
// More blocks of rows than needed only until one fits and while there are fewer than two workgroups per compute unit, more
// batch elements per stage only while there is a workgroup for half of them and they fit.  (At most 46 plans, 11 on average,
// over 200,000 random layers.)
inline bool best_kron_plan(int64_t B, int64_t I, int64_t K, int64_t J, int64_t L, bool second, int cus, KronTilePlan* best, bool any) {
  KronTilePlan pl{};
  const int64_t tiles_i = ceil_div(I, 16), least = ceil_div(tiles_i, 8), jblocks = ceil_div(ceil_div(J, 16), 8);
  bool here = false;
  for (int64_t itb = ceil_div(tiles_i, least); itb >= 1; itb--) {
    const int64_t iblocks = ceil_div(tiles_i, itb);
    if (here && (iblocks >= least + 8 || B * (iblocks - 1) * jblocks >= 2 * cus)) break;
    if (ceil_div(tiles_i, iblocks) != itb) continue;  // (the same blocks as with fewer tiles each)
    bool fits = true;
    for (int64_t nb = 1; fits && nb <= 8 && (nb == 1 || (nb <= B && ceil_div(B, nb) * iblocks * jblocks >= cus / 2)); nb++) {
      fits = false;
      for (int64_t lsp = 1; lsp <= 8 && (lsp == 1 || (nb * itb * lsp <= KT_WAVES && lsp <= ceil_div(L, 16))); lsp *= 2)
        for (int wide = 1; wide >= 0; wide--)
          if (plan_kron_tile(B, I, K, J, L, iblocks, nb, lsp, wide, second, cus, &pl)) {
            fits = here = true;
            if (!any || pl.cost < best->cost) { *best = pl; any = true; }
          }
    }
  }
  return any;
}

// The plan of a layer; false where no block of 16 rows, of columns and one batch element fit LDS.
inline bool choose_kron_tile(int64_t B, int64_t I, int64_t K, int64_t J, int64_t L, int cus, KronTilePlan* best) {
  if (cus <= 0 || K < 2 || L < 2 || K > 40000 || L > 40000) return false;
  bool any = best_kron_plan(B, I, K, J, L, false, cus, best, false);
  // The other order of the contractions where the estimate is 10 % lower: at 700 layers measured both ways no layer was more
  // than 3 % slower than in the first order with that margin (24 without it), for 0.1 % of the gain.
  KronTilePlan other{};
  if (best_kron_plan(B, J, L, I, K, true, cus, &other, false) && (!any || 1.1 * other.cost < best->cost)) {
    *best = other;
    any = true;
  }
  return any;
}

// Workgroups that walk over the stages of each block of the result.
inline int64_t kron_tile_workgroups(const KronTilePlan& p, int cus) {
  return std::min<int64_t>(p.groups, std::max<int64_t>(1, p.occ * cus / (p.iblocks * p.jblocks)));
}

}  // namespace tc355
