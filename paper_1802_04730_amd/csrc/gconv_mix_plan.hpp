// What a launch of gconv_mix.hpp is made of: the host's plan, and the index arithmetic of a stage (which channels and
// images it stages, from where, to where in LDS).  Plain C++: the kernel compiles the second part for the GPU, and a test
// compiles all of it for the host and walks whole launches, element by element.
#pragma once
#include <algorithm>
#include <cstdint>

#include "tc355_host.hpp"

#ifdef __HIPCC__
#define TC355_HD __host__ __device__ __forceinline__
#else
#define TC355_HD inline
#endif

namespace tc355 {

struct GconvMixArgs {
  const float* I;     // [N][G][C][H][W]
  const float* W1;    // [G][F][C][KH][KW]
  const float* bias;  // [G*F] or nullptr
  float* O;           // [N][G][F][OH][OW]
  int N, G, C, F, H, W, KH, KW, OH, OW;
  int fblocks;         // filter blocks per group
  int fb;              // filters per block (at most 16*FT + 4*FQ)
  int imgs;            // images per job (1 unless an image has few pixels)
  int iblocks;         // ceil(N / imgs)
  int pblocks;         // pixel blocks per image (1 if imgs > 1)
  int px;              // pixels per block, a multiple of 16, at most 64*TP
  int jobs;            // G * fblocks * iblocks * pblocks
  int cus;             // compute units of the device
  int cc;              // channels per chunk
  int rows;            // input rows staged per image (at most H)
  int ps;              // LDS plane stride in doubles, = 16 (mod 32)
  int upc;             // 16-byte units per (channel, image): ceil(rows * W / 4)
  unsigned upc_magic, ow_magic, kk_magic, kw_magic, npix_magic;  // for div_magic; npix's is 0 (quotient 0) if imgs = 1
};

// ---- stages: a stage is one chunk of channels of one job -----------------------------------------------------------
struct GconvMixStage {
  int job, pb, ib, gf, c0;
};

TC355_HD int gm_min(int a, int b) { return a < b ? a : b; }

// u / d for magic = ceil(2^31 / d), while 2 u d < 2^32
TC355_HD int div_magic(int u, unsigned magic) { return (int)((unsigned long long)(2u * (unsigned)u) * magic >> 32); }

// The run of jobs of workgroup `wg` of `grid`: its first stage, and the job behind its last one.  Workgroups w, w + cus,
// w + 2 cus, ... share a compute unit: they take neighbouring runs, so that the units' sums differ by one job at most
// (in launch order, runs of 3 and 4 jobs fell on units of 9 and of 12).
TC355_HD GconvMixStage gm_first(const GconvMixArgs& p, unsigned wg, unsigned grid, int& job_end) {
  const unsigned per_cu = grid / (unsigned)p.cus;
  const unsigned slot = per_cu * (unsigned)p.cus == grid ? wg % (unsigned)p.cus * per_cu + wg / (unsigned)p.cus : wg;
  GconvMixStage s;
  s.job = (int)((int64_t)p.jobs * slot / grid);
  job_end = (int)((int64_t)p.jobs * (slot + 1) / grid);
  const int r = s.job / p.pblocks;
  s.pb = s.job - r * p.pblocks;
  s.gf = r / p.iblocks;
  s.ib = r - s.gf * p.iblocks;
  s.c0 = 0;
  return s;
}

TC355_HD void gm_advance(const GconvMixArgs& p, GconvMixStage& s) {
  s.c0 += p.cc;
  if (s.c0 < p.C) return;
  s.c0 = 0;
  s.job++;
  if (++s.pb < p.pblocks) return;
  s.pb = 0;
  if (++s.ib < p.iblocks) return;
  s.ib = 0;
  s.gf++;
}

TC355_HD int gm_images(const GconvMixArgs& p, const GconvMixStage& s) { return gm_min(p.imgs, p.N - s.ib * p.imgs); }
TC355_HD int gm_channels(const GconvMixArgs& p, const GconvMixStage& s) { return gm_min(p.cc, p.C - s.c0); }
TC355_HD int gm_units(const GconvMixArgs& p, const GconvMixStage& s) { return gm_images(p, s) * gm_channels(p, s) * p.upc; }

// first input row of a job's band: the last block's band is moved up to end with the image, so all have `rows` rows
TC355_HD int gm_first_row(const GconvMixArgs& p, const GconvMixStage& s) {
  return gm_min(div_magic(s.pb * p.px, p.ow_magic), p.H - p.rows);
}

// the element of I that a stage's offsets count from
TC355_HD int64_t gm_origin(const GconvMixArgs& p, const GconvMixStage& s) {
  const int g = s.gf / p.fblocks;
  return (((int64_t)s.ib * p.imgs * p.G + g) * p.C + s.c0) * (unsigned)(p.H * p.W) + (int64_t)gm_first_row(p, s) * p.W;
}

// Unit u of a stage with cc channels per image: its byte offset in I from the stage's origin, and its LDS offset in doubles.
// Channels x images are contiguous runs of rows * W input elements, cut into units of 4; the last unit of a run overlaps its
// neighbour instead of passing the end.
TC355_HD void gm_place(const GconvMixArgs& p, int u, int cc, unsigned& go, int& lo) {
  const int seg = p.rows * p.W, sg = div_magic(u, p.upc_magic), i = gm_min(4 * (u - sg * p.upc), seg - 4);
  const unsigned plane = (unsigned)(p.H * p.W);
  int img = 0, c = sg;
  if (p.imgs > 1) { img = sg / cc; c = sg - img * cc; }
  go = 4u * ((unsigned)img * (unsigned)(p.G * p.C) * plane + (unsigned)c * plane + (unsigned)i);
  lo = c * p.ps + img * seg + i;
}

// The first NU units of a thread (unit tid + j * threads through register j), worked out again only where the stage has
// another number of images or of channels.  (Their product does not tell: 2 images of 6 channels are as many units as 1 of 12.)
template <int NU>
struct GconvMixUnits {
  unsigned goff[NU];
  int loff[NU];
  int layout = 0;  // images and channels that goff and loff stand for

  TC355_HD void decode(const GconvMixArgs& p, const GconvMixStage& s, int tid, int threads) {
    const int imgs = gm_images(p, s), cc = gm_channels(p, s), units = imgs * cc * p.upc;
    if (layout == (imgs << 16 | cc)) return;
    layout = imgs << 16 | cc;
#ifdef __HIPCC__
#pragma unroll
#endif
    for (int j = 0; j < NU; j++) gm_place(p, gm_min(tid + j * threads, units - 1), cc, goff[j], loff[j]);
  }
};

// ---- the host's plan -----------------------------------------------------------------------------------------------
struct GconvMixPlan {
  int tp, imgs, pblocks, px, rows, ps, cc, occ;
  int64_t jobs, lds;
  double cost;
};

// Blocks of 64*tp output pixels at `occ` workgroups per compute unit: what they stage, and an estimate of the launch in
// clocks.  Returns false if the channels of a chunk would not fit.
inline bool plan_gconv_mix(const GconvMixArgs& g, int tp, int occ, int fblocks, int rec, int cus, GconvMixPlan* pl) {
  const int64_t npix = (int64_t)g.OH * g.OW, KK = (int64_t)g.KH * g.KW;
  pl->tp = tp;
  pl->occ = occ;
  int64_t tiles;  // of an image, or of the images of a job
  if (npix * 2 <= 64 * tp) {
    pl->imgs = (int)std::min<int64_t>(g.N, 64 * tp / npix);
    if (prod_reaches({pl->imgs, g.G, g.C, g.H, g.W}, 1ll << 29) || prod_reaches({pl->imgs, g.G, g.F, g.OH, g.OW}, 1ll << 29)) return false;  // 32-bit byte offsets between a job's images
    pl->pblocks = 1;
    tiles = ceil_div(pl->imgs * npix, 16);
    pl->px = (int)tiles * 16;
    pl->rows = g.H;
  } else {
    pl->imgs = 1;
    tiles = ceil_div(npix, 16);
    pl->px = 16 * (int)ceil_div(tiles, ceil_div(tiles, 4 * tp));  // equal blocks
    pl->pblocks = (int)ceil_div(npix, pl->px);
    pl->rows = (int)(std::min<int64_t>(g.OH, (pl->px - 2) / g.OW + 2) + g.KH - 1);
  }
  const int64_t len = (int64_t)pl->imgs * pl->rows * g.W;
  if (len > 16384) return false;
  pl->ps = (int)((len + 15) / 32 * 32 + 16);
  const int64_t per_c = pl->ps * 8 + (KK * rec * 8 + 3) / 4 + KK * 4, fixed = rec * 8 + 16 + 48;  // (a chunk's last step may be partial; the table is read ahead)
  const int64_t most = (160 * 1024 / occ - 512 - fixed) / per_c;
  if (most < 1) return false;
  int64_t chunks = ceil_div(g.C, most), cc = ceil_div(g.C, chunks);
  if (chunks > 1 && most >= 4) {  // equal chunks of a multiple of 4 channels (the layout without padded slots)
    cc = std::min(most / 4 * 4, ceil_div(cc, 4) * 4);
    chunks = ceil_div(g.C, cc);
  }
  if (std::min<int64_t>(cc, g.C - (chunks - 1) * cc) * KK < 4 || cc * KK > 4096) return false;  // filters are staged in units of 4 taps
  pl->cc = (int)cc;
  const int64_t steps = ceil_div(cc * KK, 4);
  pl->lds = cc * pl->ps * 8 + steps * rec * 8 + steps * 16 + 48;
  pl->jobs = (int64_t)g.G * fblocks * ceil_div(g.N, pl->imgs) * pl->pblocks;
  // A stage (one chunk of one job) in clocks of a SIMD: its MFMA steps (between the average and the largest share of a
  // wavefront), and what surrounds them (staging the band, and the filters where they change with every stage), about
  // half of it vector instructions, which no MFMA overlaps.  `occ` workgroups cover each other's waits but not each
  // other's instructions; alone, a step is never shorter than the LDS reads of the next one.  (The constants are fitted
  // to measured times of 16 shapes at every (tp, occ): the choice is on average 2.5 % from the best one.)
  const double turns = 0.5 * ((double)tiles / (4 * pl->pblocks) + tp), step = turns * rec + 8;
  const double around = 500 + (double)cc * len / 8 + (chunks > 1 ? 3000 + 0.5 * steps * rec : 0.0);
  const int64_t per_cu = ceil_div(pl->jobs, cus), share = std::min<int64_t>(occ, per_cu);
  pl->cost = (double)per_cu / share * chunks * std::max(share * (steps * step + 0.5 * around), steps * std::max(step, 320.0) + around);
  return pl->jobs < (1ll << 31);
}

// Fills in the plan of the shape that a's extents state, and returns it in *best; false where the kernel does not take it.
inline bool choose_gconv_mix(GconvMixArgs& a, int cus, GconvMixPlan* best) {
  if (cus <= 0 || (int64_t)a.KH * a.W < 4 || (int64_t)a.C * a.KH * a.KW < 4) return false;  // staged in units of 4 elements
  if (prod_reaches({a.C, a.H, a.W}, 1ll << 29) || prod_reaches({a.F, a.C, a.KH, a.KW}, 1ll << 29) || prod_reaches({a.F, a.OH, a.OW}, 1ll << 29))
    return false;  // 32-bit byte offsets
  a.fblocks = (int)ceil_div(a.F, 32);
  a.fb = (int)ceil_div(ceil_div(a.F, a.fblocks), 4) * 4;
  const int rec = a.fb / 16 * 64 + a.fb % 16 / 4 * 16;
  GconvMixPlan pl{};
  bool any = false;
  for (int occ = 4; occ >= 1; occ--)
    for (int tp = 4; tp >= 1; tp--)
      if (plan_gconv_mix(a, tp, occ, a.fblocks, rec, cus, &pl) && (!any || pl.cost < best->cost)) { *best = pl; any = true; }
  if (!any) return false;
  a.px = best->px; a.imgs = best->imgs; a.iblocks = (int)ceil_div(a.N, best->imgs); a.pblocks = best->pblocks;
  a.jobs = (int)best->jobs; a.cus = cus;
  a.cc = best->cc; a.rows = best->rows; a.ps = best->ps;
  a.upc = (int)ceil_div((int64_t)best->rows * a.W, 4);
  if ((int64_t)a.OH * a.OW >= (1ll << 31) / a.OW) return false;  // divisions by multiplication: 2 * dividend * divisor < 2^32
  auto magic = [](int64_t d) { return (unsigned)(((1ll << 31) + d - 1) / d); };
  a.upc_magic = magic(a.upc); a.ow_magic = magic(a.OW); a.kk_magic = magic((int64_t)a.KH * a.KW); a.kw_magic = magic(a.KW);
  a.npix_magic = best->imgs > 1 ? magic((int64_t)a.OH * a.OW) : 0;
  return true;
}

// workgroups of a launch: persistent, no more than jobs
inline unsigned gconv_mix_grid(const GconvMixArgs& a, const GconvMixPlan& pl) { return (unsigned)std::min<int64_t>(pl.jobs, (int64_t)pl.occ * a.cus); }

}  // namespace tc355
