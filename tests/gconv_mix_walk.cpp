// Walks every launch of gconv_mix.hpp on the host, with the plan and the index arithmetic that the kernel itself uses:
// every workgroup's stages in order, every thread's units.  walk() returns the number of faults of a shape (staged elements
// that are wrong, missing, or read from outside the input), -1 where the kernel does not take the shape; *plan gets the
// numbers a test wants to know.
#include <cstdio>
#include <vector>

#include "gconv_mix_plan.hpp"

using namespace tc355;

extern "C" int64_t walk(int N, int G, int C, int F, int H, int W, int KH, int KW, int cus, int* plan) {
  constexpr int T = 256, NU = 4;
  GconvMixArgs p{};
  p.N = N; p.G = G; p.C = C; p.F = F; p.H = H; p.W = W; p.KH = KH; p.KW = KW; p.OH = H - KH + 1; p.OW = W - KW + 1;
  GconvMixPlan pl{};
  if (!choose_gconv_mix(p, cus, &pl)) return -1;
  const unsigned grid = gconv_mix_grid(p, pl);
  const int64_t total = (int64_t)N * G * C * H * W;
  const int seg = p.rows * W;
  plan[0] = p.imgs; plan[1] = (C + p.cc - 1) / p.cc; plan[2] = p.jobs; plan[3] = (int)grid; plan[4] = p.pblocks; plan[5] = 0;
  int64_t faults = 0, stages = 0;
  std::vector<int64_t> lds;                        // element of I that each LDS slot of the band holds
  std::vector<GconvMixUnits<NU>> threads(T);
  for (unsigned wg = 0; wg < grid; wg++) {
    int job_end;
    GconvMixStage s = gm_first(p, wg, grid, job_end);
    for (auto& t : threads) t = GconvMixUnits<NU>();
    int last_units = -1, last_imgs = -1;
    for (; s.job < job_end; gm_advance(p, s)) {
      stages++;
      const int units = gm_units(p, s), imgs = gm_images(p, s), cc = gm_channels(p, s);
      plan[5] += units == last_units && imgs != last_imgs;  // stages of as many units as the one before, laid out otherwise
      last_units = units; last_imgs = imgs;
      const int64_t origin = gm_origin(p, s);
      lds.assign((size_t)p.cc * p.ps, -1);
      auto put = [&](int64_t go, int lo) {
        for (int e = 0; e < 4; e++) {
          const int64_t at = origin + go / 4 + e;
          if (go % 4 != 0 || at < 0 || at >= total || lo < 0 || lo + e >= p.cc * p.ps) faults++;
          else lds[lo + e] = at;
        }
      };
      for (int tid = 0; tid < T; tid++) {
        threads[tid].decode(p, s, tid, T);
        for (int j = 0; j < NU; j++)
          if (j * T < units) put(threads[tid].goff[j], threads[tid].loff[j]);
          else if (origin + threads[tid].goff[j] / 4 + 3 >= total) faults++;  // (loaded all the same)
        for (int u = tid + NU * T; u < units; u += T) {
          unsigned go;
          int lo;
          gm_place(p, u, cc, go, lo);
          put(go, lo);
        }
      }
      // what the contraction reads: every channel's rows of every image
      const int h0 = gm_first_row(p, s), g = s.gf / p.fblocks;
      for (int img = 0; img < imgs; img++)
        for (int c = 0; c < cc; c++)
          for (int i = 0; i < seg; i++) {
            const int64_t want = ((((int64_t)(s.ib * p.imgs + img) * G + g) * C + s.c0 + c) * H + h0) * W + i;
            if (lds[(size_t)c * p.ps + img * seg + i] != want) faults++;
          }
      // the block's pixels lie inside the staged rows
      if (p.imgs == 1) {
        const int last = std::min(p.px * (s.pb + 1), p.OH * p.OW) - 1;
        if (p.px * s.pb / p.OW < h0 || last / p.OW + KH > h0 + p.rows) faults++;
      }
    }
  }
  if (stages != (int64_t)p.jobs * plan[1]) faults++;
  return faults;
}
