// Grouped convolution (Section 7, listing gconv) for channel counts, filter counts, filter sizes and images that fit
// no compile-time kernel:
//
//   O(n,g,o,h,w) = sum_{i,kh,kw} I(n,g,i,h+kh,w+kw) * W1(g,o,i,kh,kw) + bias(g*F+o)
//
// Two MFMA shapes share one B operand (k slot q, pixel r16), so a block of filters is cut into FT tiles of 16
// (v_mfma_f64_16x16x4_f64, 64 clocks) and FQ quads of 4 (v_mfma_f64_4x4x4_4b_f64, 16 clocks; layout in
// gconv_quad.hpp): 20 filters are one tile and one quad, 80 clocks per 16 pixels and 4 taps, where tiles alone would
// spend 128.  The padding is at most 3 filters.
//
// A job is one group, one block of filters, and up to 64*TP consecutive output pixels (of one image, or of several whole
// small images).  The input rows that these pixels touch are widened to fp64 and staged in LDS as [channel][pixel],
// the filters as A operands in the order in which the steps read them, and a table holds the LDS offset of each tap:
// a step is one table read, FT + FQ reads of A, and per pixel tile one add, one read of B and FT + FQ MFMAs.  Long
// reductions are walked in chunks of channels that fit LDS.  Persistent workgroups take contiguous runs of jobs, groups
// outermost, so that filters and table are staged again only where the group (or the chunk) changes; the next band
// travels in registers while the present one is contracted, and a job's outputs leave after the next band is parked.
// All loads are 16 bytes of 4-byte aligned elements: no size is rounded up in memory.
//
// Bound by the fp64 matrix pipe and by the vector instructions that do not overlap it (counters at
// (N,G,C,F,H,W) = (16,24,12,20,33,45), 3 x 3: pipe busy 54 % of the cycles, vector instructions 16 %, LDS bank conflicts 12 %).
// Measured there 53 us = 41 TFLOP/s, 25 of it without the MFMAs, where gconv_wave.hpp (operands gathered from global memory, 32 filters' worth of
// MFMAs) takes 200 us; (2,22,23,31,27,48) 5 x 5: 54 us against 132, (7,32,8,8,58,58) 3 x 3: 28 against 99, a small
// (2,1,7,4,17,20) 3 x 2: 4.2 against 12.2.  Deals of tiles and workgroups: equal blocks of pixels with the longer shares
// rotating over the wavefronts instead of 64*TP pixels each: (13,6,40,40,20,28) 35 us against 41; neighbouring runs on
// one compute unit instead of launch order: 54 against 58 us at the first shape (runs of 3 and 4 jobs).
#pragma once
#include <type_traits>

#include "gconv_mix_plan.hpp"
#include "tc355_device.hpp"

namespace tc355 {

template <int FT, int FQ, int TP>
__global__ __launch_bounds__(WG_THREADS, 2) void gconv_mix_kernel(GconvMixArgs p) {
  constexpr int REC = FT * 64 + FQ * 16;  // doubles of A operands per step
  constexpr int NU = 4;                   // units of the band that a thread holds in registers ahead of their use
  constexpr int FTA = FT > 0 ? FT : 1, FQA = FQ > 0 ? FQ : 1;
  extern __shared__ __attribute__((aligned(16))) double gm_lds[];
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int r16 = lane & 15, q = lane >> 4;
  const int KK = p.KH * p.KW, W = p.W, OW = p.OW, PS = p.ps;
  const int npix = p.OH * OW;
  const int seg = p.rows * W;
  double* band = gm_lds;                                                // [cc][PS], images of a plane `seg` apart
  double* fil = gm_lds + p.cc * PS;                                     // [step][REC]
  int* tab = reinterpret_cast<int*>(fil + ((p.cc * KK + 3) >> 2) * REC);  // [step][4]: byte offset of k slot q's tap; 12 spare entries

  // ---- stages (job, chunk of channels), in order
  int job_end;
  GconvMixStage cur = gm_first(p, blockIdx.x, gridDim.x, job_end);
  if (cur.job >= job_end) return;  // (the host launches no more workgroups than jobs)

  // ---- band: units of 4 elements (gm_place); the first NU of a thread are fetched a stage ahead
  GconvMixUnits<NU> at;
  f4_any pre[NU];
  auto band_of = [&](const GconvMixStage& s) { return reinterpret_cast<const char*>(p.I + gm_origin(p, s)); };
  auto fetch = [&](const GconvMixStage& s) {
    at.decode(p, s, tid, WG_THREADS);
    const char* in = band_of(s);
#pragma unroll
    for (int j = 0; j < NU; j++) pre[j] = *reinterpret_cast<const f4_any*>(in + at.goff[j]);
  };
  auto put = [&](int lo, const f4_any& v) {
    double* o = band + lo;
    o[0] = (double)v[0]; o[1] = (double)v[1]; o[2] = (double)v[2]; o[3] = (double)v[3];
  };
  auto park = [&](const GconvMixStage& s) {
    const int units = gm_units(p, s);
#pragma unroll
    for (int j = 0; j < NU; j++)
      if (j * WG_THREADS < units) put(at.loff[j], pre[j]);
    if (units > NU * WG_THREADS) {  // a band of more than 4096 elements: the rest is not fetched ahead
      const char* in = band_of(s);
      for (int u0 = tid + NU * WG_THREADS; u0 < units; u0 += 4 * WG_THREADS) {
        f4_any v[4];
        int lo[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
          unsigned go;
          gm_place(p, min(u0 + j * WG_THREADS, units - 1), gm_channels(p, s), go, lo[j]);
          v[j] = *reinterpret_cast<const f4_any*>(in + go);
        }
#pragma unroll
        for (int j = 0; j < 4; j++) put(lo[j], v[j]);
      }
    }
  };
  // ---- filters of (group, block, chunk) as A operands, and the table of the taps' LDS offsets.  k slot q of step s is
  // channel 4*c4 + q of one tap (s = tap * cc/4 + c4) if the chunk has a multiple of 4 channels, else tap 4s + q in
  // W1's order.
  int staged_gf = -1, staged_c0 = -1;
  d4 bz[FTA];
  double bzq[FQA];
  auto filters = [&](const GconvMixStage& st) {
    const int g = st.gf / p.fblocks, f0 = (st.gf - g * p.fblocks) * p.fb, nf = min(p.fb, p.F - f0);
    const int cc = min(p.cc, p.C - st.c0), kc = cc * KK, steps = (kc + 3) >> 2;
    const bool cminor = (cc & 3) == 0;
    const int cq = cc >> 2;
    // a filter's taps of this chunk are contiguous in W1: units of 4, the last one of a filter overlapping its neighbour
    const char* wg = reinterpret_cast<const char*>(p.W1 + ((int64_t)(g * p.F + f0) * p.C + st.c0) * KK);
    const int units = nf * steps;
    const unsigned magic = (0x7fffffffu + (unsigned)steps) / (unsigned)steps;
    auto batch = [&](int u0, auto nb) {  // nb loads in flight per thread
      constexpr int NB = decltype(nb)::value;
      f4_any w[NB];
      int fk[NB];
#pragma unroll
      for (int j = 0; j < NB; j++) {
        const int u = min(u0 + j * WG_THREADS, units - 1);
        const int f = div_magic(u, magic), k = min(4 * (u - f * steps), kc - 4);
        w[j] = *reinterpret_cast<const f4_any*>(wg + 4u * (unsigned)(f * (p.C * KK) + k));
        fk[j] = f << 16 | k;
      }
      if (u0 == tid) {  // (while the first loads are in flight)
        for (int i = tid; i < 4 * steps; i += WG_THREADS) {
          int c, kk;
          if (cminor) {
            kk = (i >> 2) / cq;
            c = 4 * ((i >> 2) - kk * cq) + (i & 3);
          } else {
            const int k = min(i, kc - 1);
            c = div_magic(k, p.kk_magic);
            kk = k - c * KK;
          }
          const int kh = div_magic(kk, p.kw_magic);
          tab[i] = (c * PS + kh * W + (kk - kh * p.KW)) * 8;
        }
      }
#pragma unroll
      for (int j = 0; j < NB; j++) {
        const int f = fk[j] >> 16, k0 = fk[j] & 0xffff;
        const bool quad = FT == 0 || f >= 16 * FT;
        const int fp = quad ? FT * 64 + ((f - 16 * FT) >> 2) * 16 + (f & 3) : (f >> 4) * 64 + (f & 15), qs = quad ? 4 : 16;
        int c = div_magic(k0, p.kk_magic), kk = k0 - c * KK;
#pragma unroll
        for (int e = 0; e < 4; e++) {
          const int s = cminor ? kk * cq + (c >> 2) : (k0 + e) >> 2, kq = cminor ? c & 3 : (k0 + e) & 3;
          fil[s * REC + fp + kq * qs] = (double)w[j][e];
          if (++kk == KK) { kk = 0; c++; }
        }
      }
    };
    if (units <= WG_THREADS) batch(tid, std::integral_constant<int, 1>{});
    else
      for (int u0 = tid; u0 < units; u0 += 4 * WG_THREADS) batch(u0, std::integral_constant<int, 4>{});
    if (kc & 3) {  // k slots past the reduction: zero (in both operands, see below)
      for (int r = tid; r < REC; r += WG_THREADS) {
        const int kq = r < FT * 64 ? (r & 63) >> 4 : (r & 15) >> 2;
        if (kq >= (kc & 3)) fil[(steps - 1) * REC + r] = 0.0;
      }
    }
    if (staged_gf != st.gf) {
      if (p.bias) {
        const float* bp = p.bias + g * p.F + f0;
#pragma unroll
        for (int ft = 0; ft < FT; ft++)
#pragma unroll
          for (int v = 0; v < 4; v++) bz[ft][v] = (double)bp[min(16 * ft + d_row(q, v), nf - 1)];
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) bzq[fq] = (double)bp[min(16 * FT + 4 * fq + q, nf - 1)];
      } else {
#pragma unroll
        for (int ft = 0; ft < FT; ft++) bz[ft] = d4_zero();
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) bzq[fq] = 0.0;
      }
    }
    staged_gf = st.gf;
    staged_c0 = st.c0;
  };

  int base[TP];
  d4 acc[TP][FTA];
  double accq[TP][FQA];
  fetch(cur);
  filters(cur);
  park(cur);
  for (;;) {
    GconvMixStage nxt = cur;
    gm_advance(p, nxt);
    const bool more = nxt.job < job_end;
    if (more) fetch(nxt);  // in flight while this stage is contracted
    __syncthreads();

    const int P0 = cur.pb * p.px;
    const int npx = min(p.px, min(p.imgs, p.N - cur.ib * p.imgs) * npix - P0);  // pixels of this job
    // Its tiles are dealt to the wavefronts in turn, from another one with every job: where they do not divide by four,
    // the wavefronts (and with them the SIMDs of the unit) take the longer shares in turn.
    const int rank = (wave + cur.job + blockIdx.x / p.cus) & 3;
    const int tiles = (npx + 15) >> 4, cnt = (tiles + 3 - rank) >> 2;
    const int t0 = rank * (tiles >> 2) + min(rank, tiles & 3);  // this wavefront's tiles: t0 ... t0 + cnt - 1
    if (cur.c0 == 0) {
      const int h0 = gm_first_row(p, cur);
#pragma unroll
      for (int t = 0; t < TP; t++) {  // LDS byte offset of this lane's output pixel in each of its tiles
        int px = min((t0 + t) * 16 + r16, npx - 1) + P0;
        const int img = div_magic(px, p.npix_magic);
        px -= img * npix;
        const int h = div_magic(px, p.ow_magic);
        base[t] = (img * seg + (h - h0) * W + (px - h * OW)) * 8;
#pragma unroll
        for (int ft = 0; ft < FT; ft++) acc[t][ft] = bz[ft];
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) accq[t][fq] = bzq[fq];
      }
    }
    auto contract = [&](auto nt) {  // the first nt tiles
      constexpr int NT = decltype(nt)::value;
      const int kc = min(p.cc, p.C - cur.c0) * KK, steps = (kc + 3) >> 2;
      const char* bb = reinterpret_cast<const char*>(band);
      const double* fl = fil + lane;
      const double* fqp = fil + FT * 64 + 4 * q + (lane & 3);
      // two sets of operands in turn: the reads of step s + 1 are issued before the MFMAs of step s
      struct Ops { double a[FTA], aq[FQA], b[NT]; } x, y;
      auto load = [&](int s, int off, Ops& r) {
#pragma unroll
        for (int ft = 0; ft < FT; ft++) r.a[ft] = fl[s * REC + 64 * ft];
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) r.aq[fq] = fqp[s * REC + 16 * fq];
#pragma unroll
        for (int t = 0; t < NT; t++) r.b[t] = *reinterpret_cast<const double*>(bb + (base[t] + off));
      };
      auto mul = [&](const Ops& r) {
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; t++) {
#pragma unroll
          for (int ft = 0; ft < FT; ft++) acc[t][ft] = mfma_f64(r.a[ft], r.b[t], acc[t][ft]);
#pragma unroll
          for (int fq = 0; fq < FQ; fq++) accq[t][fq] = __builtin_amdgcn_mfma_f64_4x4x4f64(r.aq[fq], r.b[t], accq[t][fq], 0, 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
      };
      auto last = [&](Ops& r) {  // k slots past the reduction: zero in both operands (0 * Inf would be NaN)
        if (4 * (steps - 1) + q >= kc) {
#pragma unroll
          for (int t = 0; t < NT; t++) r.b[t] = 0.0;
        }
        mul(r);
      };
      const int* tq = tab + q;  // (read up to two steps ahead of the last one: spare entries, not used)
      int o0 = tq[0], o1 = tq[4];
      load(0, o0, x);
      int s = 0;
      for (; s + 2 < steps; s += 2) {
        load(s + 1, o1, y);
        o0 = tq[4 * s + 8];
        mul(x);
        load(s + 2, o0, x);
        o1 = tq[4 * s + 12];
        mul(y);
      }
      if (s + 1 < steps) {
        load(s + 1, o1, y);
        mul(x);
        last(y);
      } else {
        last(x);
      }
    };
    if (cnt >= TP) contract(std::integral_constant<int, TP>{});
    else if (TP > 2 && cnt == TP - 1) contract(std::integral_constant<int, TP - 1>{});
    else if (TP > 1 && cnt > 0) contract(std::integral_constant<int, TP / 2>{});
    __syncthreads();  // everybody has read this stage's band and filters
    if (more) {
      if (nxt.gf != staged_gf || nxt.c0 != staged_c0) filters(nxt);
      park(nxt);
    }
    if (cur.c0 + p.cc >= p.C) {  // the job's last chunk: its outputs
      const int g = cur.gf / p.fblocks, f0 = (cur.gf - g * p.fblocks) * p.fb, nf = min(p.fb, p.F - f0);
      char* op = reinterpret_cast<char*>(p.O + (((int64_t)cur.ib * p.imgs * p.G + g) * p.F + f0) * npix);
      const unsigned fs = 4u * (unsigned)npix;
      auto emit = [&](auto whole) {  // (every filter of the block exists: no per-filter choice)
#pragma unroll
        for (int t = 0; t < TP; t++) {
          const int pl = t < cnt ? (t0 + t) * 16 + r16 : npx;
          const unsigned o = 4u * (unsigned)(P0 + pl) + ((unsigned)q + (unsigned)(div_magic(pl, p.npix_magic) * (p.G * p.F - 1))) * fs;
          if (pl < npx) {
#pragma unroll
            for (int ft = 0; ft < FT; ft++)
#pragma unroll
              for (int v = 0; v < 4; v++)
                if (whole || 16 * ft + d_row(q, v) < nf)
                  *reinterpret_cast<float*>(op + (o + (unsigned)(16 * ft + 4 * v) * fs)) = (float)acc[t][ft][v];
#pragma unroll
            for (int fq = 0; fq < FQ; fq++)
              if (whole || 16 * FT + 4 * fq + q < nf)
                *reinterpret_cast<float*>(op + (o + (unsigned)(16 * FT + 4 * fq) * fs)) = (float)accq[t][fq];
          }
        }
      };
      if (nf == 16 * FT + 4 * FQ) emit(std::true_type{});
      else emit(std::false_type{});
    }
    if (!more) return;
    cur = nxt;
  }
}

}  // namespace tc355
