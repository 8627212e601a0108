// Strided convolution (Section 3, listing sconv2d) with few blocks of 64 filters x 32 pixels: the contraction of
// sconv_tile.hpp (rows = filters, columns = all output pixels of the batch, reduction = the taps in W's order), with its
// reduction split inside the workgroup.
//
// What bounds it: one image of 400 output pixels is 13 such blocks, on 256 compute units, and every one walks all C*KH*KW
// taps in chunks of 16 behind a barrier: (1,21,64,46,46) with 7 x 7 filters took 40 us, 64 times what the matrix core needs.
// Here a workgroup of 4 wavefronts owns (16 TF) filters x (16 TP) pixels and every wavefront all of them, for a quarter of
// every chunk of 64 taps, so there are 4 to 8 times as many workgroups and a quarter as many chunks.  A thread gathers
// taps tid/16 + 16 j of pixels tid%16 + 16 i; the taps' offsets from a pixel's first input element come from a table in LDS
// (built once: no carries, no divisions).  Filters travel 64 consecutive taps per wavefront and load.  Both are fetched two
// chunks ahead, widened once and staged in double-buffered fp64 LDS; taps past the end count as zeros in both operands.
// The four partial blocks are added through LDS in a fixed order, bias first.
// Measured: 40.8 -> 10.8 us for the layer above, (11,202,64,28,28) with 7 x 7 filters at stride 2 349 -> 106 us; larger blocks
// (16 x 32, 32 x 32: 17 and 23 us for the first layer) leave compute units idle.
#pragma once
#include "sconv_tile.hpp"

namespace tc355 {

constexpr int SS_KC = 64;
constexpr int SS_RSA = SS_KC + 2;  // filter rows: 2*RSA = 4 (mod 64) words

template <int TF, int TP>
struct SconvSplitGeom {
  static constexpr int RSB = 16 * TP + (TP % 2 ? 0 : 16);  // tap rows: = 16 (mod 32) doubles
  static constexpr int BUF = 16 * TF * SS_RSA + SS_KC * RSB;
  static constexpr int STAGES = 2 * BUF * 8;               // bytes; the table of tap offsets follows
  static_assert(TF * TP * 16 * WAVE <= 2 * BUF, "the partial sums fit the stages");
};

template <int TF, int TP>
__global__ __launch_bounds__(WG_THREADS, 2) void sconv_split_kernel(SconvArgs p) {
  using Gm = SconvSplitGeom<TF, TP>;
  extern __shared__ __attribute__((aligned(16))) double ss_lds[];
  unsigned* table = reinterpret_cast<unsigned*>(ss_lds + 2 * Gm::BUF);
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int r16 = lane & 15, q = lane >> 4;
  const int K = p.K, P = p.P, F = p.F, OHW = p.OH * p.OW;
  const int f0 = (int)(blockIdx.x % p.tiles_f) * 16 * TF, p0 = (int)(blockIdx.x / p.tiles_f) * 16 * TP;
  const int nck = (K + SS_KC - 1) / SS_KC;

  // the taps' byte offsets, in W's order (c, kh, kw); past the end any element of I (the value is dropped)
  {
    const int HW = p.H * p.W, KW = p.KW, KHW = p.KH * p.KW;
    for (int k = tid; k < nck * SS_KC; k += WG_THREADS) {
      const int c = k / KHW, t = k - c * KHW, kh = t / KW, kw = t - kh * KW;
      table[k] = k < K ? 4u * (unsigned)(c * HW + kh * p.W + kw) : 0u;
    }
  }
  const int b_p = tid & 15, b_k = tid >> 4;
  unsigned pixbase[TP];  // byte offset of the pixel's first input element
#pragma unroll
  for (int i = 0; i < TP; i++) {
    const int px = min(p0 + 16 * i + b_p, P - 1);  // pixels past the end repeat the last one (never stored)
    const int n = px / OHW, r = px - n * OHW, oh = r / p.OW, ow = r - oh * p.OW;
    pixbase[i] = 4u * (unsigned)((n * p.C * p.H + p.sh * oh) * p.W + p.sw * ow);
  }
  unsigned aoff[4 * TF];  // byte offsets of the filter rows wave + 4 i
#pragma unroll
  for (int i = 0; i < 4 * TF; i++) aoff[i] = (unsigned)min(f0 + wave + 4 * i, F - 1) * (unsigned)K * 4u;

  struct Regs {
    float a[4 * TF];
    float b[TP][4];
  };
  const char* I = reinterpret_cast<const char*>(p.I);
  const char* Wt = reinterpret_cast<const char*>(p.Wt);
  auto fetch = [&](Regs& r, int c) {
    const int k0 = min(c, nck - 1) * SS_KC;
    const unsigned ak = (unsigned)min(k0 + lane, K - 1) * 4u;
#pragma unroll
    for (int i = 0; i < 4 * TF; i++) r.a[i] = *reinterpret_cast<const float*>(Wt + (aoff[i] + ak));
#pragma unroll
    for (int j = 0; j < 4; j++) {
      const unsigned off = table[k0 + b_k + 16 * j];
#pragma unroll
      for (int i = 0; i < TP; i++) r.b[i][j] = *reinterpret_cast<const float*>(I + (pixbase[i] + off));
    }
  };
  auto stage = [&](const Regs& r, int c, double* buf) {
    const int left = K - c * SS_KC;  // taps from this chunk's start on
    double* As = buf + wave * SS_RSA + lane;
    double* Bs = buf + 16 * TF * SS_RSA + b_k * Gm::RSB + b_p;
    if (left >= SS_KC) {  // uniform
#pragma unroll
      for (int i = 0; i < 4 * TF; i++) As[4 * i * SS_RSA] = (double)r.a[i];
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int i = 0; i < TP; i++) Bs[16 * j * Gm::RSB + 16 * i] = (double)r.b[i][j];
    } else {
#pragma unroll
      for (int i = 0; i < 4 * TF; i++) As[4 * i * SS_RSA] = lane < left ? (double)r.a[i] : 0.0;
#pragma unroll
      for (int j = 0; j < 4; j++)
#pragma unroll
        for (int i = 0; i < TP; i++) Bs[16 * j * Gm::RSB + 16 * i] = b_k + 16 * j < left ? (double)r.b[i][j] : 0.0;
    }
  };

  d4 acc[TF][TP];
#pragma unroll
  for (int i = 0; i < TF; i++)
#pragma unroll
    for (int j = 0; j < TP; j++) acc[i][j] = d4_zero();

  __syncthreads();  // the table
  Regs ring[2];
  fetch(ring[0], 0);
  fetch(ring[1], 1);
  stage(ring[0], 0, ss_lds);
  fetch(ring[0], 2);
  __syncthreads();
  for (int c0 = 0; c0 < nck; c0 += 2) {
#pragma unroll
    for (int h = 0; h < 2; h++) {
      const int c = c0 + h;
      if (c < nck) {  // uniform
        const double* As = ss_lds + h * Gm::BUF + r16 * SS_RSA + 16 * wave + q;
        const double* Bs = ss_lds + h * Gm::BUF + 16 * TF * SS_RSA + (16 * wave + q) * Gm::RSB + r16;
        double a[TF][4], b[TP][4];  // this wavefront's quarter of the chunk: read first, staging runs meanwhile
#pragma unroll
        for (int s = 0; s < 4; s++) {
#pragma unroll
          for (int i = 0; i < TF; i++) a[i][s] = As[i * 16 * SS_RSA + 4 * s];
#pragma unroll
          for (int j = 0; j < TP; j++) b[j][s] = Bs[4 * s * Gm::RSB + 16 * j];
        }
        if (c + 1 < nck) stage(ring[h ^ 1], c + 1, ss_lds + (h ^ 1) * Gm::BUF);
        fetch(ring[h ^ 1], c + 3);
#pragma unroll
        for (int s = 0; s < 4; s++)
#pragma unroll
          for (int i = 0; i < TF; i++)
#pragma unroll
            for (int j = 0; j < TP; j++) acc[i][j] = mfma_f64(a[i][s], b[j][s], acc[i][j]);
        __syncthreads();
      }
    }
  }

  // partial blocks: [tile][v][wave][lane]; wavefront w finishes rows 4 w + q of every tile
#pragma unroll
  for (int i = 0; i < TF; i++)
#pragma unroll
    for (int j = 0; j < TP; j++)
#pragma unroll
      for (int v = 0; v < 4; v++) ss_lds[(((i * TP + j) * 4 + v) * 4 + wave) * WAVE + lane] = acc[i][j][v];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < TP; j++) {
    const int px = p0 + 16 * j + r16, pc = min(px, P - 1);
    const int n = pc / OHW, r = pc - n * OHW;
    float* out = p.O + (int64_t)n * F * OHW + r;
#pragma unroll
    for (int i = 0; i < TF; i++) {
      const int f = f0 + 16 * i + d_row(q, wave);
      const double* part = ss_lds + ((i * TP + j) * 4 + wave) * 4 * WAVE + lane;
      double x = p.bias ? (double)p.bias[min(f, F - 1)] : 0.0;  // the listing's first statement
      x += part[0];
      x += part[WAVE];
      x += part[2 * WAVE];
      x += part[3 * WAVE];
      if (px < P && f < F) out[(int64_t)f * OHW] = (float)x;
    }
  }
}

}  // namespace tc355
