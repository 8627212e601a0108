// Grouped convolution (Section 7, listing gconv) for FEW channels per group
// (C and F multiples of 4, up to 8; the paper's table shapes (4,4,56,56) and
// (8,8,28,28), and the same with a border of one pixel: widths 58 and 30), image width known at compile time:
//
//   O(n,g,o,h,w) = sum_{i,kh,kw} I(n,g,i,h+kh,w+kw) * W1(g,o,i,kh,kw) + bias(g*F+o)
//
// With 4 or 8 filters a 16 x 16 MFMA tile would be three quarters or half
// padding.  v_mfma_f64_4x4x4_4b_f64 multiplies four independent 4 x 4 x 4 blocks
// per instruction at the same flop rate; measured layout (one-hot probe), lane =
// 16*k + 4*blk + idx:
//   A: lane supplies A_blk[i = idx][k]      B: lane supplies B_blk[k][j = idx]
//   D: lane 16*i + 4*blk + j holds D_blk[i][j]
// Here all four blocks share A = the weights of 4 filters x 4 channels for one
// filter tap, and take 4 different pixel quads: one instruction contracts 4
// channels of one tap for 4 filters x 16 pixels, with no padding.  In the
// terms of the 16-wide kernels (r16 = lane % 16, q = lane / 16) the B operand
// is again I[channel 4*c4 + q][pixel r16], one 8-byte LDS read at a
// compile-time immediate; the A operand is W1[filter 4*fq + lane % 4][channel
// 4*c4 + q]; and the lane ends up with O[filter 4*fq + q][pixel r16].
//
// One workgroup per band of ROWS output rows of an (image, group) pair: the band is widened to fp64 once and staged in LDS
// ([channel][pixels], plane stride = 16 mod 32 doubles); the filter bank sits in registers; the tiles of a band are dealt to
// the four wavefronts round-robin and advance TN at a time with the LDS reads one step ahead of the MFMAs.  Several
// workgroups per compute unit cover each other's staging.
//
// What bounds it: fp64 MFMAs and vector instructions of a SIMD exclude each other, and with 4 filters every MFMA takes an LDS
// read of its own, 16 clocks of the unit's LDS for 17 of the matrix core.  So: the weights and the band in one round trip,
// addresses as immediates (no division per load or tile), no two channel rows of a tile on the same banks, and small
// bands, so that few pairs fill the chip and a launch does not end with a whole image on every third unit.  Against one
// workgroup per pair that walks over its bands (us; pairs of 4 channels 56 x 56 / 58 x 58, of 8 channels 28 x 28 / 30 x 30): 1024
// pairs 32.4 -> 25.4 / 34.1 -> 28.1 / 21.6 -> 20.9 / 27.6 -> 25.8, 256 pairs 14.0 -> 8.9 / 14.9 -> 10.0 / 7.7 -> 7.1 / 9.9 -> 8.0, 128 pairs
// 13.0 -> 5.5 / 14.1 -> 6.3 / 7.3 -> 5.1 / 9.4 -> 5.5.  Taken back: persistent workgroups that keep the bank and load the next band
// while one is contracted (25.4 -> 26.3, 20.9 -> 20.7); predicated loads (25.4 -> 28.7).
#pragma once
#include "tc355_device.hpp"

namespace tc355 {

struct GconvQuadArgs {
  const float* I;
  const float* W1;
  const float* bias;  // or nullptr
  float* O;
  int64_t NG;  // images times groups
  int G, H;
  unsigned first;  // number of the launch's first workgroup (a multiple of 8)
};

template <int C, int F, int KH, int KW, int W, int ROWS, int TN>
struct GconvQuadGeom {
  static constexpr int OW = W - KW + 1;
  static constexpr int IN_ROWS = ROWS + KH - 1;
  static constexpr int LEN = IN_ROWS * W;                          // floats per channel plane of a band
  static constexpr int PS = ((LEN + 31 - 16) / 32) * 32 + 16;      // plane stride in doubles, = 16 (mod 32), >= LEN
  static constexpr int WN = F * C * KH * KW;                       // weights of a group
  static constexpr int ROUND = WAVES_PER_WG * TN * 16;             // pixels of a round of tiles
  static constexpr int PIXELS = (ROWS * W + ROUND - 1) / ROUND * ROUND;  // pixels contracted, the columns between two rows among them
  static constexpr int LAST = (C - 1) * PS + PIXELS + (KH - 1) * W + KW - 1;  // doubles up to the last one that is read
  static constexpr int WEIGHTS = (LAST > C * PS ? LAST : C * PS) * 8;         // byte offset of the weights, as they come
  static constexpr int LDS_BYTES = WEIGHTS + WN * 4;
  static constexpr int CQ = C / 4, FQ = F / 4;
  static constexpr int NS = KH * KW * CQ;                          // reduction steps per tile
  static_assert(C % 4 == 0 && F % 4 == 0 && C <= 8 && F <= 8, "4 or 8 channels and filters per group");
  static constexpr int VEC = W % 4 == 0 ? 4 : 2;                   // floats per staging load: rows start 16- or 8-byte aligned
  static_assert(W % 2 == 0, "8-byte loads at least: every row starts 8-byte aligned");
  static constexpr int CT = WG_THREADS / C;                        // threads that stage one channel
  static constexpr int NLD = (LEN + VEC * CT - 1) / (VEC * CT);    // loads per thread
  static_assert(LEN % VEC == 0, "whole loads");
  static_assert((4 * (CQ - 1) * PS + (KH - 1) * W + KW - 1 + 64 * (TN - 1)) * 8 < 65536, "LDS immediates out of range");
};

template <int C, int F, int KH, int KW, int W, int ROWS, int TN, int MINW>
__global__ __launch_bounds__(WG_THREADS, MINW) void gconv_quad_kernel(GconvQuadArgs p) {
  using Gm = GconvQuadGeom<C, F, KH, KW, W, ROWS, TN>;
  constexpr int OW = Gm::OW, PS = Gm::PS, NS = Gm::NS, LEN = Gm::LEN, CQ = Gm::CQ, FQ = Gm::FQ, WN = Gm::WN, VEC = Gm::VEC;
  extern __shared__ __attribute__((aligned(16))) double gq_band[];  // [C][PS], then the weights
  float* wl = reinterpret_cast<float*>(reinterpret_cast<char*>(gq_band) + Gm::WEIGHTS);

  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int r16 = lane & 15, q = lane >> 4;
  const int H = p.H, OH = H - KH + 1;
  const int npix = OH * OW;
  // the bands of a pair are on one XCD (workgroups equal modulo 8), whose L2 keeps the rows that two bands read
  const unsigned nbands = (unsigned)((OH + ROWS - 1) / ROWS), wg = p.first + blockIdx.x, oct = wg / (8 * nbands);
  const int64_t ng = (int64_t)oct * 8 + wg % 8;  // n*G + g
  if (ng >= p.NG) return;  // (the whole workgroup)
  const int h0 = (int)((wg - oct * 8 * nbands) / 8) * ROWS;
  const int g = (int)(ng % p.G);
  const int64_t plane = (int64_t)H * W;

  // ---- one round trip to memory: the group's weights and the band, rows h0 .. of every channel.  W is a multiple of 4 (of 2),
  // so planes, band starts and row ends are 16-byte (8-byte) aligned.  CT threads per channel: loads and LDS writes are one
  // address each and immediates.
  {
    constexpr int CT = Gm::CT, NLD = Gm::NLD, WLD = (WN + WG_THREADS - 1) / WG_THREADS;
    const int c = tid / CT, i0 = VEC * (tid % CT);
    const int avail = min((H - h0) * W, LEN);  // floats of each plane that belong to this band (a multiple of VEC)
    const float* src = p.I + (ng * C + c) * plane + (int64_t)h0 * W;
    const float* wg = p.W1 + (int64_t)g * WN;
    float wv[WLD];
    Vec<float, VEC> v[NLD];
#pragma unroll
    for (int j = 0; j < WLD; j++) wv[j] = wg[min(tid + j * WG_THREADS, WN - 1)];
#pragma unroll
    for (int j = 0; j < NLD; j++)
      v[j] = load_vec<float, VEC>(src + min(i0 + j * VEC * CT, avail - VEC));  // clamped: predicated, they would wait for each other
#pragma unroll
    for (int j = 0; j < WLD; j++)
      if (tid + j * WG_THREADS < WN) wl[tid + j * WG_THREADS] = wv[j];
    double* d = gq_band + c * PS + i0;  // PS and i0 are even: 16-byte aligned pairs
#pragma unroll
    for (int j = 0; j < NLD; j++) {  // widened once; rows past the image are skipped
      if (i0 + j * VEC * CT < avail) {
#pragma unroll
        for (int e = 0; e < VEC; e += 2) {
          const dbl2 pr = {(double)v[j].e[e], (double)v[j].e[e + 1]};
          *reinterpret_cast<dbl2*>(d + j * VEC * CT + e) = pr;
        }
      }
    }
  }
  double bz[FQ];  // the lane's outputs belong to filter 4*fq + q
#pragma unroll
  for (int fq = 0; fq < FQ; fq++) bz[fq] = p.bias ? (double)p.bias[g * F + 4 * fq + q] : 0.0;
  __syncthreads();
  // ---- filter bank -> registers: a[s][fq] = W1[g][4*fq + lane%4][4*c4 + q][kh][kw], s = (kh*KW + kw)*CQ + c4
  double a[NS][FQ];
  {
    const float* wq = wl + ((lane & 3) * C + q) * (KH * KW);
#pragma unroll
    for (int kk = 0; kk < KH * KW; kk++)
#pragma unroll
      for (int c4 = 0; c4 < CQ; c4++)
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) a[kk * CQ + c4][fq] = (double)wq[(4 * fq * C + 4 * c4) * (KH * KW) + kk];
  }

  // ---- tiles of 16 consecutive pixels of the band's input rows (a tile that stepped over the KW - 1 columns that have no
  // output would put two of its four channel rows on the same LDS banks), dealt round-robin: wavefront w takes tiles w, w + 4,
  // ...; TN of them advance together.  What lies between two rows and behind the last one is contracted and not stored.
  const int end = min(ROWS, OH - h0) * W;
  float* dst = p.O + ng * (int64_t)F * npix + h0 * OW;
  int px = 16 * wave + r16, col = px % W, out = q * npix + px / W * OW + col;  // of the first tile: input pixel, its column, offset in O
  const double* bp = gq_band + q * PS + px;
  for (int p0 = 16 * wave; p0 < end; p0 += Gm::ROUND) {
    double acc[TN][FQ], bcur[TN], bnxt[TN];
#pragma unroll
    for (int t = 0; t < TN; t++) {
#pragma unroll
      for (int fq = 0; fq < FQ; fq++) acc[t][fq] = bz[fq];  // start from the bias: one add less per output
      bcur[t] = bp[64 * t];
    }
#pragma unroll
    for (int s = 0; s < NS; s++) {
      if (s + 1 < NS) {
        const int kk = (s + 1) / CQ, c4 = (s + 1) % CQ;
        const int off = 4 * c4 * PS + (kk / KW) * W + (kk % KW);
#pragma unroll
        for (int t = 0; t < TN; t++) bnxt[t] = bp[off + 64 * t];
      }
      __builtin_amdgcn_sched_barrier(0);  // reads of step s+1, then the MFMAs of step s
#pragma unroll
      for (int t = 0; t < TN; t++)
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) acc[t][fq] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[s][fq], bcur[t], acc[t][fq], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < TN; t++) bcur[t] = bnxt[t];
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int t = 0; t < TN; t++) {
      if (px < end && col < OW) {
#pragma unroll
        for (int fq = 0; fq < FQ; fq++) (dst + 4 * fq * (int64_t)npix)[(unsigned)out] = (float)acc[t][fq];
      }
      // 64 pixels on
      px += 64;
      col += 64 % W;
      out += 64 / W * OW + 64 % W;
      if (col >= W) {
        col -= W;
        out -= KW - 1;
      }
    }
    bp += Gm::ROUND;
  }
}

}  // namespace tc355
