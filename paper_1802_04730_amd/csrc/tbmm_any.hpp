// Transposed batched matmul of small matrices of any size (Section 7, "Transposed Batched Matrix Multiplication",
// listing tbmm): what tbmm_lds.hpp does, without its conditions on alignment and with room for larger matrices.
//
//     Z(b,n,m) = sum_k X(b,n,k) * Y(b,m,k)
//
// What bounds it: HBM at large batches (27 x 61 x 35: 18.9 KB and 72 MFMAs per batch element), which the wave-level
// kernel did not reach because it fetched operands row by row, 4 bytes per lane where K is odd.
// A job is one batch element, a strip of 16 TN rows of X_b and a strip of 16 TM rows of Y_b, done by one wavefront in its
// private LDS region, without barriers; the next job's operands travel in registers meanwhile.
//   * A strip is a contiguous run of memory that may start and end anywhere.  It is fetched as 16-byte pieces from the
//     16-byte boundary before it (tensors start on one), parked as it comes, and read from its first element on.  The
//     piece that holds a tensor's last elements is loaded from 4 elements before the end and moved into place: nothing
//     beyond the tensor is read.
//   * PAD (K a multiple of 16): 16 rows at such a stride share a few LDS banks, so a spare piece follows every 16.
//   * Results are laid out in the region and leave as contiguous streams: 16-byte pieces of the whole block where the
//     strip covers all of M (first and last piece element by element where they are shared), else row by row.
// MFMA roles and the order of m inside a tile are those of tbmm_lds.hpp.
// Measured, wave-level kernel -> this one: (B,N,M,K) = (4000,27,61,35) 37.1 -> 22.3 us (3.4 TB/s; 18.9 KB per element travel
// once, 8 % of the MFMA work is padding), (5972,36,47,73) 108 -> 60, (13047,58,14,17) 49 -> 23, (35,55,75,81) 13.5 -> 4.1.
#pragma once
#include "tc355_device.hpp"

namespace tc355 {

struct TbmmAnyArgs {
  const float* X;  // [B][N][K]
  const float* Y;  // [B][M][K]
  float* Z;        // [B][N][M]
  int N, M, K;
  int strips_n, strips_m;
  int jobs;              // B * strips_n * strips_m  (< 2^31, checked by the host)
  int wave_lds_units;    // 16-byte units of LDS per wavefront
  int64_t xtotal, ytotal;  // elements of X and Y, at least 4
};

// 16-byte pieces of a strip of `rows` rows of K elements at the worst alignment, in load instructions of a wavefront.
constexpr int tbmm_any_loads(int rows, int kmax) { return (rows * kmax + 6) / 4 / WAVE + 1; }

// Requests one strip: pieces 64*i + lane from element `first` (a multiple of 4) of a tensor of `total` elements on; lanes
// past the strip's end repeat its last piece (same address, same value, same LDS slot).
template <int U>
__device__ __forceinline__ void tbmm_any_fetch(f4 (&r)[U], const float* base, int64_t first, int64_t total, int pieces, int lane) {
  const char* at = reinterpret_cast<const char*>(base + first);
  if (first + 4 * (int64_t)pieces <= total) {  // uniform
#pragma unroll
    for (int i = 0; i < U; i++) r[i] = *reinterpret_cast<const f4*>(at + 16u * (unsigned)min(i * WAVE + lane, pieces - 1));
  } else {  // the strip ends with the tensor, inside a piece: that piece is loaded from total - 4
    const int back = (int)(first + 4 * (int64_t)pieces - total);  // 1 .. 3
#pragma unroll
    for (int i = 0; i < U; i++) {
      const int u = min(i * WAVE + lane, pieces - 1);
      const bool end = u == pieces - 1;
      const f4_any t = *reinterpret_cast<const f4_any*>(at + (16 * u - (end ? 4 * back : 0)));
      f4 v = t;
      if (end) {
        v[0] = back == 1 ? t[1] : back == 2 ? t[2] : t[3];
        v[1] = back == 1 ? t[2] : t[3];
        v[2] = t[3];
      }
      r[i] = v;
    }
  }
}

template <int TN, int TM, int KMAX, bool PAD>
__global__ __launch_bounds__(WG_THREADS, 2) void tbmm_any_kernel(TbmmAnyArgs p) {
  constexpr int NX = tbmm_any_loads(16 * TN, KMAX), NY = tbmm_any_loads(16 * TM, KMAX);
  extern __shared__ __attribute__((aligned(16))) char tbmm_smem[];
  const int lane = threadIdx.x & (WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int r16 = lane & 15, q = lane >> 4;
  const int N = p.N, M = p.M, K = p.K;
  char* lds = tbmm_smem + (size_t)wave * p.wave_lds_units * 16;
  float* ldsf = reinterpret_cast<float*>(lds);
  const unsigned stride = gridDim.x * WAVES_PER_WG;
  unsigned job = blockIdx.x * WAVES_PER_WG + wave;
  if (job >= (unsigned)p.jobs) return;  // whole wavefront leaves together; there is no barrier in this kernel

  struct Geo {
    unsigned b;
    int n0, m0;
    int xoff, yoff;  // elements between the 16-byte boundary and the strip
    int xu, yu;      // 16-byte pieces of the strips
  };
  struct Pre {
    f4 x[NX];
    f4 y[NY];
  };
  auto geometry = [&](unsigned j) {
    Geo g;
    const unsigned rest = j / (unsigned)p.strips_m;
    const int sm = (int)(j - rest * (unsigned)p.strips_m);
    g.b = rest / (unsigned)p.strips_n;
    g.n0 = (int)(rest - g.b * (unsigned)p.strips_n) * 16 * TN;
    g.m0 = sm * 16 * TM;
    g.xoff = (int)(((g.b * (unsigned)N + (unsigned)g.n0) * (unsigned)K) & 3u);  // (the low bits survive the wrap)
    g.yoff = (int)(((g.b * (unsigned)M + (unsigned)g.m0) * (unsigned)K) & 3u);
    g.xu = (g.xoff + min(16 * TN, N - g.n0) * K + 3) >> 2;
    g.yu = (g.yoff + min(16 * TM, M - g.m0) * K + 3) >> 2;
    return g;
  };
  auto fetch = [&](const Geo& g, Pre& r) {
    tbmm_any_fetch(r.x, p.X, ((int64_t)g.b * N + g.n0) * K - g.xoff, p.xtotal, g.xu, lane);
    tbmm_any_fetch(r.y, p.Y, ((int64_t)g.b * M + g.m0) * K - g.yoff, p.ytotal, g.yu, lane);
  };
  auto slot = [](int piece) { return PAD ? piece + (piece >> 4) : piece; };
  auto word = [](int w) { return PAD ? w + ((w >> 6) << 2) : w; };
  auto park = [&](const Geo& g, const Pre& r) {
#pragma unroll
    for (int i = 0; i < NX; i++) *reinterpret_cast<f4*>(lds + 16 * slot(min(i * WAVE + lane, g.xu - 1))) = r.x[i];
#pragma unroll
    for (int i = 0; i < NY; i++) *reinterpret_cast<f4*>(lds + 16 * slot(g.xu + min(i * WAVE + lane, g.yu - 1))) = r.y[i];
  };
  const int ksteps = (K + 3) >> 2;

  Geo geo = geometry(job);
  Pre pre;
  fetch(geo, pre);
  for (;;) {
    const Geo g = geo;
    park(g, pre);
    const unsigned next = job + stride;
    const bool more = next < (unsigned)p.jobs && next > job;  // uniform (32-bit wrap: no further job)
    if (more) {
      geo = geometry(next);
      fetch(geo, pre);  // in flight while this job is contracted
    }

    // LDS word of element k = q of this lane's rows (row clamped into the strip; such rows are never stored)
    int aidx[TM], bidx[TN];
#pragma unroll
    for (int t = 0; t < TM; t++) aidx[t] = 4 * g.xu + g.yoff + min(16 * t + 4 * (r16 & 3) + (r16 >> 2), M - 1 - g.m0) * K + q;
#pragma unroll
    for (int t = 0; t < TN; t++) bidx[t] = g.xoff + min(16 * t + r16, N - 1 - g.n0) * K + q;

    d4 acc[TN][TM];
#pragma unroll
    for (int tn = 0; tn < TN; tn++)
#pragma unroll
      for (int tm = 0; tm < TM; tm++) acc[tn][tm] = d4_zero();

    // One step = 4 reduction elements; in the last one the slots past K are zeroed in BOTH operands: what was read there
    // is the next row's data, possibly an Inf.
    auto step = [&](int s, bool last) {
      float af[TM], bf[TN];
#pragma unroll
      for (int t = 0; t < TM; t++) af[t] = ldsf[word(aidx[t] + 4 * s)];
#pragma unroll
      for (int t = 0; t < TN; t++) bf[t] = ldsf[word(bidx[t] + 4 * s)];
      if (last && 4 * s + q >= K) {
#pragma unroll
        for (int t = 0; t < TM; t++) af[t] = 0.0f;
#pragma unroll
        for (int t = 0; t < TN; t++) bf[t] = 0.0f;
      }
#pragma unroll
      for (int tm = 0; tm < TM; tm++)
#pragma unroll
        for (int tn = 0; tn < TN; tn++) acc[tn][tm] = mfma_f64((double)af[tm], (double)bf[tn], acc[tn][tm]);
    };
    for (int s = 0; s < ksteps - 1; s++) step(s, false);
    step(ksteps - 1, true);

    // write-back: Z[b][n0 + 16*tn + r16][m0 + 16*tm + 4*q + v] = acc[tn][tm][v], through the region
    const int rows = min(16 * TN, N - g.n0), cols = min(16 * TM, M - g.m0);
    const bool flat = cols == M;  // one contiguous block (uniform)
    const int64_t z0 = ((int64_t)g.b * N + g.n0) * M + g.m0;
    const int zoff = flat ? (int)((g.b * (unsigned)N + (unsigned)g.n0) * (unsigned)M & 3u) : 0;
#pragma unroll
    for (int tn = 0; tn < TN; tn++)
#pragma unroll
      for (int tm = 0; tm < TM; tm++)
#pragma unroll
        for (int v = 0; v < 4; v++)
          if (16 * tn + r16 < rows && 16 * tm + 4 * q + v < cols)
            ldsf[zoff + (16 * tn + r16) * cols + 16 * tm + 4 * q + v] = (float)acc[tn][tm][v];
    if (flat) {
      const int end = zoff + rows * M, zu = (end + 3) >> 2;
      float* zs = p.Z + (z0 - zoff);
      for (int u = lane; u < zu; u += WAVE) {
        const f4 v = *reinterpret_cast<const f4*>(lds + 16 * u);
        if (4 * u >= zoff && 4 * u + 4 <= end) {
          store_stream(reinterpret_cast<f4*>(zs + 4 * u), v);
        } else {
#pragma unroll
          for (int e = 0; e < 4; e++)
            if (4 * u + e >= zoff && 4 * u + e < end) zs[4 * u + e] = v[e];
        }
      }
    } else {
      // 16*TM columns (fewer in the last strip): whole rows by 64 lanes, or 2 or 4 rows side by side
      constexpr int RP = TM == 1 ? 4 : TM == 2 ? 2 : 1;
      const int r0 = lane / (WAVE / RP), c0 = lane % (WAVE / RP);
      float* zs = p.Z + z0;
      for (int r = r0; r < rows; r += RP)
        for (int c = c0; c < cols; c += WAVE / RP) zs[(int64_t)r * M + c] = ldsf[r * cols + c];
    }
    if (!more) return;
    job = next;
  }
}

}  // namespace tc355
