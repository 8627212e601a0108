// Lookup-table sums (Section 7, production model; appendix listing 2LUT):
//   O_t(i,j) +=! LUT_t(Idx_t(i,k), j)          for every table t of the call
// A pure gather: B*L rows of D floats out of a table of E rows (the paper's
// sizes: E = 10^7, D = 64, L = 50, B = 128: 1.6 MB gathered out of 2.56 GB),
// summed per output row.  Nothing here is a contraction; what matters is that
// every load of a row is in flight at once instead of one after the other
// (the paper's two-stage loading serves the same end): a thread first reads
// all its indices (one round trip), then all its table rows (a second one).
//
// A workgroup takes `rows` output rows of one table.  A row of D floats is read as units of V floats (V = 4: 16-byte
// loads at whatever alignment D leaves; the last unit of a D that is no multiple of 4 starts at D - 4 and repeats columns
// of the one before); an output row has `slots` groups of `cpw` threads: thread (slot s, column unit u) sums the lookups
// k = s, s + slots, ... of its unit in fp64, and the slots are combined in a fixed order, inside a wavefront by cross-lane
// moves, then through LDS.  The host takes as few slots as leave a thread LUT_NB lookups: all of them travel together, so
// more slots save nothing.  (A workgroup per output row whatever its lookups, 16 slots at D = 64, single columns where D is
// no multiple of 4: 18.8 us -> 2.8 at (3 tables, batch 2136, 1 lookup, D = 16), 18.7 -> 4.1 at (3, 2106, 18, 16), 23.0 -> 5.1 at
// (3, 2922, 29, 16), 6.6 -> 6.35 at (3, 573, 35, 128), whose floor is 5.9; 1.69 times on average at 150 random calls, 15.0 -> 15.6
// at worst of those above 4 us.)  At the paper's size (D = 64, L = 50, batch 128) it is one row of 16 slots of 16 threads,
// four lookups each: two round trips to memory behind a launch.  Every sum is exact up to the final rounding to fp32 (fp64
// holds the sum of 2^29 floats of equal exponent range exactly enough: the error is far below one fp32 rounding).
//
// An index outside [0, E) has no meaning in the comprehension: nothing is read
// for it, and the whole output row is NaN (every thread of its slot makes its sum NaN).
#pragma once
#include "tc355_device.hpp"

namespace tc355 {

constexpr int LUT_MAX_TABLES = 8;
constexpr int LUT_NB = 4;  // lookups in flight per thread and round

struct LutArgs {
  const float* LUT[LUT_MAX_TABLES];  // [E][D]
  const int* Idx[LUT_MAX_TABLES];    // [B][L]
  float* O[LUT_MAX_TABLES];          // [B][D]
  long long E[LUT_MAX_TABLES];
  int L[LUT_MAX_TABLES];
  int D, B;
  int cpw;     // column units per workgroup: a power of two, <= 256
  int slots;   // threads that share an output row's lookups: a power of two, cpw * slots <= 256
  int blocks;  // column blocks per row: ceil(ceil(D / V) / cpw)
};

template <int V>
__global__ __launch_bounds__(WG_THREADS) void lut_sum_kernel(LutArgs p) {
  __shared__ double part[WG_THREADS * V];
  const int tid = threadIdx.x;
  const int cpw = p.cpw, slots = p.slots, per_row = cpw * slots;
  const int ul = tid & (cpw - 1), s = (tid & (per_row - 1)) / cpw;
  const int cb = blockIdx.x % p.blocks;
  const int64_t i = (int64_t)(blockIdx.x / p.blocks) * (WG_THREADS / per_row) + tid / per_row;
  const int t = blockIdx.y;
  const int u = cb * cpw + ul;
  const bool on = (unsigned)u < ((unsigned)p.D + V - 1) / V && i < p.B;
  const int col = (int)min((unsigned)u * V, (unsigned)(p.D - V));
  const int L = on ? p.L[t] : 0;
  const long long E = p.E[t];
  const int* idx = p.Idx[t] + (on ? i * L : 0);
  const float* tab = p.LUT[t] + col;

  double acc[V];
#pragma unroll
  for (int e = 0; e < V; e++) acc[e] = 0.0;
  bool bad = false;
  for (int k0 = s; k0 < L; k0 += slots * LUT_NB) {
    int row[LUT_NB];
    // stage 1: the indices of this round
#pragma unroll
    for (int j = 0; j < LUT_NB; j++) {
      const int k = k0 + j * slots;
      row[j] = k < L ? idx[k] : 0;
    }
    // stage 2: the table rows, all requested before the first is used (a default for the ones that are not there, written to
    // the same registers, would make every request wait for the one before it)
    bool ok[LUT_NB];
#pragma unroll
    for (int j = 0; j < LUT_NB; j++) {
      const bool there = k0 + j * slots < L, inside = row[j] >= 0 && (long long)row[j] < E;
      bad = bad || (there && !inside);
      ok[j] = there && inside;
    }
    Vec<float, V> val[LUT_NB];
#pragma unroll
    for (int j = 0; j < LUT_NB; j++) {
      if (ok[j]) {
        const float* src = tab + (int64_t)row[j] * p.D;
        if constexpr (V == 4) val[j] = load_vec_any<float, 4>(src);
        else val[j].e[0] = *src;
      }
    }
#pragma unroll
    for (int j = 0; j < LUT_NB; j++) {
      if (ok[j]) {
#pragma unroll
        for (int e = 0; e < V; e++) acc[e] += (double)val[j].e[e];
      }
    }
  }
  if (bad) {
#pragma unroll
    for (int e = 0; e < V; e++) acc[e] = __builtin_nan("");
  }
  for (int m = cpw; m < WAVE && m < per_row; m *= 2) {  // (uniform) slots of one wavefront
#pragma unroll
    for (int e = 0; e < V; e++) acc[e] += __shfl_xor(acc[e], m);
  }
  const int step = max(1, WAVE / cpw);  // slots per wavefront
  if (slots > step) {  // (uniform) several wavefronts share a row
    if ((s & (step - 1)) == 0) {
#pragma unroll
      for (int e = 0; e < V; e++) part[e * WG_THREADS + tid] = acc[e];
    }
    __syncthreads();
    if (s == 0) {
      for (int o = step; o < slots; o += step)
#pragma unroll
        for (int e = 0; e < V; e++) acc[e] += part[e * WG_THREADS + tid + o * cpw];
    }
  }
  if (s == 0 && on) {
    float* out = p.O[t] + i * p.D + col;
    if constexpr (V == 4) {
      *reinterpret_cast<f4_any*>(out) = f4_any{(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
    } else {
      *out = (float)acc[0];
    }
  }
}

}  // namespace tc355
