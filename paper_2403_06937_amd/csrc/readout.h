// Per-step readout of rho's diagonal by one workgroup, shared by the readout
// kernels and by the small product kernel (whose first product of a step reads
// the records of the state that it multiplies).
#pragma once
#include "common.h"

namespace tcm {

constexpr int READOUT_NT = 512;                  // threads of the workgroup
constexpr int READOUT_NW = READOUT_NT / 64;
constexpr int READOUT_LDS = 3 * READOUT_NW;      // doubles

__device__ __forceinline__ double readout_wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// map == NULL: rho is in the basis order; else basis state s sits at row and
// column map[s] of rho (the excitation-sorted order of the sector stepper).
// off != NULL: rho holds the states of one sector k only, whose states with m
// photons (k - m excited atoms) sit at positions off[m] .. off[m + 1] - 1.
// Writes pop = sum_s |l(s)| Re rho_ss, pdist[m] = sum_{photon(s) = m} Re rho_ss
// and pstate[m] = P({m>) of Eq. (13) (m photons and n - m excited atoms),
// m = 0 .. min(n, c); each output may be NULL.
//
// Bound by the latency of the diagonal's scattered loads (each its own cache
// line): the photon blocks are spread over the waves, several waves to a block
// when there are fewer blocks than waves, and a lane issues four loads at a
// time.  The sums run in an order fixed by n and c alone.
template <typename E>
__device__ __forceinline__ void readout_body(int n, int c, const E* __restrict__ rho, int64_t ld,
                                             const int32_t* __restrict__ map,
                                             const int32_t* __restrict__ off, int k_sector,
                                             double* __restrict__ pop, double* __restrict__ pdist,
                                             double* __restrict__ pstate, double* sh) {
  const int64_t per = int64_t(1) << n;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int seg = c + 1 >= READOUT_NW ? 1 : READOUT_NW / (c + 1);   // waves to a photon block
  const int units = (c + 1) * seg;
  double tot = 0.0;
  for (int u = wave; u < units; u += READOUT_NW) {
    const int mm = u / seg;
    const int64_t s0 = off ? int64_t(off[mm]) : int64_t(mm) << n;
    const int64_t count = off ? int64_t(off[mm + 1]) - s0 : per;
    double part = 0.0, st = 0.0;
    const int64_t step = int64_t(seg) * 64;
    for (int64_t l0 = (u - mm * seg) * 64 + lane; l0 < count; l0 += 4 * step) {
      int64_t q[4];
      double d[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int64_t l = l0 + k * step;
        q[k] = l < count ? (map ? int64_t(map[s0 + l]) : s0 + l) : -1;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) d[k] = q[k] >= 0 ? double(rho[q[k] * ld + q[k]].re) : 0.0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        if (q[k] < 0) continue;                 // past the block
        const int pc = off ? k_sector - mm : __popcll(uint64_t(l0 + k * step));
        part += d[k];
        tot += double(pc) * d[k];
        if (pc == n - mm) st += d[k];
      }
    }
    if (pdist) part = readout_wave_sum(part);
    if (pstate && mm <= n) st = readout_wave_sum(st);
    if (lane == 0) {
      if (seg == 1) {
        if (pdist) pdist[mm] = part;
        if (pstate && mm <= n) pstate[mm] = st;
      } else {
        sh[u] = part;
        sh[READOUT_NW + u] = st;
      }
    }
  }
  tot = readout_wave_sum(tot);
  if (lane == 0) sh[2 * READOUT_NW + wave] = tot;
  __syncthreads();
  if (seg > 1 && int(threadIdx.x) <= c) {
    const int mm = threadIdx.x;
    double part = 0.0, st = 0.0;
    for (int k = 0; k < seg; ++k) {
      part += sh[mm * seg + k];
      st += sh[READOUT_NW + mm * seg + k];
    }
    if (pdist) pdist[mm] = part;
    if (pstate && mm <= n) pstate[mm] = st;
  }
  if (threadIdx.x == 0 && pop) {
    double t = 0.0;
    for (int w = 0; w < READOUT_NW; ++w) t += sh[2 * READOUT_NW + w];
    *pop = t;
  }
}

}  // namespace tcm
