// hm_totals.h -- fixed-order sums of per-shift (or per-workgroup) FP64 sums by one workgroup, and the
// finalised Renyi entropies (Eq. sre).  The tree over the threads runs by lane shuffles, then over the
// waves in LDS: one barrier instead of one per halving and slot (256 shifts: 4.0 -> 3.1 us per launch, most
// of it the launch itself; mana's 256 x 3 sums 7.2 -> 3.4 us), in an order that depends on the workgroup size only.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hm_tile.h"

namespace hm {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sums of s[k], k < nacc (<= K, uniform), over the NT threads of the workgroup into tot[k] (shared); red holds
// K * NT / 64 doubles.  Every thread must call it; tot may be read by all threads afterwards.
template <int NT, int K>
__device__ __forceinline__ void block_sums(const double (&s)[K], int nacc, double *red, double *tot) {
  constexpr int NW = NT / 64;
  const uint32_t t = threadIdx.x;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (k < nacc) {
      const double v = wave_sum(s[k]);
      if ((t & 63u) == 0) red[k * NW + (t >> 6)] = v;
    }
  }
  __syncthreads();
  if (t < (uint32_t)nacc) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) v += red[t * NW + w];
    tot[t] = v;
  }
  __syncthreads();
}

// Sum of rows [0, n) of nacc doubles: thread t adds the rows t, t + NT, ..., then the tree.
template <int NT>
__device__ __forceinline__ void block_rows_sum(const double *rows_, int64_t n, int nacc, double *red, double *tot) {
  double s[HM_MAX_Q + 1];
#pragma unroll
  for (int k = 0; k <= HM_MAX_Q; ++k) s[k] = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += NT) {
    const double *row = rows_ + i * nacc;
#pragma unroll
    for (int k = 0; k <= HM_MAX_Q; ++k)
      if (k < nacc) s[k] += row[k];
  }
  block_sums<NT, HM_MAX_Q + 1>(s, nacc, red, tot);
}

// out = {M_q..., lost_norm} of N qubits from the sums over all shifts, one index per thread.
__device__ __forceinline__ void sre_finalize_into(const double *tot, int N, const QArgs &qa, double *out) {
  const int i = (int)threadIdx.x;
  if (i > qa.nq) return;
  const double D = ldexp(1.0, N);
  if (i == qa.nq) {
    out[i] = 1.0 - tot[0] / D;
  } else {
    const double q = qa.q[i];
    out[i] = (q == 1.0) ? -tot[1 + i] / D : log2(tot[1 + i] / D) / (1.0 - q);
  }
}

}  // namespace hm
