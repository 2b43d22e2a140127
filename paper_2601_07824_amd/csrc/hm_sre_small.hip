// hm_sre_small.hip -- a whole evaluation of M_q for up to seven (FP64: six) qubits in one launch of one workgroup
// (Algorithm 2, Eqs. Z_FT_qubits and sre).
//
// All 2^N shift vectors of 2^(N-1) folded values are at most 2^13 values, one workgroup tile.  What such a call
// costs is its launches: the tile pass over several workgroups and the sum over the shifts are 6.3 + 3.1 us of
// kernels and a gap, one workgroup doing both takes 8.9 us at N = 7 (a whole call: 9.1 us at N = 7, 8.0 to 8.5 us
// at N <= 6, against 10.7 us in two launches at N = 8).  Above the line the one workgroup's own work is the
// longer: complex64 N = 8 14.9 against 10.7 us, complex128 N = 7 with q = (1, 2, 3) 20.6 against 16.3 us.  The
// tile is the resident row pass's (same rounds, same sums per shift).
#include "hm_sre_kern.h"
#include "hm_totals.h"

namespace hm {
namespace {

template <typename T, int NT, int RB, int NL, int QM>
__global__ __launch_bounds__(NT) void k_sre_small(RowPassArgs A, int N, double *sums, double *out) {
  using Sh = RowShape<T, NT, RB, NL, true>;
  __shared__ typename Sh::Elem lds[Sh::LDS_N];
  __shared__ double red[(HM_MAX_Q + 1) * NT / 64];
  __shared__ double tot[HM_MAX_Q + 1];
  rowpass_tiles<T, NT, RB, NL, false, QM, true, RowPassArgs, true>(A, 0, 1, lds, red);
  __syncthreads();  // the per-shift sums are written, red is free
  block_rows_sum<NT>(A.shift_sums, A.n_slots, A.nacc, red, tot);
  if (sums && threadIdx.x < (uint32_t)A.nacc) sums[threadIdx.x] = tot[threadIdx.x];
  if (out) sre_finalize_into(tot, N, A.qa, out);
}

// Threads of the workgroup: the tile holds all 2^(2 NL + 1) values.
constexpr int small_nt(int NL, int RB) {
  const int bits = 2 * NL + 1 - RB;
  return bits < 6 ? 64 : 1 << bits;
}

template <typename T, int NL>
void launch_small(RowPassArgs A, int N, double *sums, double *out, hipStream_t st) {
  constexpr int RBM = ResidentRB<T>::value, RB = NL < RBM ? NL : RBM, NT = small_nt(NL, RB);
  A.n_tiles = row_tiles<NT, RB, NL>(A);
  ProfScope prof("sre_small", st);
  const int qm = q_mode(A.qa);
  if (qm == 2) hipLaunchKernelGGL((k_sre_small<T, NT, RB, NL, 2>), dim3(1), dim3(NT), 0, st, A, N, sums, out);
  else if (qm == 1) hipLaunchKernelGGL((k_sre_small<T, NT, RB, NL, 1>), dim3(1), dim3(NT), 0, st, A, N, sums, out);
  else hipLaunchKernelGGL((k_sre_small<T, NT, RB, NL, 0>), dim3(1), dim3(NT), 0, st, A, N, sums, out);
}

template <typename T>
int small_t(const SrePlan &p, const RowPassArgs &A, double *sums, double *out, hipStream_t st) {
  switch (p.nf) {
    case 0: launch_small<T, 0>(A, p.N, sums, out, st); break;
    case 1: launch_small<T, 1>(A, p.N, sums, out, st); break;
    case 2: launch_small<T, 2>(A, p.N, sums, out, st); break;
    case 3: launch_small<T, 3>(A, p.N, sums, out, st); break;
    case 4: launch_small<T, 4>(A, p.N, sums, out, st); break;
    case 5: launch_small<T, 5>(A, p.N, sums, out, st); break;
    case 6:
      if constexpr (sizeof(T) == 4) launch_small<T, 6>(A, p.N, sums, out, st);
      else return fail(E_UNSUPPORTED, "one-launch SRE: n = %d", p.N);
      break;
    default: return fail(E_UNSUPPORTED, "one-launch SRE: n = %d", p.N);
  }
  return hipPeekAtLastError() == hipSuccess ? OK : fail(E_HIP, "SRE launch: %s", hipGetErrorString(hipGetLastError()));
}

}  // namespace

int sre_small_run(const SrePlan &p, const void *psi, const QArgs &qa, double *shift_sums, double *sums, double *out,
                  hipStream_t st) {
  RowPassArgs A{};
  A.psi = psi;
  A.nf = p.nf;
  A.n_slots = (int64_t)1 << p.N;
  A.shift_sums = shift_sums;
  A.nacc = nacc_of(qa);
  A.qa = qa;
  return p.dbl ? small_t<double>(p, A, sums, out, st) : small_t<float>(p, A, sums, out, st);
}

}  // namespace hm
