// hm_mixed.hip -- mana of a mixed qutrit state (Sec. "Mana of mixed states via a fast tensor-product
// transform" of "Computing quantum magic of state vectors", Eq. MN_factor_mana and its Algorithm) and
// the reduced density matrix of a pure state (Sec. "Mana calculation", subsystem mana).
//
// All 9^N values w_u = Tr(rho A_u) are one tensor power of a 9 x 9 single-qutrit matrix applied to the
// vectorised density matrix.  On the GPU the density matrix (row-major, rho[r 3^N + c] = <r|rho|c>,
// qutrit k = base-3 digit k of r and c) is reordered so that qutrit k's pair (r_k, c_k) is the base-9
// digit k of the position (p = sum_k (3 r_k + c_k) 9^k), and the single-qutrit matrix is applied along
// every digit.  Several digits share one HBM-streaming pass through LDS:
//   * the first pass reads a 27 x 27 block of rho (qutrits 0..2 of its rows and columns vary, 27
//     contiguous columns per row), applies the matrix along digits 0, 1, 2 and writes the 729 values
//     contiguously in digit order (the reordering costs no pass of its own);
//   * each further pass takes up to three digits k .. k + ND - 1 with J contiguous lower positions along
//     for the coalescing, in place: the first digit is transformed on the way in (a thread loads whole
//     fibres), the last on the way out, so LDS holds the tile between two digits only;
//   * the last pass does not write back: it reduces sum_u |w_u|, sum_u w_u and sum_u w_u^2 in FP64
//     (fixed order) instead.
// The passes are bound by HBM (read and write rate of a plain copy 4.75 TB/s), so their number decides:
// N = 8 streams the 9^N values 3 times (read + write twice, read once).  With at most two digits per later
// pass it was 4 times: N = 8 complex128 1019 us then, 740 us now.
//
// The single-qutrit matrix, from A_ab|x> = omega^{2b(a-x)} |2a - x> (the phase-space point operators of
// Eq. phase-space up to a relabelling of the points): with x_mu = rho_{r,c} at mu = 3 r + c,
//   w_{3a+b} = sum_c omega^{2b(a-c)} x_{3((2a - c) mod 3) + c},
// three non-zero entries per row (the F_3 blocks of the paper's factorisation M = P (F3+F3+F3) P').
// Mana = log2(sum_u |w_u| / 3^N) (Eq. mana with W = Tr(rho A)/3^N).
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "hm_internal.h"
#include "hm_tile.h"

namespace hm {

// The single-qutrit transform of one fibre x[0..8] -> y[0..8].
template <typename T>
__device__ __forceinline__ void mixed_fibre(const vec2<T> (&x)[9], vec2<T> (&y)[9]) {
  const T h = T(-0.5), s = T(0.86602540378443864676372317075294);  // omega = h + i s
#pragma unroll
  for (int a = 0; a < 3; ++a)
#pragma unroll
    for (int b = 0; b < 3; ++b) {
      T re = T(0), im = T(0);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        const vec2<T> z = x[3 * ((2 * a - c + 3) % 3) + c];
        const int m = (2 * b * (a - c + 3)) % 3;  // omega^m
        if (m == 0) {
          re += z.x;
          im += z.y;
        } else {
          const T si = m == 1 ? s : -s;
          re += h * z.x - si * z.y;
          im += h * z.y + si * z.x;
        }
      }
      y[3 * a + b].x = re;
      y[3 * a + b].y = im;
    }
}

static constexpr int MIXED_NT = 256;
static constexpr int MIXED_RED_BLOCKS = 2048;

// Fibres of 9 values at stride ST inside an LDS tile of NF fibres: fibre f starts at
// (f / ST) * 9 ST + f % ST; thread t takes fibres t, t + MIXED_NT, ...
template <int ST>
__device__ __forceinline__ int fibre_base(int f) {
  return (f / ST) * ST * 9 + f % ST;
}
template <typename T, int NF, int ST>
__device__ __forceinline__ void lds_digit(vec2<T> *t) {
  for (int f = threadIdx.x; f < NF; f += MIXED_NT) {
    const int base = fibre_base<ST>(f);
    vec2<T> x[9], y[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) x[a] = t[base + a * ST];
    mixed_fibre<T>(x, y);
#pragma unroll
    for (int a = 0; a < 9; ++a) t[base + a * ST] = y[a];
  }
}
// The fibre sums {sum |w|, sum w, sum w^2} of the real parts into acc (FP64).
template <typename T>
__device__ __forceinline__ void fibre_sums(const vec2<T> (&y)[9], double (&acc)[3]) {
#pragma unroll
  for (int a = 0; a < 9; ++a) {
    const double w = (double)y[a].x;  // real for a Hermitian rho
    acc[0] += fabs(w);
    acc[1] += w;
    acc[2] = fma(w, w, acc[2]);
  }
}

// Fixed-order workgroup sums of acc into part[blockIdx.x].
__device__ __forceinline__ void block_sums_out(double (&acc)[3], double *part) {
  __shared__ double red[3][MIXED_NT];
  for (int k = 0; k < 3; ++k) red[k][threadIdx.x] = acc[k];
  __syncthreads();
  for (unsigned w = MIXED_NT / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 3; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0)
    for (int k = 0; k < 3; ++k) part[blockIdx.x * 3 + k] = red[k][0];
}

// First pass: tile q (q < 9^(N - M)) is the 3^M x 3^M block of rho whose rows and columns share the
// base-3 digits M.. of q's pairs (mu_k = 3 r_k + c_k = base-9 digit k - M of q).  A thread loads the 3 x 3
// entries of a digit-0 fibre, transforms and stores them at p_lo = sum_{j < M} mu_j 9^j in LDS; digits 1 ..
// M - 1 follow there, the last of them on the way to v[q 9^M + p_lo] (REDUCE: into the sums instead).
// M = min(N, 3).
template <typename T, int M, bool REDUCE>
__global__ __launch_bounds__(MIXED_NT) void k_mixed_first(const vec2<T> *__restrict__ rho, uint64_t D, uint64_t n_tiles,
                                                           vec2<T> *__restrict__ v, double *part) {
  constexpr int B = M == 1 ? 3 : M == 2 ? 9 : 27;  // 3^M
  constexpr int TILE = B * B;                       // 9^M
  constexpr int NF = TILE / 9, LST = TILE / 9;      // fibres; stride of the last digit
  __shared__ vec2<T> t[M > 1 ? TILE : 1];
  double acc[3] = {0.0, 0.0, 0.0};
  for (uint64_t b = blockIdx.x; b < n_tiles; b += gridDim.x) {
    // neighbouring blocks share cache lines at their edges: keep them on one XCD's L2
    const uint64_t q = (uint64_t)xcd_tile((int64_t)b, (int64_t)n_tiles);
    // high row / column parts of the block
    uint64_t R = 0, C = 0, w3 = B, qq = q;
    while (qq) {
      const uint32_t mu = (uint32_t)(qq % 9);
      qq /= 9;
      R += (mu / 3) * w3;
      C += (mu % 3) * w3;
      w3 *= 3;
    }
    vec2<T> *o = v + q * TILE;
    auto put = [&](const vec2<T>(&y)[9], int base) {
      if constexpr (REDUCE) {
        fibre_sums<T>(y, acc);
      } else {
#pragma unroll
        for (int a = 0; a < 9; ++a) o[base + a * LST] = y[a];
      }
    };
    if constexpr (M > 1) __syncthreads();  // the previous tile's LDS reads are done
    for (int f = threadIdx.x; f < NF; f += MIXED_NT) {
      // fibre f: row group f / (B / 3), column group f % (B / 3) (the digits above digit 0)
      const int rg = f / (B / 3), cg = f % (B / 3);
      vec2<T> x[9], y[9];
      const vec2<T> *src = rho + (R + 3 * rg) * D + C + 3 * cg;
#pragma unroll
      for (int a = 0; a < 9; ++a) x[a] = src[(a / 3) * D + a % 3];
      mixed_fibre<T>(x, y);
      int p = 0, w9 = 9, r = rg, c = cg;
#pragma unroll
      for (int j = 1; j < M; ++j, w9 *= 9, r /= 3, c /= 3) p += (3 * (r % 3) + (c % 3)) * w9;
      if constexpr (M == 1) {
        put(y, p);
      } else {
#pragma unroll
        for (int a = 0; a < 9; ++a) t[p + a] = y[a];
      }
    }
    if constexpr (M == 3) {
      __syncthreads();
      lds_digit<T, NF, 9>(t);
    }
    if constexpr (M > 1) {
      __syncthreads();
      for (int f = threadIdx.x; f < NF; f += MIXED_NT) {
        vec2<T> x[9], y[9];
        const int base = fibre_base<LST>(f);
#pragma unroll
        for (int a = 0; a < 9; ++a) x[a] = t[base + a * LST];
        mixed_fibre<T>(x, y);
        put(y, base);
      }
    }
  }
  if constexpr (REDUCE) block_sums_out(acc, part);
}

// Later pass: digits k .. k + ND - 1 (S = 9^k their lowest stride), J contiguous positions below them along
// (J divides S): tile q covers base + j + m S, j < J, m < 9^ND, base = (q mod (S / J)) J + (q div (S / J)) 9^ND S;
// LDS layout [m][j].  In place, or summed (REDUCE).
template <typename T, int ND, int J, bool REDUCE>
__global__ __launch_bounds__(MIXED_NT) void k_mixed_pass(vec2<T> *__restrict__ v, uint64_t n_tiles, uint64_t n_lo,
                                                          uint64_t S, double *part) {
  constexpr int P9 = ND == 1 ? 9 : ND == 2 ? 81 : 729;  // 9^ND
  constexpr int TILE = J * P9, NF = TILE / 9, LST = NF;
  __shared__ vec2<T> t[ND > 1 ? TILE : 1];
  double acc[3] = {0.0, 0.0, 0.0};
  for (uint64_t b = blockIdx.x; b < n_tiles; b += gridDim.x) {
    // consecutive tiles share the cache lines their segments straddle: keep them on one XCD's L2
    const uint64_t q = (uint64_t)xcd_tile((int64_t)b, (int64_t)n_tiles);
    vec2<T> *w = v + (q % n_lo) * J + (q / n_lo) * S * P9;
    auto at = [&](int e) -> vec2<T> * { return w + (e % J) + (uint64_t)(e / J) * S; };  // LDS position e
    auto put = [&](const vec2<T>(&y)[9], int base) {
      if constexpr (REDUCE) {
        fibre_sums<T>(y, acc);
      } else {
        vec2<T> *o = at(base);
#pragma unroll
        for (int a = 0; a < 9; ++a) o[(uint64_t)a * (LST / J) * S] = y[a];
      }
    };
    if constexpr (ND > 1) __syncthreads();
    for (int f = threadIdx.x; f < NF; f += MIXED_NT) {
      vec2<T> x[9], y[9];
      const int base = fibre_base<J>(f);
      const vec2<T> *src = at(base);
#pragma unroll
      for (int a = 0; a < 9; ++a) x[a] = src[(uint64_t)a * S];
      mixed_fibre<T>(x, y);
      if constexpr (ND == 1) {
        put(y, base);
      } else {
#pragma unroll
        for (int a = 0; a < 9; ++a) t[base + a * J] = y[a];
      }
    }
    if constexpr (ND == 3) {
      __syncthreads();
      lds_digit<T, NF, 9 * J>(t);
    }
    if constexpr (ND > 1) {
      __syncthreads();
      for (int f = threadIdx.x; f < NF; f += MIXED_NT) {
        vec2<T> x[9], y[9];
        const int base = fibre_base<LST>(f);
#pragma unroll
        for (int a = 0; a < 9; ++a) x[a] = t[base + a * LST];
        mixed_fibre<T>(x, y);
        put(y, base);
      }
    }
  }
  if constexpr (REDUCE) block_sums_out(acc, part);
}

__global__ __launch_bounds__(256) void k_mixed_total(const double *part, int nblk, int N, double *out) {
  __shared__ double red[3][256];
  for (int k = 0; k < 3; ++k) {
    double s = 0.0;
    for (int i = threadIdx.x; i < nblk; i += 256) s += part[i * 3 + k];
    red[k][threadIdx.x] = s;
  }
  __syncthreads();
  for (unsigned w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int k = 0; k < 3; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double D = pow(3.0, (double)N);
    out[0] = log2(red[0][0] / D);  // Eq. mana: log2 sum_u |W(u)|, W = Tr(rho A_u) / 3^N
    out[1] = red[1][0] / D;        // sum_u W(u) = Tr rho
    out[2] = red[2][0] / D;        // 3^N sum_u W(u)^2 = Tr rho^2
  }
}

// rho_A[i D_A + j] = sum_b psi[i + D_A b] conj(psi[j + D_A b]) (FP64 sums): the subsystem of the
// qutrits 0..n_a-1 (low digits); one block row of 256 columns j per thread block.
template <typename T>
__global__ __launch_bounds__(256) void k_reduced_density(const vec2<T> *psi, uint64_t DA, uint64_t DB, vec2<T> *rho) {
  const uint64_t i = blockIdx.y + ((uint64_t)blockIdx.z << 16);
  const uint64_t j = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= DA || j >= DA) return;
  double re = 0.0, im = 0.0;
  for (uint64_t b = 0; b < DB; ++b) {
    const vec2<T> p = psi[i + DA * b], q = psi[j + DA * b];
    // p conj(q)
    re = fma((double)p.x, (double)q.x, fma((double)p.y, (double)q.y, re));
    im = fma((double)p.y, (double)q.x, fma(-(double)p.x, (double)q.y, im));
  }
  vec2<T> o;
  o.x = (T)re;
  o.y = (T)im;
  rho[i * DA + j] = o;
}

static uint64_t pow_u(uint64_t b, int e) {
  uint64_t r = 1;
  while (e-- > 0) r *= b;
  return r;
}

// [partials][reordered vector 9^N values]
int mixed_workspace(int N, int dbl, size_t *bytes) {
  if (N < 1 || N > 10) return fail(E_SIZE, "mixed mana: n = %d outside [1, 10]", N);
  const uint64_t D = pow_u(3, N);
  *bytes = align256(MIXED_RED_BLOCKS * 3 * sizeof(double)) + align256(D * D * (dbl ? 16 : 8));
  return OK;
}

// One workgroup per tile, or a grid-stride loop over `cap` workgroups (a multiple of 8, so that the
// tiles a workgroup takes stay on its XCD's share).
static unsigned grid_of(uint64_t tiles, uint64_t cap) { return (unsigned)(tiles < cap ? tiles : cap); }

template <typename T, int M>
static void launch_first(bool reduce, const void *rho, uint64_t D, uint64_t tiles, vec2<T> *v, double *part,
                         unsigned *red_grid, hipStream_t st) {
  ProfScope prof(reduce ? "mixed_last" : "mixed_first", st);
  if (reduce) {
    *red_grid = grid_of(tiles, MIXED_RED_BLOCKS);
    hipLaunchKernelGGL((k_mixed_first<T, M, true>), dim3(*red_grid), dim3(MIXED_NT), 0, st, (const vec2<T> *)rho, D,
                       tiles, v, part);
  } else {
    hipLaunchKernelGGL((k_mixed_first<T, M, false>), dim3(grid_of(tiles, 1u << 20)), dim3(MIXED_NT), 0, st,
                       (const vec2<T> *)rho, D, tiles, v, part);
  }
}

template <typename T, int ND, int J>
static void launch_pass(bool reduce, uint64_t V, int k, vec2<T> *v, double *part, unsigned *red_grid, hipStream_t st) {
  const uint64_t S = pow_u(9, k), tiles = V / (pow_u(9, ND) * J);
  ProfScope prof(reduce ? "mixed_last" : "mixed_pass", st);
  if (reduce) {
    *red_grid = grid_of(tiles, MIXED_RED_BLOCKS);
    hipLaunchKernelGGL((k_mixed_pass<T, ND, J, true>), dim3(*red_grid), dim3(MIXED_NT), 0, st, v, tiles, S / J, S, part);
  } else {
    hipLaunchKernelGGL((k_mixed_pass<T, ND, J, false>), dim3(grid_of(tiles, 1u << 20)), dim3(MIXED_NT), 0, st, v, tiles,
                       S / J, S, part);
  }
}

template <typename T>
static int mixed_t(int N, const void *rho, double *out, void *ws, hipStream_t st) {
  const uint64_t D = pow_u(3, N), V = D * D;
  char *w = (char *)ws;
  double *part = (double *)w;
  vec2<T> *v = (vec2<T> *)(w + align256(MIXED_RED_BLOCKS * 3 * sizeof(double)));
  const int M = N < 3 ? N : 3;
  const uint64_t tiles_a = V / pow_u(9, M);
  unsigned red_grid = 0;
  if (M == 1) launch_first<T, 1>(N == M, rho, D, tiles_a, v, part, &red_grid, st);
  else if (M == 2) launch_first<T, 2>(N == M, rho, D, tiles_a, v, part, &red_grid, st);
  else launch_first<T, 3>(N == M, rho, D, tiles_a, v, part, &red_grid, st);
  // The remaining digits in as few passes as three digits each allow (four left: two and two).  Three
  // digits carry 9 positions (144 / 72-byte segments, 105 / 52 KB of LDS; with 3 positions N = 9 took 7.1
  // instead of 6.7 ms in complex128 and 4.8 instead of 3.6 in complex64).
  for (int k = M; k < N;) {
    const int left = N - k, nd = left == 4 ? 2 : left < 3 ? left : 3;
    const bool last = left == nd;
    if (nd == 3) launch_pass<T, 3, 9>(last, V, k, v, part, &red_grid, st);
    else if (nd == 2) launch_pass<T, 2, 27>(last, V, k, v, part, &red_grid, st);
    else launch_pass<T, 1, 243>(last, V, k, v, part, &red_grid, st);
    k += nd;
  }
  hipLaunchKernelGGL(k_mixed_total, dim3(1), dim3(256), 0, st, (const double *)part, (int)red_grid, N, out);
  return hipPeekAtLastError() == hipSuccess ? OK : fail(E_HIP, "mixed mana launch: %s", hipGetErrorString(hipGetLastError()));
}

int mixed_launch(int N, int dbl, const void *rho, double *out, void *ws, hipStream_t st) {
  return dbl ? mixed_t<double>(N, rho, out, ws, st) : mixed_t<float>(N, rho, out, ws, st);
}

int reduced_density_launch(int N, int NA, int dbl, const void *psi, void *rho, hipStream_t st) {
  const uint64_t DA = pow_u(3, NA), DB = pow_u(3, N - NA);
  const dim3 grid((unsigned)((DA + 255) / 256), (unsigned)(DA < 65536 ? DA : 65536), (unsigned)((DA + 65535) >> 16));
  ProfScope prof("reduced_density", st);
  if (dbl) hipLaunchKernelGGL(k_reduced_density<double>, grid, dim3(256), 0, st, (const double2 *)psi, DA, DB, (double2 *)rho);
  else hipLaunchKernelGGL(k_reduced_density<float>, grid, dim3(256), 0, st, (const float2 *)psi, DA, DB, (float2 *)rho);
  return hipPeekAtLastError() == hipSuccess ? OK : fail(E_HIP, "reduced density launch: %s", hipGetErrorString(hipGetLastError()));
}

}  // namespace hm
