// hm_sre_dev.h -- device pieces of the qubit SRE path shared by the forward and adjoint kernels:
// the round schedule of the row pass and the folded product step (see hm_sre.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hm_tile.h"

namespace hm {

__host__ __device__ constexpr int rp_S(int NL, int RB, int k) { return NL - RB * (k + 1) > 0 ? NL - RB * (k + 1) : 0; }
__host__ __device__ constexpr int rp_H(int NL, int RB, int k) { return RB < NL - RB * k ? RB : NL - RB * k; }

template <typename T>
__device__ __forceinline__ void cmul_conj(vec2<T> y, vec2<T> x, T &re, T &im) {
  // conj(y) * x
  re = fmaT(y.x, x.x, y.y * x.y);
  im = fmaT(y.x, x.y, -(y.y * x.x));
}

// Product step of the row pass: for the thread's R values (row-task ch, thread part tlo, register
// r at row position tlo + (r << S0)) form the folded vector u of shift a (see the file comment).
// CH bounds how many registers' loads may be in flight: a scheduling fence after every CH values
// keeps the compiler from hoisting all 2R gathers (register pressure decides occupancy).
//
// Row-tasks of whole waves (S0 >= 6; a, ch and the state the same for all lanes of a wave): the element
// index of every gather is a per-lane part (row and thread bits, the same for all registers) plus a
// part that depends on the register and the shift only.  The loads take the first as their lane offset
// and the second as their scalar offset, so the 2R addresses cost no vector instruction (as global loads
// two each, 4 of about 46 per folded value).  Shorter rows (several per wave) measured slower that way
// (rows of 2^9 in the two-pass row pass: 56 -> 61 us per 2^25 values) and keep the global loads.
template <typename T, int RB, int NL, int CH = (1 << RB)>
__device__ __forceinline__ void sre_product(const vec2<T> *__restrict__ psi, uint32_t half, uint64_t a, uint64_t ch,
                                            uint32_t tlo, bool active, T (&re)[1 << RB], T (&im)[1 << RB]) {
  constexpr int R = 1 << RB;
  constexpr int S0 = NL - RB;
  constexpr int SEG = 1 << S0;
  if (!active) {
#pragma unroll
    for (int r = 0; r < R; ++r) re[r] = im[r] = T(0);
  } else if (a == 0) {
    // a = 0: fold on the top qubit; u_c = (r0 + r1) + i (r0 - r1).
    const uint32_t cb = ((uint32_t)ch << NL) | tlo;
    const vec2<T> *p1b = psi + half;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t c = cb + ((uint32_t)r << S0);
      const vec2<T> p0 = ld32(psi, c), p1 = ld32(p1b, c);
      const T r0 = fmaT(p0.x, p0.x, p0.y * p0.y);
      const T r1 = fmaT(p1.x, p1.x, p1.y * p1.y);
      re[r] = r0 + r1;
      im[r] = r0 - r1;
      if constexpr (CH < R) {
        if ((r + 1) % CH == 0) __builtin_amdgcn_sched_barrier(0);
      }
    }
  } else if constexpr (S0 >= 6) {
    // Fold bit j is inserted into the row index (j >= NL), the register bits (S0 <= j < NL: register
    // part ins0(r, j - S0)) or the thread bits (j < S0: the register bits move up by one, ins0(r, 0) = 2r).
    constexpr uint32_t VB = sizeof(vec2<T>);
    const uint32_t a32 = (uint32_t)a;  // below 2^26
    const int j = 31 - __builtin_clz(a32);
    const uint32_t xr = j >= NL ? ins0_32((uint32_t)ch, j - NL) : (uint32_t)ch << 1;
    const uint32_t yr = j >= NL ? xr ^ (a32 >> NL) : xr;
    const uint32_t xt = j >= S0 ? tlo : ins0_32(tlo, j);
    const uint32_t yt = xt ^ (a32 & (uint32_t)(SEG - 1));
    const int jj = j < S0 ? 0 : j >= NL ? RB : j - S0;
    const uint32_t lomask = (1u << jj) - 1u, amid = (a32 >> S0) & (uint32_t)(R - 1);
    const uint32_t vx = ((xr << NL) + xt) * VB, vy = ((yr << NL) + yt) * VB;
    const __amdgpu_buffer_rsrc_t rs = buf_view(uniform_ptr(psi), half * 2u * VB);
    // two groups of G registers in flight: group g + 1 is requested before the products wait for group g
    constexpr int G = R < 4 ? R : 4, NG = R / G;
    vec2<T> px[2][G], py[2][G];
    auto request = [&](int g) {
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const uint32_t r = (uint32_t)(g * G + i);
        const uint32_t e = 2u * r - (r & lomask);  // ins0(r, jj)
        px[g & 1][i] = buf_ld((vec2<T> *)nullptr, rs, vx, (e << S0) * VB);
        py[g & 1][i] = buf_ld((vec2<T> *)nullptr, rs, vy, ((e ^ amid) << S0) * VB);
      }
    };
    request(0);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g + 1 < NG) request(g + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < G; ++i) cmul_conj<T>(py[g & 1][i], px[g & 1][i], re[g * G + i], im[g * G + i]);
      __builtin_amdgcn_sched_barrier(0);
    }
  } else {
    const int j = 63 - __builtin_clzll(a);
    if (j >= NL) {
      // fold bit inside the row index: columns are untouched, rows map c_h -> insert0(c_h, j - NL)
      const uint32_t xr = ins0_32((uint32_t)ch, j - NL);
      const uint32_t yr = xr ^ (uint32_t)(a >> NL);
      const uint32_t alo = (uint32_t)a & (SEG - 1);
      const uint32_t amid = ((uint32_t)(a >> S0)) & (R - 1);
      const uint32_t xb = (xr << NL) | tlo;
      const uint32_t yb = (yr << NL) | (tlo ^ alo);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const vec2<T> px = ld32(psi, xb + ((uint32_t)r << S0));
        const vec2<T> py = ld32(psi, yb + ((uint32_t)(r ^ amid) << S0));
        cmul_conj<T>(py, px, re[r], im[r]);
        if constexpr (CH < R) {
          if ((r + 1) % CH == 0) __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else if (j >= S0) {
      // fold bit among the register bits of the first round
      const uint32_t base = (uint32_t)ch << (NL + 1);
      const int jj = j - S0;
      const uint32_t alo = (uint32_t)a & (SEG - 1);
      const uint32_t ahi = (uint32_t)(a >> S0);
      const uint32_t xb = base | tlo;
      const uint32_t yb = base | (tlo ^ alo);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t e = ins0_32((uint32_t)r, jj);
        const vec2<T> px = ld32(psi, xb + (e << S0));
        const vec2<T> py = ld32(psi, yb + ((e ^ ahi) << S0));
        cmul_conj<T>(py, px, re[r], im[r]);
        if constexpr (CH < R) {
          if ((r + 1) % CH == 0) __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
      // small shifts (a < 2^S0): generic index arithmetic
      const uint32_t base = (uint32_t)ch << (NL + 1);
      const uint32_t a32 = (uint32_t)a;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const uint32_t c = tlo | ((uint32_t)r << S0);
        const uint32_t x = base | ins0_32(c, j);
        const vec2<T> px = ld32(psi, x);
        const vec2<T> py = ld32(psi, x ^ a32);
        cmul_conj<T>(py, px, re[r], im[r]);
        if constexpr (CH < R) {
          if ((r + 1) % CH == 0) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

}

// Adjoint seeds: every real value x becomes |k x|^{2q-2} x (k = 2 for a != 0, 1 for a = 0).  q = 3 has a form
// of its own (with pow for every value the gradient of M_3 took three times that of M_2); other q call
// pow, two registers per pass of a rotating loop.
template <typename T, int R, bool Q2>
__device__ __forceinline__ void adjoint_seeds(T (&re)[R], T (&im)[R], T k, double q) {
  if (Q2) {
    each_real(re, im, [&](T &x) { x = (k * k) * (x * x) * x; });
  } else if (q == 3.0) {
    each_real(re, im, [&](T &x) {
      const T t = (k * k) * (x * x);
      x = t * t * x;
    });
  } else {
    each_real_rotating<T, R, (R < 2 ? R : 2), 1>(re, im, [&](T &x) {
      const T ax = fabs(k * x);
      x = ax > T(0) ? (T)pow(ax, (T)(2.0 * q - 2.0)) * x : T(0);
    });
  }
}

}  // namespace hm
