// hm_tile.h -- device building blocks shared by the gfx950 kernels of libhmag.
//
// A "tile" is 2^TB complex values held by NT = 2^LT threads of one workgroup, R = 2^RB values per
// thread in registers.  A round layout with start S places the register index bits at tile-index
// positions [S, S+RB) and the thread index bits at the remaining positions, in order:
//     idx = (tau & (2^S - 1)) | (rho << S) | ((tau >> S) << (S + RB)).
// Butterflies act on register bits; moving to a layout with another S is one pass through LDS.
// LDS addresses are padded with one slot per R values (phys = idx + idx/R): for every layout above,
// any 32 consecutive lanes (8-byte values) or 16 lanes (16-byte values) then hit distinct banks, and
// the per-register part of the address stays a compile-time constant.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hm_internal.h"

namespace hm {

template <typename T> struct vec2_of;
template <> struct vec2_of<float> { using type = float2; };
template <> struct vec2_of<double> { using type = double2; };
template <typename T> using vec2 = typename vec2_of<T>::type;

__host__ __device__ constexpr int ilog2c(int x) { return x <= 1 ? 0 : 1 + ilog2c(x >> 1); }

// Fused multiply-add in the precision of T (the plain builtin would promote floats to double).
__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Load / store element idx of an array given by a uniform base pointer and a 32-bit element index
// (the byte offset stays in one 32-bit register; every buffer here is smaller than 4 GiB).
template <typename V>
__device__ __forceinline__ V ld32(const V *base, uint32_t idx) {
  return *reinterpret_cast<const V *>(reinterpret_cast<const char *>(base) + (uint32_t)(idx * (uint32_t)sizeof(V)));
}
template <typename V>
__device__ __forceinline__ void st32(V *base, uint32_t idx, V v) {
  *reinterpret_cast<V *>(reinterpret_cast<char *>(base) + (uint32_t)(idx * (uint32_t)sizeof(V))) = v;
}

// Raw buffer view of n_bytes of global memory (gfx9 buffer descriptor: no stride, no format
// conversion).  Loads through it take a per-lane byte offset and a uniform byte offset (an SGPR), so
// an address that is a per-thread part plus a wave-uniform part costs no vector instruction; an
// offset past n_bytes reads zero.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_view(const void *p, uint32_t n_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)n_bytes, 0x00020000);
}
__device__ __forceinline__ float2 buf_ld(float2 *, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)voff, (int)soff, 0));
}
__device__ __forceinline__ double2 buf_ld(double2 *, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, (int)soff, 0));
}
// A pointer that is the same in every lane, in scalar registers (a buffer view of one held in vector
// registers would be looped over its distinct values).
template <typename V>
__device__ __forceinline__ const V *uniform_ptr(const V *p) {
  const uint64_t u = (uint64_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return (const V *)(((uint64_t)hi << 32) | lo);
}

template <int S, int RB>
__device__ __forceinline__ uint32_t lay(uint32_t tau, uint32_t rho) {
  return (tau & ((1u << S) - 1u)) | (rho << S) | ((tau >> S) << (S + RB));
}

template <int RB>
__host__ __device__ __forceinline__ constexpr uint32_t ldspad(uint32_t idx) { return idx + (idx >> RB); }

// lay<S, RB>(tau, rho) split into its thread part and its register part.  The two occupy disjoint
// bit fields, so lay = base + off and ldspad(lay) = ldspad(base) + ldspad(off): the register part
// is a compile-time constant that folds into the immediate offset of the LDS instruction.
template <int S, int RB>
__device__ __forceinline__ uint32_t lay_base(uint32_t tau) {
  return (tau & ((1u << S) - 1u)) | ((tau >> S) << (S + RB));
}
template <int S, int RB>
__host__ __device__ __forceinline__ constexpr uint32_t lay_off(int rho) { return (uint32_t)rho << S; }

// insert a zero bit at position j: bits >= j move up by one.
__device__ __forceinline__ uint64_t ins0(uint64_t c, int j) {
  uint64_t lo = c & ((1ull << j) - 1ull);
  return lo | ((c - lo) << 1);
}
__device__ __forceinline__ uint32_t ins0_32(uint32_t c, int j) {
  uint32_t lo = c & ((1u << j) - 1u);
  return lo | ((c - lo) << 1);
}

// Unnormalised Walsh-Hadamard butterflies over register bits [K0, K1).
template <typename T, int R, int K0, int K1>
__device__ __forceinline__ void wht_regs(T (&re)[R], T (&im)[R]) {
#pragma unroll
  for (int k = K0; k < K1; ++k) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      if (!((i >> k) & 1)) {
        const int j = i | (1 << k);
        T a = re[i], b = re[j];
        re[i] = a + b;
        re[j] = a - b;
        a = im[i];
        b = im[j];
        im[i] = a + b;
        im[j] = a - b;
      }
    }
  }
}

// Walsh-Hadamard stages on the KB <= 2 lowest tile-index bits where they sit in the lowest lane bits,
// without LDS: x + s p with p the partner's value (one DPP quad permutation per word) and s = +1 / -1 by
// the lane's bit, the same rounding as a butterfly.  The lanes with s = -1 hold the negative of the
// transform, a sign that depends on the index only: sums of |x|^2q and stages along other bits do not
// see it.
template <int CTRL>
__device__ __forceinline__ float lane_move(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double lane_move(double x) {
  const uint64_t u = __builtin_bit_cast(uint64_t, x);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <typename T, int R, int CTRL>
__device__ __forceinline__ void lane_move_all(vec2<T> (&v)[R]) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    v[r].x = lane_move<CTRL>(v[r].x);
    v[r].y = lane_move<CTRL>(v[r].y);
  }
}
template <typename T, int R, int CTRL>
__device__ __forceinline__ void lane_stage(T (&re)[R], T (&im)[R], T s) {
#pragma unroll
  for (int r = 0; r < R; ++r) re[r] = fmaT(lane_move<CTRL>(re[r]), s, re[r]);
#pragma unroll
  for (int r = 0; r < R; ++r) im[r] = fmaT(lane_move<CTRL>(im[r]), s, im[r]);
}
template <typename T, int R, int KB>
__device__ __forceinline__ void wht_lanes(T (&re)[R], T (&im)[R], uint32_t tau) {
  static_assert(KB <= 2, "quad permutations");
  if constexpr (KB >= 1) lane_stage<T, R, 0xB1>(re, im, (tau & 1u) ? T(-1) : T(1));  // quad_perm 1,0,3,2
  if constexpr (KB >= 2) lane_stage<T, R, 0x4E>(re, im, (tau & 2u) ? T(-1) : T(1));  // quad_perm 2,3,0,1
}

// Moving a tile from layout SA to layout SB through LDS.  In a layout with S <= 6 the thread bits
// above the lane (tau >> 6) are the top bits of the tile index, so a wave holds the contiguous index
// range [w 2^(6+RB), (w+1) 2^(6+RB)), which is also its own stretch of the LDS buffer:
//   * SA <= 6 and SB <= 6: the values never leave the wave.  LDS instructions of one wave execute in
//     order, so no workgroup barrier is needed, only that the compiler keeps the order (wave_order).
//   * otherwise a barrier separates the writes from the reads.  One before the writes is needed only
//     when they go to other waves' stretches (SA > 6): consecutive moves chain (the layout read last is
//     the layout written next), so for SA <= 6 every wave last read its own stretch.
// So a move orders the traffic of its own buffer only, and only along a chain of moves.  A caller may not use it as
// a barrier for other LDS arrays, and a loop whose moves end in a layout other than the one written first puts a
// barrier between its iterations or asserts that both have S <= 6.
// Without the barriers the waves of a workgroup drift apart and one wave's LDS traffic overlaps
// another's butterflies (barriers per FP32 row tile of 2^15 values: 8 -> 4, of 2^11 values: 8 -> 0).
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__host__ __device__ constexpr bool in_wave(int SA, int SB) { return SA <= 6 && SB <= 6; }
template <bool BARRIER>
__device__ __forceinline__ void lds_order() {
  if constexpr (BARRIER) __syncthreads();
  else wave_order();
}

// All NT threads must call it.  Threads with act == false (padding threads of a block larger than the
// tile) skip the LDS traffic.
template <typename T, int R, int RB, int SA, int SB>
__device__ __forceinline__ void relayout(T (&re)[R], T (&im)[R], vec2<T> *lds, uint32_t tau, bool act = true) {
  const uint32_t ba = ldspad<RB>(lay_base<SA, RB>(tau));
  const uint32_t bb = ldspad<RB>(lay_base<SB, RB>(tau));
  lds_order<(SA > 6)>();  // earlier readers of the written stretch are done
  if (act) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      vec2<T> v;
      v.x = re[r];
      v.y = im[r];
      lds[ba + ldspad<RB>(lay_off<SA, RB>(r))] = v;
    }
  }
  lds_order<!in_wave(SA, SB)>();
  if (act) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      vec2<T> v = lds[bb + ldspad<RB>(lay_off<SB, RB>(r))];
      re[r] = v.x;
      im[r] = v.y;
    }
  }
}

// Same as relayout, for tiles too large to stage both components at once: the real parts, then the
// imaginary parts, go through a scalar LDS buffer of 2^TB (+ padding) values.  SECOND: the buffer was
// just read in layout SB (the other component), possibly by other waves.
template <typename T, int R, int RB, int SA, int SB, bool SECOND>
__device__ __forceinline__ void relayout_one(T (&v)[R], T *lds, uint32_t tau) {
  const uint32_t ba = ldspad<RB>(lay_base<SA, RB>(tau));
  const uint32_t bb = ldspad<RB>(lay_base<SB, RB>(tau));
  lds_order<(SECOND ? !in_wave(SA, SB) : SA > 6)>();
#pragma unroll
  for (int r = 0; r < R; ++r) lds[ba + ldspad<RB>(lay_off<SA, RB>(r))] = v[r];
  lds_order<!in_wave(SA, SB)>();
#pragma unroll
  for (int r = 0; r < R; ++r) v[r] = lds[bb + ldspad<RB>(lay_off<SB, RB>(r))];
}
template <typename T, int R, int RB, int SA, int SB>
__device__ __forceinline__ void relayout_split(T (&re)[R], T (&im)[R], T *lds, uint32_t tau) {
  relayout_one<T, R, RB, SA, SB, false>(re, lds, tau);
  relayout_one<T, R, RB, SA, SB, true>(im, lds, tau);
}

// Workgroups are dispatched round-robin over the 8 XCDs (workgroup b runs on XCD b mod 8).  This
// maps b in [0, n) to a tile so that XCD k takes the k-th contiguous share of [0, n) (a bijection
// for every n; shares differ by at most one tile): neighbouring tiles, which share cache lines of
// the exchange rows, are then read through the same L2.
__device__ __forceinline__ int64_t xcd_tile(int64_t b, int64_t n) {
  const int64_t k = b & 7, m = b >> 3;
  int64_t start = 0;
  for (int64_t i = 0; i < k; ++i) start += (n - i + 7) >> 3;
  return start + m;
}

// Deterministic sum over aligned segments of SEG consecutive threads (SEG a power of two dividing
// NT).  Returns the segment total in the first thread of each segment (other threads: partial).
// lds must hold NT/64 doubles per value.
template <int NT, int SEG>
__device__ __forceinline__ double seg_sum(double v, double *lds, uint32_t tau) {
  constexpr int WSEG = SEG < 64 ? SEG : 64;
#pragma unroll
  for (int off = 1; off < WSEG; off <<= 1) v += __shfl_xor(v, off, 64);
  if constexpr (SEG > 64) {
    constexpr int NW = SEG / 64;
    __syncthreads();
    if ((tau & 63u) == 0) lds[tau >> 6] = v;
    __syncthreads();
    if ((tau & (SEG - 1)) == 0) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += lds[(tau >> 6) + w];
      v = s;
    }
  }
  return v;
}

// Arguments describing the Renyi indices of one call (passed by value to kernels).
struct QArgs {
  int nq;
  double q[HM_MAX_Q];
};

// Sums over the 2R real values x of a thread for the reduction of Algorithm 2, with t = x^2 = |<P>|^2
// (folded form): kind 0 is sum t, otherwise sum t^q (q == 1: sum t log2 t).  The kind is uniform, so one
// q at a time runs through the registers; the kinds that call a math function handle C registers per pass
// of a loop that rotates the register arrays (back in place at its end): unrolled over all 2R values they
// made kernels of 70 kB of code, which do not stay in the instruction cache.
enum QKind { Q_NORM = 0, Q_SHANNON, Q_TWO, Q_THREE, Q_FOUR, Q_POW };
__device__ __forceinline__ QKind q_kind(double q) {
  return q == 1.0 ? Q_SHANNON : q == 2.0 ? Q_TWO : q == 3.0 ? Q_THREE : q == 4.0 ? Q_FOUR : Q_POW;
}
// FENCE > 0: a scheduling fence after every FENCE registers (bounds the temporaries in flight).
template <typename T, int R, int FENCE = 0, typename F>
__device__ __forceinline__ void each_real(T (&re)[R], T (&im)[R], F f) {
#pragma unroll
  for (int r = 0; r < R; ++r) {
    f(re[r]);
    f(im[r]);
    if constexpr (FENCE > 0) {
      if ((r + 1) % FENCE == 0) __builtin_amdgcn_sched_barrier(0);
    }
  }
}
template <typename T, int R, int C, int FENCE, typename F>
__device__ __forceinline__ void each_real_rotating(T (&re)[R], T (&im)[R], F f) {
  static_assert(R % C == 0, "whole passes");
  if constexpr (C == R) {
    each_real<T, R, FENCE>(re, im, f);
  } else {
#pragma unroll 1
    for (int p = 0; p < R / C; ++p) {
#pragma unroll
      for (int r = 0; r < C; ++r) {
        f(re[r]);
        f(im[r]);
        if ((r + 1) % FENCE == 0) __builtin_amdgcn_sched_barrier(0);
      }
      T hr[C], hi[C];
#pragma unroll
      for (int r = 0; r < C; ++r) {
        hr[r] = re[r];
        hi[r] = im[r];
      }
#pragma unroll
      for (int r = 0; r + C < R; ++r) {
        re[r] = re[r + C];
        im[r] = im[r + C];
      }
#pragma unroll
      for (int r = 0; r < C; ++r) {
        re[R - C + r] = hr[r];
        im[R - C + r] = hi[r];
      }
    }
  }
}
template <typename T, int R, bool POW>
__device__ __forceinline__ T sum_kind(T (&re)[R], T (&im)[R], QKind kind, double q) {
#pragma clang fp contract(off)
  T a = T(0);
  switch (kind) {
    case Q_NORM: each_real(re, im, [&](T x) { a += x * x; }); break;
    case Q_TWO: each_real(re, im, [&](T x) { const T t = x * x; a += t * t; }); break;
    case Q_THREE: each_real(re, im, [&](T x) { const T t = x * x; a += t * t * t; }); break;
    case Q_SHANNON: {
      // the FP32 log2 is a few instructions, the FP64 one about 80
      constexpr int C = sizeof(T) == 4 || R < 4 ? R : 4;
      each_real_rotating<T, R, C, 2>(re, im, [&](T x) {
        const T t = x * x;
        a += t > T(0) ? t * (T)log2(t) : T(0);
      });
      break;
    }
    case Q_FOUR: each_real(re, im, [&](T x) { const T t = x * x, t2 = t * t; a += t2 * t2; }); break;
    default:
      if constexpr (POW) {
        // FP64: no branch around pow, so that the two chains of a pass step overlap (8 indices, N = 14:
        // 40.4 -> 13.0 ms; N = 8 134 -> 122 us); FP32 keeps it (25.0 against 26.9 ms at N = 15, 187 against
        // 192 us at N = 8).
        constexpr int C = sizeof(T) == 4 ? 8 : 4;
        each_real_rotating<T, R, (R < C ? R : C), 1>(re, im, [&](T x) {
          const T t = x * x;
          if constexpr (sizeof(T) == 8) {
            T v = pow(t, (T)q);
            asm volatile("" : "+v"(v));
            a += t > T(0) ? v : T(0);
          } else {
            a += t > T(0) ? (T)pow(t, (T)q) : T(0);
          }
        });
      }
      break;
  }
  return a;
}

// The sums of a tile's segments of SEG threads (seg_sum): out(k, s) is called by every thread for k = 0 ..
// nacc - 1 in turn and gets the segment's total in the segment's first thread.  QM == 2: q = (2); QM == 1:
// every q is 1, 2, 3 or 4 (pow's temporaries would not fit beside the values of the largest tiles);
// QM == 0: any q.  Measured for q = (1, 2, 3) on MI355X against all kinds unrolled with one accumulator
// per q: complex64 N = 13 142 -> 78 us, N = 16 11.3 -> 6.3 ms; complex128 N = 15 15.6 -> 10.5 ms.
// Eight other indices: complex128 N = 8 163 -> 122 us, N = 14 22.5 -> 13.1 ms; complex64 N = 8 204 -> 189 us,
// N = 13 1725 -> 1713 us, N = 15 25.8 -> 24.9 ms.
template <typename T, int R, int NT, int SEG, int QM, typename F>
__device__ __forceinline__ void tile_sums(T (&re)[R], T (&im)[R], const QArgs &qa, double *red, uint32_t tau, F out) {
  if constexpr (QM == 2) {
    T a0 = T(0), a1 = T(0);
    each_real(re, im, [&](T x) {
      const T t = x * x;
      a0 += t;
      a1 = fmaT(t, t, a1);
    });
    const double s0 = seg_sum<NT, SEG>((double)a0, red, tau), s1 = seg_sum<NT, SEG>((double)a1, red, tau);
    out(0, s0);
    out(1, s1);
  } else {
#pragma unroll 1
    for (int k = 0; k <= qa.nq; ++k) {
      const double q = k ? qa.q[k - 1] : 1.0;
      // the values are the same for every k: keep the compiler from holding their squares across the loop
#pragma unroll
      for (int r = 0; r < R; ++r) asm volatile("" : "+v"(re[r]), "+v"(im[r]));
      const T a = sum_kind<T, R, QM == 0>(re, im, k ? q_kind(q) : Q_NORM, q);
      out(k, seg_sum<NT, SEG>((double)a, red, tau));
    }
  }
}

// Scale folded per-shift sum k to the unfolded convention: a != 0 shifts were folded on one bit,
// |chi|^2 = f t with f = 4; the a == 0 shift is folded without the factor (f = 1).  s0 is the folded
// sum 0.
__device__ __forceinline__ double unfold_sum(int k, double s, double s0, const QArgs &qa, bool a_is_zero) {
  if (a_is_zero) return s;
  const double f = 4.0;
  if (k == 0) return f * s;
  const double q = qa.q[k - 1];
  return q == 1.0 ? f * (s + 2.0 * s0)  // f (sum t log2 t + log2(f) sum t)
                  : exp2(2.0 * q) * s;
}
__device__ __forceinline__ void unfold_scale(double *s, int nacc, const QArgs &qa, bool a_is_zero) {
  const double s0 = s[0];
  for (int k = 0; k < nacc; ++k) s[k] = unfold_sum(k, s[k], s0, qa, a_is_zero);
}

}  // namespace hm
