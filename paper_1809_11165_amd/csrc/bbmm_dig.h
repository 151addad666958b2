// What the two products on the 8-bit matrix pipe share (kernels_dig.hip, kernels_words.hip): digits of entries and
// blocks, the rule for blocks that suit them, and the way from accumulators to partial results.
#pragma once

#include "bbmm_dev.h"

#include <type_traits>

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) char lds_char;
typedef const __attribute__((address_space(3))) i32x4* lds_i32x4;
typedef const __attribute__((address_space(3))) f32x4* lds_f32x4;

namespace {

// A[m = lane%16][k = 16 (lane/16) + byte], B[k][n = lane%16]; register r of the result holds
// C[m = 4 (lane/16) + r][n = lane%16] (layout checked against A B on the device).
__device__ inline i32x4 mfma_i8(i32x4 a, i32x4 b, i32x4 c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0); }

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

constexpr int kDigits = 0x00808080;
// Scale of the entries: below 2^31 less the largest balanced lower digits, and a multiple of 2^23, so that it is exact in fp32.
constexpr float kX = 2055208960.f;
// Adding kDigits to the scaled entry rounds it to a whole number, to nearest and in the one rounding of the fma (the
// sum is above 2^23), and is the addition that the digits need.  (Adding 1/2 and truncating rounds twice: entries
// came out half a unit high, or 4e-8 of themselves below 2^-8; so does any rounding of ties to one side, since the
// product lies on a grid of halves, quarters, ...)  An entry keeps 23 bits at least from 2^-8 up.
constexpr float kRound = (float)kDigits;

// Scale exponent of a column from the largest high word of |D|: 2^e > max |D|; E == 0: the column is
// zero (to fp64 underflow) and has no digits.
__device__ inline int dig_exponent(unsigned hi) { return (int)(hi >> 20) - 1022; }

// Whether a block suits the digits, for a caller who sees the product itself.  Fixed point leaves an error of 1.4e-10 of the
// outputscale times the norm of the block's column in every row of the product: nothing beside the rounding of the entries
// where the column's entries are of a size, and too much in rows that meet only small entries of K or of the column.
// So at most n / 128 entries of a column may lie below 2^-12 of its largest power of two, and n / 16384 + 4 below 2^-20
// (a column of 200 000 normal values has 2e-3 n and about one); everything must be finite.
__device__ inline bool dig_dense(const DevState* st, const unsigned* __restrict__ counts, int n) {
  int lane = threadIdx.x & 63, q = lane & (BBMM_MAXC - 1);   // lanes 0..31: small entries, 32..63: tiny ones
  unsigned sum = 0, hi = st->dmax[q];
#pragma unroll
  for (int r = 0; r < kDigCountRows; ++r) sum += counts[r * 2 * BBMM_MAXC + lane];
  bool bad = hi >= 0x7ff00000u || (hi != 0u && sum > (unsigned)(lane < BBMM_MAXC ? n / 128 : n / 16384 + 4));
  return !__any(bad) && st->xbad == 0;
}

// What a block column with a non-finite entry adds to its (zero) digits' product: the sum of K D for K > 0; an X that
// is none for the digits (xbad) makes everything NaN.
__device__ __forceinline__ double dig_special(unsigned hi, int flag, int xbad) {
  double x = 0.0;
  if (hi >= 0x7ff00000u) x = (flag & 4) || flag == 3 ? __builtin_nan("") : (flag == 1 ? __builtin_inf() : -__builtin_inf());
  return xbad ? __builtin_nan("") : x;
}

// Sum t = sum_w 256^-w acc_w -> partial result of the product for block column q (inv_x: entries per unit).
__device__ __forceinline__ double dig_value(double t, double inv_x, int q, int xbad, const DevState* __restrict__ st) {
  unsigned hi = st->dmax[q];
  return ldexp(t * inv_x, dig_exponent(hi) + 18) + dig_special(hi, st->dflag[q], xbad);
}

// Accumulators of 16 output columns -> partial results.  acc[q][r]: lane (jc, g) holds pair
// 16 q + 4 g + r, i.e. right-hand side 2 q + g / 2, weight 4 (g % 2) + r, of output column jc.  T: LDS,
// 16 x (LD + 1) doubles of the wave.  q0: block column of the first.
template <int NG, int LD>
__device__ __forceinline__ void dig_store(const i32x4 (&acc)[NG], double inv_x, double* __restrict__ T, int jc, int g,
                                          const DevState* __restrict__ st, double* __restrict__ vrow, int q0 = 0) {
  constexpr int TP = LD + 1;
#pragma unroll
  for (int q = 0; q < LD / 2; ++q) {
    double t = 0.0;
    if (q < NG) {
      const i32x4& a = acc[q < NG ? q : 0];
      t = (double)a[0] + 0x1p-8 * (double)a[1] + 0x1p-16 * (double)a[2] + 0x1p-24 * (double)a[3];
      if (g & 1) t *= 0x1p-32;
      t += __shfl_xor(t, 16, 64);
    }
    if (!(g & 1)) T[jc * TP + 2 * q + (g >> 1)] = t;
  }
  __builtin_amdgcn_wave_barrier();
  int xbad = st->xbad;
#pragma unroll
  for (int nq = 0; nq < LD / 16; ++nq) {
    f64x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      int q = 16 * nq + 4 * r + g;
      v[r] = dig_value(T[jc * TP + q], inv_x, q0 + q, xbad, st);
    }
    *(f64x4*)(vrow + nq * 16 + g * 4) = v;
  }
  __builtin_amdgcn_wave_barrier();
}

// s_waitcnt vmcnt(N) alone
template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

}  // namespace
