// Two-way f16 split of fp32 operands for the f16 matrix instructions of gfx950.
//
// A float a, times a power of two, is taken as h + m with h = f16(a) and m = f16(a - h), m kept times 2^11 so that both have the
// exponents of the operand (the scheme of Ootomo and Yokota, "Recovering single precision accuracy from Tensor Cores while
// surpassing the FP32 theoretical peak performance", 2022): 22 to 24 of its bits, off by 2^-23 of it at most.  A
// product is the three partial products hh, hm, mh, each exact, summed in fp32 by the matrix unit; what is left out (mm) is below
// 2^-22 |ab|.  Half the matrix instructions of the three-way bf16 split (split_bf16.h), two thirds of the bytes in LDS and
// registers.
//
// Precision.  What a sum of K products loses is not the products' 2^-24 but the matrix unit's rounding of the running sum: against
// 64 bits 0.097 sqrt(K) units of 2^-24 in the 2-norm (1216: 3.3, 2304: 4.7, 9216: 10.4, the same for both splits' instructions
// and both shapes), beside 1.3 units for the operands as held here.  The kernels take the large sum's leading bits out of the
// matrix unit's accumulator every few hundred indices (Leading16 below), so that it rounds short sums only; the rule in api.cpp
// takes this split where both together are below what the three-way split loses.
//
// Range.  f16 ends at 65504 and keeps 11 bits down to 2^-14: the power of two puts the largest of a sample at 2^12 to 2^13, which
// leaves 2^3 above.  A value is held as said from 2^-14 on and, within 2^-36, to 2^-20 of itself from 2^-16 on: 2^-28 of the
// sample's largest, where one of 10^8 normally distributed ones is.  A value that is not held -- above 65504, not a number, or below
// 2^-16 and not zero -- keeps the chunk or the step that it is in out of these sums; the kernels add those behind, on the three-way
// split.  That goes by each value and not by the largest of some: neighbours need not be terms of the same sums, nor meet weights of
// one size.
#pragma once

#include <hip/hip_runtime.h>

#include "device_utils.h"
#include "split_bf16.h"

namespace mi355conv {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kHalfShift = 11;             // m is held times 2^11
constexpr float kHalfUp = (float)(1 << kHalfShift), kHalfDown = 1.f / kHalfUp;
constexpr int kHalfTop = 12;               // exponent of the sample's largest operand
constexpr int kHalfLeast = -16;            // of the power of two: fp32's smallest denormals are not scaled to zero
constexpr uint32_t kHalfFloor = 2u * 0x37800000u - 1u;  // nonzero_order of 2^-16, the smallest operand that is held
constexpr float kHalfCeil = 65504.f;                    // the largest

// Power of two for a sample whose largest magnitude has these bits (0: an empty or all-zero sample).
__device__ __forceinline__ int half_scale(uint32_t bits) {
  if (bits == 0) return 0;
  const int e = kHalfTop - (bits >> 23 ? (int)(bits >> 23) - 127 : 31 - __builtin_clz(bits) - 149);
  return e < kHalfLeast ? kHalfLeast : e;
}

// Bits of |v| for the sample; infinities and NaN do not count.
__device__ __forceinline__ uint32_t sample_bits(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v) & 0x7fffffffu;
  return u < 0x7f800000u ? u : 0u;
}

__device__ __forceinline__ float scale_by(float v, int e) { return __builtin_amdgcn_ldexpf(v, e); }

// Largest magnitude, NaN if there is one.
__device__ __forceinline__ float max3_abs(float a, float b, float c) {
  float r;
  asm("v_maximum3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// Bits of |v| twice, less one: the smallest of them is that of the smallest operand that is not zero.
__device__ __forceinline__ uint32_t nonzero_order(float v) { return (__builtin_bit_cast(uint32_t, v) << 1) - 1u; }

__device__ __forceinline__ uint32_t least3(uint32_t a, uint32_t b, uint32_t c) {
  const uint32_t m = a < b ? a : b;
  return m < c ? m : c;
}

// Range of operands: the smallest nonzero_order and the largest magnitude so far.
struct HalfRange {
  uint32_t least = 0xffffffffu;
  float most = 0.f;
  __device__ __forceinline__ void add(const float (&s)[8]) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      least = least3(nonzero_order(s[e]), nonzero_order(s[e + 1]), least);
      most = max3_abs(s[e], s[e + 1], most);
    }
  }
  // Of scaled operands: whether one is not held.
  __device__ __forceinline__ bool unheld() const { return least < kHalfFloor || !(most <= kHalfCeil); }
};

struct SplitHalf8 {  // eight consecutive reduction indices of one row or column
  u32x4 h, m;
};

__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  f16x2 v;
  v[0] = (_Float16)a;
  v[1] = (_Float16)b;
  return __builtin_bit_cast(uint32_t, v);
}

// Of scaled operands.
__device__ __forceinline__ SplitHalf8 split_half8(const float (&s)[8]) {
  SplitHalf8 r;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float a = s[2 * p], b = s[2 * p + 1];
    uint32_t pair = pack_f16(a, b);
    asm("" : "+v"(pair));  // or each half is converted once more by itself
    r.h[p] = pair;
    const f16x2 h = __builtin_bit_cast(f16x2, pair);
    float ra = __builtin_fmaf((float)h[0], -kHalfUp, a * kHalfUp), rb = __builtin_fmaf((float)h[1], -kHalfUp, b * kHalfUp);
    asm("" : "+v"(ra), "+v"(rb));  // or both are multiply-adds into half a register, which take 2.6 times an instruction's time each
    r.m[p] = pack_f16(ra, rb);
  }
  return r;
}

template <int MT>
__device__ __forceinline__ void mfma_f16(const u32x4& a, const u32x4& b, typename Mfma<MT>::Acc& c) {
  const f16x8 av = __builtin_bit_cast(f16x8, a), bv = __builtin_bit_cast(f16x8, b);
  if constexpr (MT == 32)
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(av, bv, c, 0, 0, 0);
  else
    c = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bv, c, 0, 0, 0);
}

// hi[j] += h h, lo[j] += m h + h m (2^11 times its value), of one row block and NB column blocks.
template <int MT, int NB>
__device__ __forceinline__ void mfma_split(const u32x4 (&a)[2], const u32x4 (&b)[NB][2],
                                           typename Mfma<MT>::Acc (&hi)[NB], typename Mfma<MT>::Acc (&lo)[NB]) {
#pragma unroll
  for (int j = 0; j < NB; ++j) mfma_f16<MT>(a[1], b[j][0], lo[j]);
#pragma unroll
  for (int j = 0; j < NB; ++j) mfma_f16<MT>(a[0], b[j][0], hi[j]);
#pragma unroll
  for (int j = 0; j < NB; ++j) mfma_f16<MT>(a[0], b[j][1], lo[j]);
}

// Leading bits of running sums, two to a word as bf16: take() moves them out of the accumulators, which keep the exact rest
// (below 2^-8 of the whole), give() adds them back.  Every take rounds the whole sum to fp32 once.
struct Leading16 {
  SplitSel minus;
  // Plain additions: the dot product rounds towards zero, which leaves the exact differences of take() as they are but shrinks a
  // sum that is added up many times (2304 indices in two slices: 3.85 units against 2.5).
  static __device__ __forceinline__ void give(uint32_t word, float& a, float& b) {
    a += __builtin_bit_cast(float, word << 16);
    b += __builtin_bit_cast(float, word & 0xffff0000u);
  }
  __device__ __forceinline__ uint32_t take(float& a, float& b) const {
    const uint32_t word = pack_bf16(a, b);
    a = minus_half(word, minus.lo, a);
    b = minus_half(word, minus.hi, b);
    return word;
  }
};

}  // namespace mi355conv
