// Two-way f16 split of fp32 operands for the f16 matrix instructions of gfx950.
//
// A float a, times a power of two that is the same for the whole blob, is taken as h + m with h = f16(a) and m = f16(a - h),
// m kept times 2^11 so that both have the exponents of the operand: 22 to 24 of its bits, off by 2^-23 of it at most.  A
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
// Range.  f16 ends at 65504 and keeps 11 bits down to 2^-14: the power of two puts the largest of a sample of the blob at 2^11,
// which leaves 2^5 above and 2^23 below.  An operand beyond 65504 makes its sums infinite or NaN, and eight neighbours whose largest
// is below 2^-12 and not zero are given a NaN on purpose; the kernels compute sums that are not finite again on the fp32 matrix
// instructions, from operands that hold every bit.
#pragma once

#include <hip/hip_runtime.h>

#include "device_utils.h"
#include "split_bf16.h"

namespace mi355conv {

typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kHalfShift = 11;             // m is held times 2^11
constexpr int kHalfTop = 11;               // exponent of the sample's largest operand
constexpr float kHalfTiny = 0x1p-12f;      // eight operands below that are not held well
constexpr uint32_t kHalfNans = 0x7e007e00u;

// Power of two for a blob whose sample's largest magnitude has these bits (0: an empty or all-zero sample).
__device__ __forceinline__ int half_scale(uint32_t bits) {
  if (bits == 0) return 0;
  const int e = bits >> 23 ? (int)(bits >> 23) - 127 : 31 - __builtin_clz(bits) - 149;
  return kHalfTop - e;
}

// Bits of |v| for the sample; infinities and NaN do not count.
__device__ __forceinline__ uint32_t sample_bits(float v) {
  const uint32_t u = __builtin_bit_cast(uint32_t, v) & 0x7fffffffu;
  return u < 0x7f800000u ? u : 0u;
}

__device__ __forceinline__ float scale_by(float v, int e) { return __builtin_amdgcn_ldexpf(v, e); }

// One blob's power of two, and the unscaled bound below which eight neighbours are too small (minus one, in bits).
struct HalfScale {
  int e;
  uint32_t tiny;
  __device__ __forceinline__ explicit HalfScale(int exponent) : e(exponent) {
    const uint32_t u = __builtin_bit_cast(uint32_t, scale_by(kHalfTiny, -exponent));
    tiny = u ? u - 1 : 0;
  }
};

__device__ __forceinline__ float max3_abs(float a, float b, float c) {
  float r;
  asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

__device__ __forceinline__ bool half_too_small(const float (&v)[8], const HalfScale& s) {
  const float mx = max3_abs(max3_abs(max3_abs(v[0], v[1], v[2]), v[3], v[4]), max3_abs(v[5], v[6], v[7]), 0.f);
  return __builtin_bit_cast(uint32_t, mx) - 1u < s.tiny;
}

struct SplitHalf8 {  // eight consecutive reduction indices of one row or column
  u32x4 h, m;
};

__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
  f16x2 v;
  v[0] = (_Float16)a;
  v[1] = (_Float16)b;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ SplitHalf8 split_half8(const float (&v)[8], const HalfScale& s) {
  SplitHalf8 r;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float a = v[2 * p], b = v[2 * p + 1];
    uint32_t pair = pack_f16(scale_by(a, s.e), scale_by(b, s.e));
    asm("" : "+v"(pair));  // or each half is converted once more by itself
    r.h[p] = pair;
    const f16x2 h = __builtin_bit_cast(f16x2, pair);
    constexpr float up = (float)(1 << kHalfShift);
    r.m[p] = pack_f16(__builtin_fmaf((float)h[0], -up, scale_by(a, s.e + kHalfShift)),
                      __builtin_fmaf((float)h[1], -up, scale_by(b, s.e + kHalfShift)));
  }
  if (half_too_small(v, s)) r.h[0] = kHalfNans;
  return r;
}

// The same for the pack kernel, with a third term that holds the bits that are left.  A weight that the terms cannot hold, or
// one of eight that are too small, becomes a NaN with its own bits in the other two terms.
constexpr uint16_t kHalfEscape = 0x7e00;

__device__ __forceinline__ void split_half1(float a, int e, bool escape, uint16_t& h, uint16_t& m, uint16_t& l) {
  const float s = scale_by(a, e);
  if (!(__builtin_fabsf(s) < 65504.f) || (escape && a != 0.f)) {
    const uint32_t u = __builtin_bit_cast(uint32_t, a);
    h = kHalfEscape;
    m = (uint16_t)(u >> 16);
    l = (uint16_t)u;
    return;
  }
  constexpr float up = (float)(1 << kHalfShift);
  const _Float16 th = (_Float16)s;
  const float r = (s - (float)th) * up;
  const _Float16 tm = (_Float16)r;
  h = __builtin_bit_cast(uint16_t, th);
  m = __builtin_bit_cast(uint16_t, tm);
  l = __builtin_bit_cast(uint16_t, (_Float16)((r - (float)tm) * up));
}

__device__ __forceinline__ float join_f16(uint16_t h, uint16_t m, uint16_t l, int e) {
  if (h == kHalfEscape) return __builtin_bit_cast(float, (uint32_t)m << 16 | l);
  auto term = [](uint16_t x) { return (float)__builtin_bit_cast(_Float16, x); };
  constexpr float down = 1.f / (float)(1 << kHalfShift);
  return scale_by(term(h) + (term(m) + term(l) * down) * down, -e);
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
