// Exact three-way bf16 split of fp32 operands for the bf16 matrix instructions of gfx950.
//
// A float a (24 significant bits) is h + m + l with h = bf16(a), m = bf16(a - h), l = a - h - m, each
// rounded to nearest: both differences are exact, and l has at most eight significant bits left, so the
// three terms hold every bit of a.  A product a*b is taken as the six partial products down to 2^-18 of
// it -- hh, hm, mh, mm, hl, lh -- each exact, summed in fp32 by the matrix unit; what is left out (ml, lm,
// ll) is below 2^-24 |ab|, 2^-28 on average and of either sign.  Six bf16 instructions of 16 reduction
// indices take 6 x 32 cycles where the fp32 instructions they replace take 512: a register-only loop of
// them sustains 2002 TFLOP/s = 334 TFLOP/s of fp32 products, against 143 for the 32x32x2 fp32 instruction.
//
// The third term has an exponent 16 below the operand's and bf16 the range of fp32, so both operands are multiplied by 2^16
// before they are split and the sums by 2^-32 at the end: every fp32 value below 2^111, denormals included, keeps its bits.
// Without the factors operands under 2^-109 lost some (2^-118: results off by 8.8e-6; fp32 denormals: all of them).  They
// cost two vector instructions to the split's seven, up to 0.3 % of a layer's step (96 -> 256 in two groups, 5x5 at 27x27,
// batch 128: 817 -> 819 us) and 0.7 % on the folded form, whose loads are busiest (3 -> 96, 11x11, stride 4: 448 -> 451).
//
// An operand that is not finite or from 2^111 on, or a sum from 2^96 on, makes the differences or the sums infinite or NaN; the
// kernels look for non-finite sums at their end and compute those again on the fp32 matrix instructions.
#pragma once

#include <hip/hip_runtime.h>

#include "device_utils.h"

namespace mi355conv {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kSplitScale = 0x1p16f, kSplitUnscale = 0x1p-32f;  // of an operand, of the sums

struct Split8 {  // eight consecutive reduction indices of one row or column
  u32x4 h, m, l;
};

// The two selectors of the split: dot2(pair, sel, x) = x - (low or high half of the pair).  They live in
// scalar registers: as a literal the low one is taken for the fp32 constant -1.0 and picks the high half.
struct SplitSel {
  uint32_t lo, hi;
  __device__ __forceinline__ SplitSel() {
    asm("s_mov_b32 %0, 0xbf80" : "=s"(lo));
    asm("s_mov_b32 %0, 0xbf800000" : "=s"(hi));
  }
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 v;
  v[0] = (__bf16)a;
  v[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float minus_half(uint32_t pair, uint32_t sel, float x) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, sel), x, false);
}

// Nine vector instructions per pair.
__device__ __forceinline__ Split8 split8(const float (&v)[8], const SplitSel& s) {
  Split8 r;
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float a = v[2 * p] * kSplitScale, b = v[2 * p + 1] * kSplitScale;
    const uint32_t h = pack_bf16(a, b);
    const float ra = minus_half(h, s.lo, a), rb = minus_half(h, s.hi, b);
    const uint32_t m = pack_bf16(ra, rb);
    r.h[p] = h;
    r.m[p] = m;
    r.l[p] = pack_bf16(minus_half(m, s.lo, ra), minus_half(m, s.hi, rb));
  }
  return r;
}

// The same for the pack kernels.  A weight that the scaled terms cannot hold -- 2^111 and above, infinities, NaNs -- becomes
// a NaN with its own bits in the other two terms, so that its sums are computed again and join_bf16 knows it.
constexpr uint16_t kSplitEscape = 0x7fc0;

__device__ __forceinline__ void split1(float a, uint16_t& h, uint16_t& m, uint16_t& l) {
  const uint32_t u = __builtin_bit_cast(uint32_t, a);
  if ((u & 0x7fffffffu) >= 0x77000000u) {
    h = kSplitEscape;
    m = (uint16_t)(u >> 16);
    l = (uint16_t)u;
    return;
  }
  auto rne = [](float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); };
  auto up = [](uint16_t x) { return __builtin_bit_cast(float, (uint32_t)x << 16); };
  const float s = a * kSplitScale;
  h = rne(s);
  const float r = s - up(h);
  m = rne(r);
  l = rne(r - up(m));
}

__device__ __forceinline__ float join_bf16(uint16_t h, uint16_t m, uint16_t l) {
  if (h == kSplitEscape) return __builtin_bit_cast(float, (uint32_t)m << 16 | l);
  auto up = [](uint16_t x) { return __builtin_bit_cast(float, (uint32_t)x << 16); };
  return ((up(h) + up(m)) + up(l)) * (1.f / kSplitScale);
}

// bf16 matrix instructions with the accumulator layout of the fp32 ones (Mfma<MT> in device_utils.h):
//   MT = 32: 16 k-values, lane l feeds A[l%32][8*(l/32) .. +7] and B[8*(l/32) .. +7][l%32]
//   MT = 16: 32 k-values, lane l feeds A[l%16][8*(l/16) .. +7] and B[8*(l/16) .. +7][l%16]
template <int MT>
__device__ __forceinline__ void mfma_bf16(const u32x4& a, const u32x4& b, typename Mfma<MT>::Acc& c) {
  const bf16x8 av = __builtin_bit_cast(bf16x8, a), bv = __builtin_bit_cast(bf16x8, b);
  if constexpr (MT == 32)
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, c, 0, 0, 0);
  else
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv, c, 0, 0, 0);
}

// hi[j] += h h, lo[j] += the five smaller partial products, of one row block and NB column blocks.  Two
// accumulators because every instruction rounds the sum it adds to: the large one is rounded once per 16
// (MT = 32) or 32 reduction indices, where the fp32 instructions round eight times, and what the small
// one is rounded by is 2^-8 of that -- with all six products in one accumulator the sums of a 2304-long
// reduction were 7 % further from exact than the fp32 instructions' (rms 8.8e-7 against 8.2e-7).
template <int MT, int NB>
__device__ __forceinline__ void mfma_split(const u32x4 (&a)[3], const u32x4 (&b)[NB][3],
                                           typename Mfma<MT>::Acc (&hi)[NB], typename Mfma<MT>::Acc (&lo)[NB]) {
  constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
#pragma unroll
  for (int q = 0; q < 5; ++q)
#pragma unroll
    for (int j = 0; j < NB; ++j) mfma_bf16<MT>(a[pa[q]], b[j][pb[q]], lo[j]);
#pragma unroll
  for (int j = 0; j < NB; ++j) mfma_bf16<MT>(a[0], b[j][0], hi[j]);
}

// Folded layers (SplitFold): where channel v of a grid position sits relative to the position's own pixel -- byte offset, and
// row and column displacement in one word (15 and 16 bits).  A channel past the last one sits beyond any blob (which is at
// most 2^30 bytes): its loads read as zero.
struct FoldEntry {
  uint32_t off, rc;
};

__device__ __forceinline__ int fold_row(const FoldEntry& f) { return (int)(f.rc >> 16); }
__device__ __forceinline__ int fold_col(const FoldEntry& f) { return (int)(f.rc & 0xffffu); }

__device__ __forceinline__ void fill_fold_table(FoldEntry* tab, int count, const SplitFold& f, int width, int plane, int t,
                                                int threads) {
  for (int v = t; v < count; v += threads) {
    const uint32_t c = mdiv((uint32_t)v, f.mFF), rem = (uint32_t)v - c * (uint32_t)f.ff;
    const uint32_t ir = mdiv(rem, f.mFw), jr = rem - ir * (uint32_t)f.fw;
    FoldEntry e;
    const bool real = v < f.V;
    e.off = real ? 4u * (c * (uint32_t)plane + ir * (uint32_t)(f.dh * width) + jr * (uint32_t)f.dw) : 0x80000000u;
    e.rc = real ? (ir * (uint32_t)f.dh) << 16 | jr * (uint32_t)f.dw : 0u;
    tab[v] = e;
  }
}

// Eight channels of the grid position whose own pixel has byte offset `at` (modulo 2^32), row and column: two quads of four
// pixels side by side that start on a column of a multiple of four, so only the right border of the image cuts a quad
// (what lies behind the blob reads as zero element by element).
__device__ __forceinline__ void load_folded(__amdgpu_buffer_rsrc_t rsrc, const FoldEntry* fe, uint32_t at, int row, int col,
                                            int H, int W, float (&v)[8]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const FoldEntry f = fe[4 * q];
    const int c = col + fold_col(f);
    const bool ok = ((uint32_t)(row + fold_row(f)) < (uint32_t)H) & ((uint32_t)c < (uint32_t)W);
    const u32x4 x =
        __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, ok ? at + f.off : 0x80000000u, 0, 0));
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * q + e] = c + e < W ? __builtin_bit_cast(float, (uint32_t)x[e]) : 0.f;
  }
}

__device__ __forceinline__ bool not_finite(float v) {
  return (__builtin_bit_cast(uint32_t, v) & 0x7f800000u) == 0x7f800000u;
}

}  // namespace mi355conv
