// Implicit-GEMM correlation on the bf16 matrix instructions with fp32 operands split exactly in three
// (split_bf16.h), for gathers whose input rows fit LDS: forward and, through the sub-pixel rewriting,
// backward data.  Same problem and epilogue as corr_kernel (kernels_corr.hip):
//
//   D[m][col] = sum_k A[m][k] * in[n, g*Cg + c, a*sh - ph + i*dh, b*sw - pw + j*dw],  col = (n, a, b)
//
// The reduction runs as (chunk of 16 channels, tap, channel).  A workgroup keeps the raw input rows that its
// columns touch -- a zero-padded patch of 16 channels -- in LDS, already split: [half of the chunk][position]
// [h, m, l][8 channels], 48 bytes per position and half.  An element is loaded and split once per tile and
// chunk however many taps use it, the MFMA B operand of a tap is a 16-byte read at the column's base
// plus a uniform offset, and padding, ragged borders and columns past the batch are resolved by the range
// check of the patch's loads.  48 is an odd multiple of 16: a run of consecutive positions spreads over the banks.  Where a
// tile's columns go on in the next image row the runs break, and with the stores 5 to 15 M conflict cycles a launch
// remain on the large layers below (11 % of the cycles of the 48x256 tile, 4 to 10 % of the others').
//
// The A operand is packed in fragment order -- [m tile][step][row block][h, m, l][lane][8 k] -- so a wave
// loads what its lanes feed with coalesced 16-byte loads straight from L2 into registers, one step ahead: A
// never touches LDS, and the waves of a workgroup meet at a barrier once per chunk (T steps) only.
//
// Bound by the matrix unit (busy 67-78 % of the compute units' cycles on large layers, at the 1.9 GHz that the chip holds
// under this load), then by the prologue on small problems.  With the pack kernel, against the fp32 kernels: 57.3 GFLOP (96 ->
// 256 in two groups, 5x5 at 27x27, batch 128) forward 431 -> 247 us, backward data 459 -> 235; 38.3 GFLOP (256 -> 384, 3x3 at
// 13x13) 292 -> 174 and 309 -> 200; 6.7 GFLOP (45 -> 77, 3x5 at 51x67, stride 2 x 1) 92 -> 52 and 87 -> 50; 1.3 GFLOP (32 ->
// 32, 5x5 at 16x16, batch 100) 29 -> 21.  172 and 115 us are the matrix instructions of the first two at 2000 TFLOP/s.
//
// HALF: long reductions on two f16 terms (split_f16.h), half the matrix instructions.  The stage is [h, m][half][position] then,
// 16 bytes a position.  The same passes: 57.3 GFLOP 249 -> 171 us and 269 -> 172, 38.3 GFLOP 172 -> 115 and 206 -> 141, 6.7 GFLOP 49
// -> 40 and 53 -> 44 (without the test of every value 2 % less); the pack kernel, which samples both blobs and writes both splits, 1
// to 2.5 us more.  The matrix unit is busy 50 to 55 % of the cycles, at the clock that the chip's power leaves (1.7 GHz); a quarter to
// two fifths of the waves' time are waits for weights, patches and barriers.  Weights two steps ahead gave nothing (108 -> 112 us where
// the registers hold them, spills elsewhere).
// AGAIN: what a workgroup's HALF sums had to leave out, chunk by chunk, it adds on the bf16 terms behind them.  A chunk of 5.6 M values
// that is left out costs 7 to 11 us, all of them 1.8 times a pass (57.3 GFLOP, forward: 168 -> 316 us, of which weights far below the
// others are the cause for a third of the rows).  Both splits' instructions on one set of accumulators, chunk by chunk, cost hundreds of
// spilled registers.
//
// Forms (SplitFold).  Folded taps: 3 -> 96 channels, 11x11, stride 4 at 227x227, batch 128, forward 254 -> 195 us; busy 46 %,
// the folded patch's loads and splits (3 vector instructions to a matrix one) and 30 % of padding take the rest.  Columns
// of 1x1 kernels use a patch element once per row tile, so splitting weighs most there: inner product 128 x 9216 -> 4096, data
// gradient 97 -> 64 us, filter gradient 106 -> 78 (151 MB written, 30 us), busy 36-51 %; one-pixel images: its forward pass
// 90 -> 72.
#include <hip/hip_runtime.h>

#include "corr_epilogue.h"
#include "device_utils.h"
#include "internal.h"
#include "split_bf16.h"
#include "split_f16.h"

namespace mi355conv {

namespace {

constexpr int kThreads = 256;

enum SplitTerms { BF16, HALF, AGAIN };  // three bf16 terms; two f16 terms; the bf16 terms of what those left out

template <int MT, int MB, int NB, int WM, int WN, SplitTerms KIND = BF16, int EPT = 4>
struct SplitCfg {
  static constexpr int BM = WM * MB * MT;
  static constexpr int BN = WN * NB * MT;
  static constexpr int BLOCKS = WM * MB;            // row blocks of a tile
  static constexpr int TPS = MT == 32 ? 1 : 2;      // taps per step: a 16-row instruction takes 32 k values
  static constexpr uint32_t FRAG = 1024;            // bytes of one operand fragment (64 lanes x 8 bf16)
  // Fragments of a row block and step: the three bf16 terms', which two f16 terms' precede where there are such sums.
  static constexpr uint32_t BLOCK = (KIND == BF16 ? 3 : 5) * FRAG, FIRST = KIND == AGAIN ? 2 * FRAG : 0, STEP = BLOCKS * BLOCK;
  // 64x64 per wave: B operands a step ahead, two waves per SIMD.  The smaller tiles run few matrix instructions
  // per step and, on small grids, alone on their SIMD: A operands several steps ahead.
  static constexpr bool BDEEP = MT == 32 && MB * NB >= 4;
  static constexpr int DEPTH = BDEEP || MT == 16 ? 1 : MB == 3 ? 2 : NB == 2 ? 3 : 8;
  static constexpr bool LEAD_STEPS = DEPTH <= 2;  // leading bits move between steps, else between chunks
  // per SIMD; the f16 form's stages of more than two units per thread leave room for two workgroups anyway
  static constexpr int WAVES = MT == 32 && MB == 1 && NB == 2 && (KIND == BF16 || EPT == 2) ? 3 : 2;
  static_assert(WM * WN == 4, "four waves per workgroup");
};

enum SplitForm { IMAGE, FOLDED, COLUMNS, PIXELS };  // PIXELS: COLUMNS over images of one pixel

// EPT: patch units (one position x 8 channels) per thread, 2*PSZ <= 256*EPT.
// FORM: what the patch holds (SplitFold in internal.h).
// `left_out`: the chunks of the slice that the f16 terms do not hold, found by HALF, added by AGAIN.
struct LeftOut {
  uint64_t bits[2];
  __device__ __forceinline__ bool has(int i) const { return (i < 64 ? bits[0] : bits[1]) >> (i & 63) & 1; }
};
static_assert(kUnheldChunks == 128, "LeftOut");

template <int MT, int MB, int NB, int WM, int WN, int EPT, SplitForm FORM, SplitTerms KIND>
__device__ __forceinline__ void corr_split(const CorrSplitArgs& a, LeftOut& left_out) {
  using C = SplitCfg<MT, MB, NB, WM, WN, KIND>;
  using M = Mfma<MT>;
  constexpr int BM = C::BM, BN = C::BN, TERMS = KIND == HALF ? 2 : 3;
  constexpr bool FOLD = FORM == FOLDED, PIX = FORM == PIXELS, COLS = FORM == COLUMNS || PIX;
  static_assert(!(FOLD && KIND != BF16), "the folded form's reductions are short");
  // Bytes from one position of a stage to the next and from one term to the next: bf16 [half][position][h, m, l], f16
  // [h, m][half][position].
  constexpr uint32_t POS = KIND == HALF ? 16 : 48, TERM = KIND == HALF ? split_half_stage(EPT, PIX ? BN : 0) / 2 : 16;

  extern __shared__ __align__(16) float smem[];  // one or two patch stages; the epilogue's tables at the end

  int t = threadIdx.x;
  uint32_t lin = xcd_contiguous_block_id();
  if constexpr (KIND == AGAIN) {  // what depends on these is computed here again, not kept in registers over the first sums
    asm volatile("" : "+v"(t));
    asm volatile("" : "+s"(lin));
  }
  const int lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wv / WN, wn = wv % WN;

  // column tile fastest: the workgroups of an XCD share one row tile's packed weights in its L2
  const uint32_t col_tile = lin % (uint32_t)a.col_tiles;
  lin /= (uint32_t)a.col_tiles;
  const uint32_t m_tile = lin % (uint32_t)a.m_tiles;
  lin /= (uint32_t)a.m_tiles;
  const uint32_t g = lin % (uint32_t)a.G;
  const uint32_t split = lin / (uint32_t)a.G;

  // ---- geometry of this tile's patch (uniform), as in corr_patch_kernel with any stride and dilation:
  // segment 0 (image n0) starts at output row a0 and owns R0 patch rows, every later image RS of them.  The
  // zeros right of a row are those left of the next one, and the zeros below an image those above the next
  // (share_w, share_h): 5x5 "same" columns at 27x27 take 350 positions instead of 465, which is two
  // workgroups per compute unit instead of one. ----
  const int TH = a.THW / a.TW;
  const uint32_t ext = (uint32_t)((TH - 1) * a.dh + 1);
  const uint32_t col0 = col_tile * BN;
  const uint32_t n0 = mdiv(col0, a.mP);
  const uint32_t a0 = mdiv(col0 - n0 * a.P, a.mPW);
  const uint32_t R0 = ((uint32_t)a.PH - 1 - a0) * a.sh + ext - a.share_h;
  const uint32_t RS = ((uint32_t)a.PH - 1) * a.sh + ext - a.share_h;
  auto patch_row_base = [&](uint32_t n, uint32_t pa) {
    const uint32_t s = n - n0;
    return s == 0 ? (pa - a0) * a.sh : R0 + (s - 1) * RS + pa * a.sh;
  };
  uint32_t col_last = col0 + BN - 1;
  if (col_last > (uint32_t)a.ncols - 1) col_last = (uint32_t)a.ncols - 1;
  uint32_t patch_elems = (uint32_t)a.PSZ;
  if (!COLS) {
    const uint32_t n = mdiv(col_last, a.mP);
    const uint32_t pa = mdiv(col_last - n * a.P, a.mPW);
    patch_elems = (patch_row_base(n, pa) + ext) * (uint32_t)a.PWID + a.share_w;
  }

  // ---- f16: every group of images has a power of two of its own, from its sample; the few values of a weak one do not count
  // against all samples' largest.  Columns and patch positions belong to one image each. ----
  uint32_t top_sample = 0;
  if constexpr (KIND == HALF) {
#pragma unroll
    for (int i = 0; i < kSamples / 64; ++i) {
      const uint32_t u = a.scale[64 * i + lane] & ~kWeakSample;
      top_sample = u > top_sample ? u : top_sample;
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t u = (uint32_t)__shfl_xor((int)top_sample, d);
      top_sample = u > top_sample ? u : top_sample;
    }
  }
  auto image_scale = [&](uint32_t n) {
    const uint32_t s = a.scale[mdiv(n, a.mSample)];
    return half_scale(s & kWeakSample ? top_sample : s);
  };

  // ---- per-lane B columns: byte address of (column, its half of the chunk) inside a patch stage ----
  const uint32_t kgrp = lane / MT;  // which 8 k values of a step this lane feeds
  const uint32_t half = kgrp & 1;
  uint32_t lanebase[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    uint32_t col = col0 + (wn * NB + j) * MT + lane % MT;
    if (col > col_last) col = col_last;  // columns past the edge are never stored: any valid address
    const uint32_t n = mdiv(col, a.mP);
    const uint32_t pix = col - n * a.P;
    const uint32_t pa = mdiv(pix, a.mPW);
    const uint32_t pb = pix - pa * a.PW;
    lanebase[j] = POS * (COLS ? col - col0 + half * (uint32_t)a.PSZ
                              : patch_row_base(n, pa) * (uint32_t)a.PWID + pb * a.sw + half * (uint32_t)a.PSZ);
  }

  // ---- per-thread patch units: where they come from (relative to channel 0 of the group) ----
  const __amdgpu_buffer_rsrc_t in_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.in), 0, (int)a.in_bytes, 0x00020000);
  const uint32_t chan_bytes = 4u * (uint32_t)a.IHW;
  const uint32_t stage_bytes = KIND == HALF ? 2 * TERM : 96u * (uint32_t)a.PSZ;
  FoldEntry* const fold_tab =
      reinterpret_cast<FoldEntry*>(reinterpret_cast<char*>(smem) + (uint32_t)a.patch_stages * stage_bytes);
  if (FOLD) {
    fill_fold_table(fold_tab, a.NS * 16, a.fold, a.IW, a.IHW, t, kThreads);
    __syncthreads();
  }
  // Unfolded: the byte offset of the unit's first channel in chunk 0.  Folded: that of its position, whose row and
  // column the channels are checked from.
  // Of images of one pixel the channels are contiguous: a unit is two 16-byte loads, eight neighbouring lanes take the
  // eight units of a column (256 contiguous bytes), and the groups' pitch of an odd number of 48-byte positions spreads
  // their stores over the banks.
  const uint32_t slot0 = PIX ? (t & 1u) * (uint32_t)a.PSZ + ((t >> 1) & 3u) * (uint32_t)a.PWID + (uint32_t)(t >> 3) : (uint32_t)t;
  constexpr uint32_t kSlotStep = PIX ? kThreads / 8 : kThreads;  // a thread's units in the stage
  uint32_t psrc[EPT];
  int pscale[KIND == HALF ? EPT : 1];  // power of two of the unit's image
  int prow_in[FOLD ? EPT : 1], pcol_in[FOLD ? EPT : 1];
#pragma unroll
  for (int r = 0; r < EPT; ++r) {
    const uint32_t u = t + r * kThreads;
    const uint32_t hf = u >= (uint32_t)a.PSZ ? 1u : 0u;
    const uint32_t e = u - hf * (uint32_t)a.PSZ;
    uint32_t src = 0x80000000u;  // beyond the blob (which is at most 2^30 bytes): reads as zero
    if (KIND == HALF) pscale[r] = 0;
    if (FOLD) prow_in[r] = -(1 << 28), pcol_in[r] = 0;  // fails every bounds test
    if (PIX) {
      const uint32_t col = col0 + (uint32_t)(t >> 3) + r * kSlotStep;
      if (col <= col_last) src = 4u * (col * (uint32_t)a.in_img_stride + g * (uint32_t)a.in_grp_stride) + 32u * (t & 7u);
      if (KIND == HALF) pscale[r] = image_scale(col < col_last ? col : col_last);
    } else if (e < patch_elems && u < 2u * (uint32_t)a.PSZ) {
      const uint32_t prow = mdiv(e, a.mPWID);  // COLS: the group of 16 channels
      const uint32_t pcol = e - prow * a.PWID;
      uint32_t n = n0, rin = prow, alo = a0;
      int gr = 0, gc = (int)pcol;
      if (COLS) {
        const uint32_t col = col0 + pcol;
        n = mdiv(col, a.mP);
        const uint32_t pix = col - n * a.P;
        gr = (int)mdiv(pix, a.mPW);
        gc = (int)(pix - (uint32_t)gr * a.PW);
        if (col > col_last) n = (uint32_t)a.Nimg;
      } else {
        if (prow >= R0) {
          const uint32_t s1 = mdiv(prow - R0, a.mRSEG);
          n = n0 + 1 + s1;
          rin = prow - R0 - s1 * RS;
          alo = 0;
        }
        gr = (int)(alo * a.sh + rin);
      }
      const int ih = (FOLD || COLS ? gr * a.fold.Uh : gr) - a.ph, iw = (FOLD || COLS ? gc * a.fold.Uw : gc) - a.pw;
      const uint32_t at = 4u * (n * (uint32_t)a.in_img_stride + g * (uint32_t)a.in_grp_stride + (uint32_t)(ih * a.IW + iw));
      if (FOLD) {
        if (n < (uint32_t)a.Nimg) src = at, prow_in[r] = ih, pcol_in[r] = iw;
      } else if ((uint32_t)ih < (uint32_t)a.IH && (uint32_t)iw < (uint32_t)a.IW && n < (uint32_t)a.Nimg) {
        src = at + (COLS ? prow * 16u + hf * 8u : hf * 8u) * chan_bytes;
        if (KIND == HALF) pscale[r] = image_scale(n);
      }
    }
    psrc[r] = src;
  }
  // Channels past the group's last read the next group's or image's (or, past the blob, zero): their packed weights are zero.  They
  // need not be of a size with this image's, so the f16 form takes zeros.
  constexpr int kChunkChannels = COLS ? 64 : 16;
  float pr[EPT][8];
  const int T = a.THW, SPC = (T + C::TPS - 1) / C::TPS;  // taps and steps per chunk
  const int cc_first = (int)split * a.chunks_per_split;  // chunks of 16 channels
  uint32_t w_unheld = 0;  // f16: a weight of the chunk is not held
  auto patch_load = [&](int cc) {
    if constexpr (KIND == HALF) {
      const int count = SPC * C::BLOCKS;
      const uint32_t* const at = a.unheld + ((size_t)(g * a.m_tiles + m_tile) * a.NS + cc) * count;
      w_unheld = 0;
      for (int i = t; i < count; i += kThreads) w_unheld |= at[i];
    }
    const uint32_t coff = (uint32_t)(cc * kChunkChannels) * chan_bytes;
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      uint32_t src = psrc[r];
      asm volatile("" : "+v"(src));  // or the compiler keeps eight running addresses per unit in registers
      if (FOLD) {
        const uint32_t hf = t + r * kThreads >= a.PSZ ? 1u : 0u;
        const FoldEntry* fe = fold_tab + (cc * 16 + (int)hf * 8);
        load_folded(in_rsrc, fe, src, prow_in[r], pcol_in[r], a.IH, a.IW, pr[r]);
        __builtin_amdgcn_sched_barrier(0);  // one unit's table entries in registers at a time
      } else if (PIX) {
        src += coff;
        const u32x4 v0 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, src, 0, 0));
        const u32x4 v1 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(in_rsrc, src + 16u, 0, 0));
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) {
          pr[r][c4] = __builtin_bit_cast(float, (uint32_t)v0[c4]);
          pr[r][4 + c4] = __builtin_bit_cast(float, (uint32_t)v1[c4]);
        }
      } else {
        src += coff;
#pragma unroll
        for (int c8 = 0; c8 < 8; ++c8)
          pr[r][c8] = __builtin_bit_cast(
              float, __builtin_amdgcn_raw_buffer_load_b32(in_rsrc, src + c8 * chan_bytes, 0, 0));
      }
    }
  };
  const SplitSel sel;
  uint32_t* const unheld = reinterpret_cast<uint32_t*>(
      reinterpret_cast<char*>(smem) + (FORM == COLUMNS ? (uint32_t)a.patch_stages * stage_bytes + split_half_lead(BM, BN) : TERM - kUnheldBytes));
  auto patch_store = [&](uint32_t stage_off, int cc) {
    HalfRange range;
    const int left = a.fold.V - cc * kChunkChannels;
    if (KIND == HALF && left < kChunkChannels) {
      uint32_t u0 = (uint32_t)t;
      asm volatile("" : "+v"(u0));  // what depends on it is computed here, in the last chunk only
#pragma unroll
      for (int r = 0; r < EPT; ++r) {
        const uint32_t u = u0 + r * kThreads, hf = u >= (uint32_t)a.PSZ ? 1u : 0u;
        const int first = PIX ? 8 * (int)(u0 & 7u) : (int)(hf * 8u + (COLS ? mdiv(u - hf * (uint32_t)a.PSZ, a.mPWID) * 16u : 0u));
#pragma unroll
        for (int e = 0; e < 8; ++e) pr[r][e] = first + e < left ? pr[r][e] : 0.f;
      }
    }
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const uint32_t u = slot0 + r * kSlotStep;
      u32x4* dst = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(smem) + (stage_off + POS * u));
      if constexpr (KIND == HALF) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = scale_by(pr[r][e], pscale[r]);
        const SplitHalf8 s = split_half8(v);
        range.add(v);
        if (PIX || u < 2u * (uint32_t)a.PSZ) {
          dst[0] = s.h;
          dst[TERM / 16] = s.m;
        }
      } else {
        const Split8 s = split8(pr[r], sel);
        if (PIX || u < 2u * (uint32_t)a.PSZ) {
          dst[0] = s.h;
          dst[1] = s.m;
          dst[2] = s.l;
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // one unit's terms in registers at a time
    }
    if (KIND == HALF && (range.unheld() || w_unheld)) atomicOr(unheld + ((cc - cc_first) >> 5), 1u << ((cc - cc_first) & 31));
  };

  // ---- A fragments of this workgroup's steps ----
  int cc_end = cc_first + a.chunks_per_split;
  if (cc_end > a.NS) cc_end = a.NS;
  const char* Ag = reinterpret_cast<const char*>(a.A) +
                   ((size_t)(g * a.m_tiles + m_tile) * ((size_t)a.NS * SPC) + (size_t)cc_first * SPC) * C::STEP;
  const uint32_t a_bytes = (uint32_t)((cc_end - cc_first) * SPC) * C::STEP;
  const __amdgpu_buffer_rsrc_t a_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(Ag), 0, (int)a_bytes, 0x00020000);
  uint32_t alane[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) alane[i] = 16u * lane + (uint32_t)(wm * MB + i) * C::BLOCK + C::FIRST;
  constexpr int DEPTH = C::DEPTH;
  u32x4 av[DEPTH][MB][TERMS];
  auto load_a = [&](int d, uint32_t step_off, int i) {
#pragma unroll
    for (int q = 0; q < TERMS; ++q)
      av[d][i][q] = __builtin_bit_cast(
          u32x4, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, alane[i] + q * C::FRAG, (int)step_off, 0));
  };

  typename M::Acc acc[MB][NB], lo[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < M::NR; ++r) acc[i][j][r] = lo[i][j][r] = 0.f;

  // offset of the step DEPTH ahead; behind the last step it stays there (loaded again, never used)
  uint32_t a_off = 0;
  auto a_advance = [&]() {
    if (a_off + C::STEP < a_bytes) a_off += C::STEP;
  };
  auto fill_a = [&](int depth) {
#pragma unroll
    for (int d = 0; d < depth; ++d) {
#pragma unroll
      for (int i = 0; i < MB; ++i) load_a(d, a_off, i);
      a_advance();
    }
  };
  auto jump_a = [&](int cc) {  // to a chunk's first step
    const uint32_t off = (uint32_t)((cc - cc_first) * SPC) * C::STEP;
    a_off = off < a_bytes ? off : a_bytes - C::STEP;
  };
  int cc = cc_first;
  auto following = [&](int i) {  // the next chunk that was left out
    do ++i;
    while (i < cc_end && !left_out.has(i - cc_first));
    return i;
  };
  if constexpr (KIND == AGAIN) cc = following(cc_first - 1);
  patch_load(cc);
  if constexpr (KIND != AGAIN) fill_a(DEPTH);
  if constexpr (KIND == HALF) {
    if (t < kUnheldBytes / 4) unheld[t] = 0;
    __syncthreads();
  }
  patch_store(0, cc);
  __syncthreads();

  // ---- main loop: one step = one tap (two for the 16-row instruction) of one chunk ----
  // Position of the step's tap in the patch, advanced tap by tap; behind the last tap it stays (the 16-row
  // instruction reads it once more when their number is odd, against zero weights).
  const uint32_t tap_w = POS * (uint32_t)a.dw, tap_h = POS * (uint32_t)(a.dh * a.PWID) - tap_w * (uint32_t)(a.TW - 1);
  uint32_t pos = 0;
  int tap = 0, tj = 0;
  auto next_tap = [&]() {
    if (tap + 1 < T) {
      ++tap;
      if (++tj == a.TW) {
        tj = 0;
        pos += tap_h;
      } else {
        pos += tap_w;
      }
    }
  };
  auto load_b = [&](u32x4(&bv)[NB][TERMS]) {  // the step's B operands; moves on to the next step
    uint32_t off = pos;
    next_tap();
    if (MT == 16) {  // the upper two k groups take the second tap
      off = kgrp >= 2 ? pos : off;
      next_tap();
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const u32x4* src = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(smem) + (lanebase[j] + off));
#pragma unroll
      for (int q = 0; q < TERMS; ++q) bv[j][q] = src[q * (TERM / 16)];
    }
  };
  // One step.  A row block's A registers are reloaded with the step DEPTH ahead as soon as its last product
  // is under way; the scheduling barriers keep the compiler from holding more operands than the registers
  // have room for.
  auto run_step = [&](int d, const u32x4(&bv)[NB][TERMS]) {
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      mfma_split<MT, NB>(av[d][i], bv, acc[i], lo[i]);
      load_a(d, a_off, i);
      __builtin_amdgcn_sched_barrier(0);
    }
    a_advance();
  };
  const bool two = a.patch_stages == 2;
  uint32_t stage = 0;
  // f16: every a.lead_steps steps the large sums' leading bits move to LDS, a place of its own for every lane.
  constexpr int LEAD = MB * NB * M::NR / 8;  // 16-byte groups of eight sums
  const Leading16 leading;
  int since = 0;
  bool led = false;
  u32x4* const lead = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(smem) + (uint32_t)a.patch_stages * stage_bytes) + t;
  auto move_leading = [&]() {
#pragma unroll
    for (int q = 0; q < LEAD; ++q) {
      u32x4 w = {0, 0, 0, 0};
      if (led) w = lead[q * kThreads];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        float x = acc[(8 * q + 2 * p) / M::NR / NB][(8 * q + 2 * p) / M::NR % NB][(8 * q + 2 * p) % M::NR], y = acc[(8 * q + 2 * p) / M::NR / NB][(8 * q + 2 * p) / M::NR % NB][(8 * q + 2 * p) % M::NR + 1];
        leading.give(w[p], x, y);
        w[p] = leading.take(x, y);
        acc[(8 * q + 2 * p) / M::NR / NB][(8 * q + 2 * p) / M::NR % NB][(8 * q + 2 * p) % M::NR] = x;
        acc[(8 * q + 2 * p) / M::NR / NB][(8 * q + 2 * p) / M::NR % NB][(8 * q + 2 * p) % M::NR + 1] = y;
      }
      lead[q * kThreads] = w;
    }
    led = true;
  };
  auto count_steps = [&](int steps) {
    since += steps;
    if (KIND == HALF && since >= a.lead_steps) {
      move_leading();
      since = 0;
    }
  };
  auto begin_chunk = [&]() {
    if (cc + 1 < cc_end) patch_load(cc + 1);
    pos = stage;
    tap = tj = 0;
  };
  // Two stages: the next chunk's patch goes to the other one, whose last readers passed the last barrier; one
  // stage: to the only one, once every wave has read it.
  auto end_chunk = [&]() {
    if (two)
      stage = stage ? 0 : stage_bytes;
    else
      __syncthreads();
    if (++cc < cc_end) patch_store(stage, cc);
    __syncthreads();
  };
  auto leave_out = [&]() {  // whether to, uniformly
    if constexpr (KIND == HALF)
      if (cc < cc_end) return (__builtin_amdgcn_readfirstlane(unheld[(cc - cc_first) >> 5]) >> ((cc - cc_first) & 31) & 1) != 0;
    return false;
  };
  if constexpr (KIND == AGAIN) {
    u32x4 bv[NB][TERMS];
    while (cc < cc_end) {
      const int next = following(cc);
      if (next < cc_end) patch_load(next);
      pos = 0;
      tap = tj = 0;
      jump_a(cc);
      // a look at every line of the chunk's weights, which nobody else may read: from memory they are a microsecond or two away, step by step
      uint32_t seen = 0;
      for (uint32_t i = 128u * (uint32_t)t; i < (uint32_t)SPC * C::STEP; i += 128u * kThreads)
        seen |= __builtin_amdgcn_raw_buffer_load_b32(a_rsrc, i, (int)a_off, 0);
      asm volatile("" : : "v"(seen));
      fill_a(1);
#pragma unroll 1
      for (int s = 0; s < SPC; ++s) {
        load_b(bv);
        run_step(0, bv);
      }
      cc = next;
      __syncthreads();
      if (cc < cc_end) patch_store(0, cc);
      __syncthreads();
    }
  } else if constexpr (C::BDEEP) {  // the next step's B operands are read at the start of a step
    static_assert(DEPTH == 1, "A one step ahead");
    u32x4 bX[NB][TERMS], bY[NB][TERMS];
    while (cc < cc_end) {
      begin_chunk();
      if (leave_out()) {
        jump_a(cc + 1);
        fill_a(DEPTH);
      } else {
        load_b(bX);
        for (int s = 0; s < SPC; s += 2) {
          load_b(bY);
          run_step(0, bX);
          if (s + 1 < SPC) {
            load_b(bX);
            run_step(0, bY);
          }
          count_steps(2);
        }
      }
      end_chunk();
    }
  } else {
    u32x4 bv[NB][TERMS];
    int s = 0;
    auto next_chunk = [&]() {
      if constexpr (KIND == HALF)
        if (leave_out()) {  // the steps go on, on zeros: leaving the ring of weights costs the registers of both ways
#pragma unroll
          for (int r = 0; r < EPT; ++r) {
            const uint32_t u = slot0 + r * kSlotStep;
            u32x4* dst = reinterpret_cast<u32x4*>(reinterpret_cast<char*>(smem) + (stage + POS * u));
            if (PIX || u < 2u * (uint32_t)a.PSZ) dst[0] = dst[TERM / 16] = u32x4{0, 0, 0, 0};
          }
          __syncthreads();
        }
      begin_chunk();
    };
    next_chunk();
    while (cc < cc_end) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d)
        if (cc < cc_end) {
          load_b(bv);
          run_step(d, bv);
          if (C::LEAD_STEPS) count_steps(1);
          if (++s == SPC) {
            s = 0;
            if (!C::LEAD_STEPS) count_steps(SPC);
            end_chunk();
            next_chunk();
          }
        }
    }
  }
  if constexpr (KIND == HALF) {
    const int w_scale = (int)a.scale[kSamples];
    int back[NB];  // what takes the powers of two out of the sums of a column
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const uint32_t col = col0 + (wn * NB + j) * MT + lane % MT;
      back[j] = -(image_scale(mdiv(col < col_last ? col : col_last, a.mP)) + w_scale);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
      left_out.bits[i] = (uint64_t)__builtin_amdgcn_readfirstlane(unheld[2 * i + 1]) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane(unheld[2 * i]);
#pragma unroll
    for (int q = 0; q < LEAD; ++q) {
      u32x4 w = {0, 0, 0, 0};
      if (led) w = lead[q * kThreads];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const int e = 8 * q + 2 * p, i = e / M::NR / NB, j = e / M::NR % NB, r = e % M::NR;
        // the small sums first: they are of the size of what the leading bits left
        float x = __builtin_fmaf(lo[i][j][r], kHalfDown, acc[i][j][r]), y = __builtin_fmaf(lo[i][j][r + 1], kHalfDown, acc[i][j][r + 1]);
        leading.give(w[p], x, y);
        acc[i][j][r] = scale_by(x, back[j]);
        acc[i][j][r + 1] = scale_by(y, back[j]);
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < M::NR; ++r) acc[i][j][r] = (acc[i][j][r] + lo[i][j][r]) * kSplitUnscale;
  }

  // ---- sums that are not finite once more on the fp32 matrix instructions (the weights put back together exactly, the
  // inputs as they are in memory): an infinity or NaN among the operands makes the split's differences NaN where the plain
  // sum may be infinite.  Every wave for itself, over the steps of the main loop: lane for lane an fp32 instruction takes the
  // e-th of the eight k values that the lane feeds to the bf16 one.  256 -> 384, 3x3 at 13x13, batch 128, forward: one NaN
  // 190 -> 490 us, all NaN 600 (with scalar multiply-adds 16 and 18 ms).  The f16 terms' sums have finite operands. ----
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < M::NR; ++r) bad |= not_finite(acc[i][j][r]);
  if (KIND != HALF && __any(bad)) {
    int ln = lane;
    asm volatile("" : "+v"(ln));  // what depends on it is computed here again, not kept in registers over the main loop
    const uint32_t kg = (uint32_t)ln / MT, hf = kg & 1;
    int row0[NB], col0s[NB];  // the column's window on the image (or the grid), and its image
    uint32_t img[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < M::NR; ++r) acc[i][j][r] = 0.f;
      uint32_t col = col0 + (wn * NB + j) * MT + (uint32_t)ln % MT;
      if (col > col_last) col = col_last;
      const uint32_t n = mdiv(col, a.mP);
      const uint32_t pix = col - n * a.P;
      const uint32_t pa = mdiv(pix, a.mPW);
      const uint32_t pb = pix - pa * a.PW;
      row0[j] = (int)pa * a.sh;
      col0s[j] = (int)pb * a.sw;
      img[j] = n * (uint32_t)a.in_img_stride + g * (uint32_t)a.in_grp_stride;
    }
    const int channels = FOLD || COLS ? a.fold.V : a.Cg_in;
    for (int ch = cc_first; ch < cc_end; ++ch) {
      if (KIND == AGAIN && !left_out.has(ch - cc_first)) continue;
      for (int st = 0; st < SPC; ++st) {
        const uint32_t off = (uint32_t)((ch - cc_first) * SPC + st) * C::STEP;
        const int tp = st * C::TPS + (int)(kg >> 1);  // (kg >> 1) is 0 for the 32-row instruction
        const int c0 = (COLS ? ch * 64 + tp * 16 : ch * 16) + (int)hf * 8;
        const int ti = COLS ? 0 : tp / a.TW, tj = COLS ? 0 : tp - ti * a.TW;
        float b[NB][8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          int ci = c0 + e, ir = 0, jr = 0;
          // Zero: channels past the group's last, the 16-row instruction's tap past the last, and places beyond the
          // kernel's taps (there the weight is zero, but the input may be what spoilt the sum).
          bool in = tp < T && ci < channels;
          if (FOLD) {
            const int v = ci;
            ci = v / a.fold.ff;
            ir = (v - ci * a.fold.ff) / a.fold.fw;
            jr = v - ci * a.fold.ff - ir * a.fold.fw;
            in = in && ti * a.fold.fh + ir < a.fold.kh && tj * a.fold.fw + jr < a.fold.kw;
          }
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            int ih = row0[j] + ti * a.dh, iw = col0s[j] + tj * a.dw;
            if (FOLD || COLS) {
              ih = ih * a.fold.Uh + ir * a.fold.dh;
              iw = iw * a.fold.Uw + jr * a.fold.dw;
            }
            ih -= a.ph;
            iw -= a.pw;
            const bool ok = in && (uint32_t)ih < (uint32_t)a.IH && (uint32_t)iw < (uint32_t)a.IW;
            const uint32_t at = 4u * (img[j] + (uint32_t)ci * (uint32_t)a.IHW + (uint32_t)ih * (uint32_t)a.IW + (uint32_t)iw);
            b[j][e] = __builtin_bit_cast(
                float, __builtin_amdgcn_raw_buffer_load_b32(in_rsrc, ok ? at : 0x80000000u, 0, 0));
          }
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          u32x4 w[3];
#pragma unroll
          for (int q = 0; q < 3; ++q)
            w[q] = __builtin_bit_cast(
                u32x4, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, 16u * (uint32_t)ln + (uint32_t)(wm * MB + i) * C::BLOCK + C::FIRST + q * C::FRAG, (int)off, 0));
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int sh = 16 * (e & 1);
            const uint16_t wh = (uint16_t)(w[0][e >> 1] >> sh), wmid = (uint16_t)(w[1][e >> 1] >> sh), wl = (uint16_t)(w[2][e >> 1] >> sh);
            const float v = join_bf16(wh, wmid, wl);
#pragma unroll
            for (int j = 0; j < NB; ++j) M::run(v, b[j][e], acc[i][j]);
          }
        }
      }
    }
  }

  corr_epilogue<MT, MB, NB, BM, BN>(a, smem, acc, m_tile, col_tile, g, wm, wn, split, KIND == AGAIN);
}

template <int MT, int MB, int NB, int WM, int WN, int EPT, SplitForm FORM, SplitTerms KIND>
__global__ __launch_bounds__(kThreads, (SplitCfg<MT, MB, NB, WM, WN, KIND, EPT>::WAVES)) void corr_split_kernel(const CorrSplitArgs a) {
  LeftOut left_out = {{0, 0}};
  corr_split<MT, MB, NB, WM, WN, EPT, FORM, KIND>(a, left_out);
  if constexpr (KIND == HALF)
    if (left_out.bits[0] | left_out.bits[1]) {
      __syncthreads();  // the epilogue's tables have been read
      corr_split<MT, MB, NB, WM, WN, EPT, FORM, AGAIN>(a, left_out);
    }
}

// Largest of a workgroup's sampled values, in bits.
template <int COUNT>
__device__ __forceinline__ uint32_t sample_top(const float (&v)[COUNT]) {
  __shared__ uint32_t top[4];
  uint32_t m = 0;
#pragma unroll
  for (int i = 0; i < COUNT; ++i) {
    const uint32_t u = sample_bits(v[i]);
    m = u > m ? u : m;
  }
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = (uint32_t)__shfl_xor((int)m, d);
    m = u > m ? u : m;
  }
  if ((threadIdx.x & 63) == 0) top[threadIdx.x >> 6] = m;
  __syncthreads();
  const uint32_t a = top[0] > top[1] ? top[0] : top[1], b = top[2] > top[3] ? top[2] : top[3];
  return a > b ? a : b;
}

// Packs the weights into A fragments: thread = (group, m tile, step, row block, lane), eight k values each.  Few
// workgroups whose time is one chain of index arithmetic, loads and stores: the divisions are per thread, not
// per k value (96 -> 256 in two groups, 5x5: 10.2 -> 7.4 us; 128 x 4096 rows: 7.2 -> 4.9).
// TERMS 2: the f16 split and, behind its fragments, the bf16 ones.  Every workgroup takes the weights' power of two from the same 2048
// of them; behind the packing ones a wave for each group of images leaves the largest of 1024 of its gathered values.
template <int MT, int TERMS>
__global__ __launch_bounds__(256) void pack_split_kernel(const PackSplitArgs a, int blocks, int m_tiles, uint32_t total) {
  const uint32_t idx = blockIdx.x * 256u + threadIdx.x;
  float sample[TERMS == 2 ? 8 : 1];
  const uint32_t pack_blocks = (total + 255u) / 256u;
  if constexpr (TERMS == 2) {
    if (blockIdx.x >= pack_blocks) {
      const uint32_t group = (idx >> 6) - pack_blocks * 4u, lane = idx & 63u, first = group * a.sample_elems;
      uint32_t top = 0, real = 0;
      if ((uint64_t)group * a.sample_elems < a.in_elems) {  // the whole wave
        const uint32_t left = a.in_elems - first, count = left < a.sample_elems ? left : a.sample_elems;
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // four neighbours each, spread evenly; of an image of less than four values, the last
          const uint32_t at = (uint32_t)((uint64_t)(4 * lane + i) * (count - (count < 4u ? count : 4u)) / 256u);
#pragma unroll
          for (uint32_t e = 0; e < 4; ++e) {
            const uint32_t u = sample_bits(a.in[first + (at + e < count ? at + e : count - 1u)]);
            top = u > top ? u : top;
            real += (uint32_t)__popcll(__ballot(u != 0));
          }
        }
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
          const uint32_t u = (uint32_t)__shfl_xor((int)top, d);
          top = u > top ? u : top;
        }
      }
      if (lane == 0) a.scale[group] = real < 32 ? top | kWeakSample : top;
      return;
    }
    const float* const at = a.w + (uint32_t)((uint64_t)threadIdx.x * (a.w_elems - 8u) / 256u);  // eight neighbours
#pragma unroll
    for (int i = 0; i < 8; ++i) sample[i] = at[i];
  }
  if (TERMS == 3 && idx >= total) return;
  const int lane = idx & 63;
  uint32_t lin = (idx < total ? idx : total - 1) >> 6;  // whole waves: total is a multiple of 64
  const int blk = (int)(lin % (uint32_t)blocks);
  lin /= (uint32_t)blocks;
  const int T = a.tTHW, tps = MT == 32 ? 1 : 2, spc = (T + tps - 1) / tps;
  const uint32_t steps = (uint32_t)(a.split_chunks * spc);
  const int step = (int)(lin % steps);
  lin /= steps;
  const int m_tile = (int)(lin % (uint32_t)m_tiles), g = (int)(lin / (uint32_t)m_tiles);
  const int m = (m_tile * blocks + blk) * MT + lane % MT, kgrp = lane / MT;
  const int chunk = step / spc, tap = (step % spc) * tps + (kgrp >> 1);
  const int subs = a.fold.subs, c0 = (subs ? chunk * subs + tap : chunk) * 16 + (kgrp & 1) * 8;
  const int fh = a.fold.fh, fw = a.fold.fw, khw = a.kh * a.kw;
  const bool row = m < a.Mrows && tap < T;
  // In the column form the tap is the group of channels and every tap is in the channel.
  const int it = subs ? 0 : tap / a.tTW, jt = subs ? 0 : tap - it * a.tTW;
  float v[8];
  if (a.fold.ff == 1) {  // one tap and a constant stride from channel to channel
    int ki = it, kj = jt, stride = khw;
    size_t at = ((size_t)g * a.Kg + m) * a.Cg * khw;
    bool in = row;
    if (a.mode) {  // backward data: phases of this row
      const int nv = a.nvh * a.nvw, mc = m / nv, mr = m - mc * nv;
      int rh = mr / a.nvw, rw = mr - rh * a.nvw;
      if (a.tab_h) rh = a.phase_h[rh];
      if (a.tab_w) rw = a.phase_w[rw];
      const int th = a.sh * a.eh * (a.Qh - 1 - it) + rh, tw = a.sw * a.ew * (a.Qw - 1 - jt) + rw;
      ki = th / a.dh;
      kj = tw / a.dw;
      in = in && ki * a.dh == th && kj * a.dw == tw;
      stride = a.Cg * khw;
      at = ((size_t)g * a.Kg * a.Cg + mc) * khw;
    }
    in = in && ki < a.kh && kj < a.kw;
    const float* const src = a.w + at + ki * a.kw + kj;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = in && c0 + e < a.fold.V ? src[(size_t)(c0 + e) * stride] : 0.f;
  } else {  // channel (c, ir, jr) and grid tap (it, jt) -> channel c under its tap (it*fh + ir, jt*fw + jr); forward only
    int c = c0 / a.fold.ff, jr = c0 - c * a.fold.ff, ir = jr / fw;
    jr -= ir * fw;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i = it * fh + ir, j = jt * fw + jr;
      const bool in = row && c0 + e < a.fold.V && i < a.kh && j < a.kw;
      v[e] = in ? a.w[(((size_t)g * a.Kg + m) * a.Cg + c) * khw + i * a.kw + j] : 0.f;
      if (++jr == fw) {
        jr = 0;
        if (++ir == fh) ir = 0, ++c;
      }
    }
  }
  char* dst = reinterpret_cast<char*>(a.A) + (size_t)(idx >> 6) * (TERMS == 2 ? 5120u : 3072u) + 16u * lane;
  if constexpr (TERMS == 2) {
    const int scale = half_scale(sample_top(sample));
    if (idx == 0) a.scale[kSamples] = (uint32_t)scale;
    if (idx >= total) return;
    float f[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = scale_by(v[e], scale);
    HalfRange range;
    range.add(f);
    const uint64_t unheld = __ballot(range.unheld());
    if (lane == 0) a.unheld[idx >> 6] = unheld != 0;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (!(__builtin_fabsf(f[e]) <= kHalfCeil)) f[e] = 0.f;  // finite terms, for chunks that are left out as zeros
    const SplitHalf8 s = split_half8(f);
    *reinterpret_cast<u32x4*>(dst) = s.h;
    *reinterpret_cast<u32x4*>(dst + 1024) = s.m;
    dst += 2048;
  }
  uint16_t out[3][8];
#pragma unroll
  for (int e = 0; e < 8; ++e) split1(v[e], out[0][e], out[1][e], out[2][e]);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    u32x4 v;
#pragma unroll
    for (int p = 0; p < 4; ++p) v[p] = (uint32_t)out[q][2 * p] | (uint32_t)out[q][2 * p + 1] << 16;
    *reinterpret_cast<u32x4*>(dst + q * 1024) = v;
  }
}

template <int MT, int MB, int NB, int WM, int WN, int EPT, SplitForm FORM, SplitTerms KIND>
int launch_split_k(const CorrSplitArgs& a, hipStream_t s) {
  using C = SplitCfg<MT, MB, NB, WM, WN>;
  const size_t tables = 16 * (C::BM + C::BN), plain = 96 * (size_t)a.PSZ;
  size_t lds = KIND == HALF ? (size_t)split_half_stage(EPT, FORM == PIXELS ? C::BN : 0) * a.patch_stages + split_half_lead(C::BM, C::BN) +
                                  (FORM == COLUMNS ? kUnheldBytes : 0)
                            : plain * a.patch_stages + (FORM == FOLDED ? a.NS * 16 * sizeof(FoldEntry) : 0);
  if (lds < tables) lds = tables;
  if (lds < plain) lds = plain;  // one stage for what HALF leaves out
  static LdsOptIn opt_in;  // more than 64 KB of LDS needs an explicit opt-in, once per process
  if (const int e = lds_opt_in(opt_in, &corr_split_kernel<MT, MB, NB, WM, WN, EPT, FORM, KIND>, 160 * 1024)) return e;
  const uint32_t blocks = (uint32_t)a.G * a.m_tiles * a.col_tiles * a.ksplit;
  hipLaunchKernelGGL((corr_split_kernel<MT, MB, NB, WM, WN, EPT, FORM, KIND>), dim3(blocks), dim3(kThreads), lds, s, a);
  return (int)hipGetLastError();
}

template <int MT, int MB, int NB, int WM, int WN, int EPT, SplitForm FORM = IMAGE>
int launch_split_e(const CorrSplitArgs& a, hipStream_t s) {
  if constexpr (FORM != FOLDED)
    if (a.half) return launch_split_k<MT, MB, NB, WM, WN, EPT, FORM, HALF>(a, s);
  if (a.half) return (int)hipErrorInvalidValue;
  return launch_split_k<MT, MB, NB, WM, WN, EPT, FORM, BF16>(a, s);
}

// The folded and the column forms: one instance per 128-column tile, for the largest patch; no rule leads a 1x1 kernel to
// the 32-row tile.
template <int MT, int MB, int NB, int WM, int WN>
int launch_split_t(const CorrSplitArgs& a, hipStream_t s) {
  constexpr int BM = SplitCfg<MT, MB, NB, WM, WN>::BM, BN = SplitCfg<MT, MB, NB, WM, WN>::BN;
  const int units = split_patch_units(a.PSZ + a.half, BN);
  if constexpr (BN <= 128 && BM >= 64) {
    if (a.fold.pixels) return launch_split_e<MT, MB, NB, WM, WN, 4, PIXELS>(a, s);
    if (a.fold.subs) return launch_split_e<MT, MB, NB, WM, WN, 4, COLUMNS>(a, s);
  }
  if constexpr (BN <= 128) {
    if (a.fold.ff > 1) return launch_split_e<MT, MB, NB, WM, WN, 4, FOLDED>(a, s);
    if (units == 2) return launch_split_e<MT, MB, NB, WM, WN, 2>(a, s);
  }
  if (a.fold.subs || a.fold.ff > 1) return (int)hipErrorInvalidValue;
  if (units == 3) return launch_split_e<MT, MB, NB, WM, WN, 3>(a, s);
  return launch_split_e<MT, MB, NB, WM, WN, 4>(a, s);
}

}  // namespace

void split_tile_shape(int32_t tile, int32_t* bm, int32_t* bn, int32_t* mt) {
  static const int32_t shapes[SPLIT_TILE_COUNT][3] = {
      {128, 128, 32}, {64, 256, 32}, {64, 128, 32}, {96, 128, 32}, {32, 256, 32}, {32, 128, 32}, {48, 256, 16}};
  *bm = shapes[tile][0];
  *bn = shapes[tile][1];
  *mt = shapes[tile][2];
}

int launch_corr_split(int32_t tile, const CorrSplitArgs& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (tile) {  //                             MT MB NB WM WN
    case SPLIT_128x128: return launch_split_t<32, 2, 2, 2, 2>(a, s);
    case SPLIT_64x256:  return launch_split_t<32, 2, 2, 1, 4>(a, s);
    case SPLIT_64x128:  return launch_split_t<32, 1, 2, 2, 2>(a, s);
    case SPLIT_96x128:  return launch_split_t<32, 3, 1, 1, 4>(a, s);
    case SPLIT_32x256:  return launch_split_t<32, 1, 2, 1, 4>(a, s);
    case SPLIT_32x128:  return launch_split_t<32, 1, 1, 1, 4>(a, s);
    case SPLIT_48x256:  return launch_split_t<16, 3, 4, 1, 4>(a, s);
    default: return (int)hipErrorInvalidValue;
  }
}

int launch_pack_split(int32_t tile, const PackSplitArgs& a, void* stream) {
  int32_t bm, bn, mt;
  split_tile_shape(tile, &bm, &bn, &mt);
  const int tps = mt == 32 ? 1 : 2, spc = (a.tTHW + tps - 1) / tps, blocks = bm / mt;
  const int m_tiles = (a.Mrows + bm - 1) / bm;
  const uint32_t total = (uint32_t)a.G * m_tiles * (uint32_t)(a.split_chunks * spc) * blocks * 64u;
  const dim3 grid((total + 255) / 256 + (a.half ? kSamples / 4 : 0));
  auto* const kernel = mt == 32 ? a.half ? pack_split_kernel<32, 2> : pack_split_kernel<32, 3>
                                : a.half ? pack_split_kernel<16, 2> : pack_split_kernel<16, 3>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, (hipStream_t)stream, a, blocks, m_tiles, total);
  return (int)hipGetLastError();
}

}  // namespace mi355conv
