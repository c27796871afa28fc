// Backward filter on the bf16 matrix instructions with fp32 operands split exactly in three (split_bf16.h):
//   dW_g[k][(c,i,j)] = sum over pixels (n,oh,ow) of dy[n, g*Kg + k, oh, ow] * x[n, g*Cg + c, oh*sh - ph + i*dh, ...]
// Same problem, split over the pixels and partial layout as wgrad_kernel (kernels_wgrad.hip), for layers whose input
// rows fit LDS.
//
// A workgroup takes 16 input channels and up to WN*NB taps of them: a block of 16 columns is one tap of the 16
// channels.  The reduction runs over runs of eight pixels of one image (an image's last run is filled up with
// zeros of dy), four runs = 32 pixels to a step, four steps to a chunk.  Per chunk the raw input rows its pixels
// touch are loaded, split and kept in LDS as [position][h, m, l][16 channels], 96 bytes per position; the matrix
// operand wants eight consecutive pixels of one channel per lane, which is what the transposing LDS read delivers:
// 16 lanes name four positions x 16 channels and each receives its channel at the four positions.  A position is
// split once and read by every tap.  dy runs are contiguous in memory in the order the operand wants: every
// wave loads and splits the runs of its own rows straight into registers, a step ahead.
//
// Bound by the matrix unit: 57.3 GFLOP (96 -> 256 in two groups, 5x5 at 27x27, batch 128) 494 -> 300 us, 38.3 GFLOP
// (256 -> 384, 3x3 at 13x13) 327 -> 200, 6.7 GFLOP (45 -> 77, 3x5 at 51x67, stride 2 x 1) 95 -> 67, 1.3 GFLOP (32 -> 32,
// 5x5 at 16x16, batch 100) 35 -> 23, with the reduce kernel, against wgrad_kernel; 172 and 115 us are the matrix
// instructions of the first two at the 2000 TFLOP/s that a loop of them sustains.
//
// HALF: long sums on two f16 terms (split_f16.h), half the matrix instructions, positions of 64 bytes.  Every workgroup samples
// both blobs for the powers of two while its first loads are under way.  The first three layers, without the reduce kernel: 349 ->
// 236 us, 219 -> 160, 67 -> 70 (its leading bits move every chunk), of which the test of every value is 6 to 8 %: each of a row's column tiles tests it again.
// AGAIN: what a workgroup's HALF sums had to leave out, step by step, it adds on the bf16 terms behind them.  128 -> 128, 3x3 at 56x56,
// batch 64: 228 us, with one image 2^-30 of the others 235, with every image of a size of its own 345, with one channel of x and one of dy
// 2^-30 of theirs, which leaves out every step, 474 (343 on bf16 terms alone).
// FOLD: the folded grid of corr_split_kernel, so that few channels fill the blocks: 3 -> 96 channels, 11x11, stride 4 at 227x227,
// batch 128, 290 us on the fp32 kernel -> 191; 9 -> 128, 12x12 at 109x150, batch 87, 265 -> 125.  Over 59 drawn layers that take it
// 1.36 times as fast in the geometric mean, none slower.
#include <hip/hip_runtime.h>

#include "device_utils.h"
#include "internal.h"
#include "split_bf16.h"
#include "split_f16.h"

namespace mi355conv {

namespace {

constexpr int kThreads = 256;
constexpr int kStepRuns = 4, kChunkSteps = 4, kChunkRuns = kStepRuns * kChunkSteps, kChunkPix = 8 * kChunkRuns;

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* LdsTrPtr;
typedef __attribute__((address_space(3))) char* LdsChar;

enum SplitTerms { BF16, HALF, AGAIN };  // three bf16 terms; two f16 terms; the bf16 terms of what those left out

// What HALF leaves for AGAIN: the blobs' powers of two, and the 128ths of the slice with chunks that AGAIN must look at -- a step that
// was left out it knows by the same test of the same values.
struct LeftOut {
  int x_scale, dy_scale;
  uint64_t bits[2];
  __device__ __forceinline__ bool has(int i) const { return (i < 64 ? bits[0] : bits[1]) >> (i & 63) & 1; }
};

// MB x NB blocks of 16 x 16 per wave; EPT: patch units (position x 8 channels) per thread; FOLD: the channels and taps are those of a
// folded grid (SplitFold).
template <int WM, int WN, int MB, int NB, int EPT, SplitTerms KIND, bool FOLD>
__device__ __forceinline__ void wgrad_split(const WgradSplitArgs& a, LeftOut& left_out) {
  using M = Mfma<16>;
  constexpr int BM = WM * MB * 16, TERMS = KIND == HALF ? 2 : 3;
  constexpr uint32_t POS = 32 * TERMS;  // bytes of a patch position
  static_assert(WM * WN == 4, "four waves per workgroup");

  extern __shared__ __align__(16) char smem[];  // position tables of two chunks, then one or two patch stages

  int t = threadIdx.x;
  uint32_t lin = xcd_contiguous_block_id();
  if constexpr (KIND == AGAIN) {  // what depends on these is computed here again, not kept in registers over the first sums
    asm volatile("" : "+v"(t));
    asm volatile("" : "+s"(lin));
  }
  const int lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  const int wm = wv / WN, wn = wv % WN;

  const uint32_t m_tile = lin % (uint32_t)a.m_tiles;
  lin /= (uint32_t)a.m_tiles;
  const uint32_t n_tile = lin % (uint32_t)a.n_tiles;
  lin /= (uint32_t)a.n_tiles;
  const uint32_t split = lin % (uint32_t)a.S;
  const uint32_t g = lin / (uint32_t)a.S;
  const int c16 = (int)(n_tile / (uint32_t)a.tap_tiles);
  const int tap0 = (int)(n_tile % (uint32_t)a.tap_tiles) * (WN * NB) + wn * NB;  // this wave's first tap

  const int chunk_first = (int)split * a.chunks_per_split;
  int chunk_end = chunk_first + a.chunks_per_split;
  if (chunk_end > a.chunks) chunk_end = a.chunks;

  // ---- x patch of a chunk ----
  const __amdgpu_buffer_rsrc_t x_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), 0, (int)a.x_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t dy_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.dy), 0, (int)a.dy_bytes, 0x00020000);
  const uint32_t chan_bytes = 4u * (uint32_t)(a.H * a.W);
  const uint32_t chan0 = (g * (uint32_t)a.Cg + (FOLD ? 0u : (uint32_t)c16 * 16u)) * chan_bytes;
  const uint32_t stage_bytes = POS * (uint32_t)a.PSZ;
  constexpr uint32_t kTables = 2u * 4u * kChunkPix;
  const int channels = FOLD ? a.fold.V : a.Cg;
  // behind the stages: leading bits, the numbers of the last two chunks whose patch is not held with the bits of left_out, the folded
  // form's table
  char* const behind = smem + kTables + (KIND == AGAIN ? 1u : (uint32_t)a.patch_stages) * stage_bytes;
  uint32_t* const unheld = reinterpret_cast<uint32_t*>(behind + (KIND == HALF ? split_half_lead(BM, WN * NB * 16) : 0));
  FoldEntry* const fold_tab = reinterpret_cast<FoldEntry*>(reinterpret_cast<char*>(unheld) + kUnheldWgradBytes);
  const int coarse = a.chunks_per_split > 128 ? 32 - __builtin_clz((uint32_t)(a.chunks_per_split - 1) >> 7) : 0;  // of the 128ths
  if (FOLD) {
    fill_fold_table(fold_tab, (a.n_tiles / a.tap_tiles) * 16, a.fold, a.W, a.H * a.W, t, kThreads);
    __syncthreads();
  }
  // (image, first pixel) of run q
  auto run_pos = [&](uint32_t q, uint32_t& n, uint32_t& p) {
    n = mdiv(q, a.mRuns);
    p = (q - n * (uint32_t)a.runs) * 8u;
  };
  float pr[EPT][8];
  uint32_t entry = 0;  // this thread's entry of the chunk's position table (threads below kChunkPix)
  // The chunk's first segment starts at output row a0 of image n0; its patch rows and those of later images are
  // counted as in corr_split_kernel.
  // A thread's units, from its number anew for every chunk: the f16 form has no registers for what depends on it, and a word that comes
  // back from scratch memory between the loads waits for those before it (128 -> 128, 3x3 at 56x56, batch 64: 309 us so, 226 now).
  auto unit0 = [&]() {
    uint32_t u = (uint32_t)t;
    if constexpr (KIND != BF16) asm volatile("" : "+v"(u));
    return u;
  };
  auto patch_load = [&](int chunk) {
    const uint32_t u0 = unit0();
    uint32_t q0 = (uint32_t)chunk * kChunkRuns, n0, p0;
    run_pos(q0, n0, p0);
    const uint32_t a0 = mdiv(p0, a.mPW);
    const uint32_t R0 = ((uint32_t)a.PH - 1 - a0) * a.sh + a.ext - a.share_h;
    const uint32_t RS = ((uint32_t)a.PH - 1) * a.sh + a.ext - a.share_h;
    {
      uint32_t n, p;
      run_pos(q0 + (u0 >> 3) % kChunkRuns, n, p);
      p += u0 & 7;
      if (p > (uint32_t)a.P - 1) p = (uint32_t)a.P - 1;  // filled-up run: any position, dy is zero
      if (n > (uint32_t)a.N - 1) n = n0, p = p0;         // past the last image: the same
      const uint32_t pa = mdiv(p, a.mPW), pb = p - pa * a.PW;
      const uint32_t s = n - n0;
      const uint32_t row = s == 0 ? (pa - a0) * a.sh : R0 + (s - 1) * RS + pa * a.sh;
      entry = POS * (row * (uint32_t)a.PWID + pb * a.sw);
    }
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const uint32_t u = u0 + r * kThreads;
      const uint32_t hf = u >= (uint32_t)a.PSZ ? 1u : 0u;
      const uint32_t e = u - hf * (uint32_t)a.PSZ;
      const uint32_t prow = mdiv(e, a.mPWID);
      const uint32_t pcol = e - prow * a.PWID;
      uint32_t n = n0, rin = prow, alo = a0;
      if (prow >= R0) {
        const uint32_t s1 = mdiv(prow - R0, a.mRSEG);
        n = n0 + 1 + s1;
        rin = prow - R0 - s1 * RS;
        alo = 0;
      }
      if (FOLD) {
        const int ih = (int)(alo * a.sh + rin) * a.fold.Uh - a.ph, iw = (int)pcol * a.fold.Uw - a.pw;
        const bool real = n < (uint32_t)a.N && u < 2u * (uint32_t)a.PSZ;
        load_folded(x_rsrc, fold_tab + (c16 * 16 + (int)hf * 8),
                    4u * (n * (uint32_t)(a.C * a.H * a.W) + (uint32_t)(ih * a.W + iw)) + chan0, real ? ih : -(1 << 28), iw, a.H, a.W, pr[r]);
        __builtin_amdgcn_sched_barrier(0);  // one unit's table entries in registers at a time
        continue;
      }
      const int ih = (int)(alo * a.sh + rin) - a.ph, iw = (int)pcol - a.pw;
      uint32_t src = 0x80000000u;  // beyond the blob (which is at most 2^30 bytes): reads as zero
      if ((uint32_t)ih < (uint32_t)a.H && (uint32_t)iw < (uint32_t)a.W && n < (uint32_t)a.N && u < 2u * (uint32_t)a.PSZ)
        src = 4u * (n * (uint32_t)(a.C * a.H * a.W) + (uint32_t)ih * a.W + iw) + chan0 + hf * 8u * chan_bytes;
      // channels past the group's last read the next group's or image's (or, past the blob, zero): columns never stored
#pragma unroll
      for (int c8 = 0; c8 < 8; ++c8)
        pr[r][c8] = __builtin_bit_cast(
            float, __builtin_amdgcn_raw_buffer_load_b32(x_rsrc, src + c8 * chan_bytes, 0, 0));
    }
  };
  const SplitSel sel;
  auto patch_store = [&](uint32_t table, uint32_t stage, int chunk) {
    HalfRange range;
    const uint32_t u0 = unit0();
    if (u0 < kChunkPix) *reinterpret_cast<uint32_t*>(smem + table + 4u * u0) = entry;
#pragma unroll
    for (int r = 0; r < EPT; ++r) {
      const uint32_t u = u0 + r * kThreads;
      const uint32_t hf = u >= (uint32_t)a.PSZ ? 1u : 0u;
      if (KIND != BF16 && !FOLD && c16 * 16 + 16 > a.Cg)  // need not be of a size with this group's
#pragma unroll
        for (int e = 0; e < 8; ++e) pr[r][e] = c16 * 16 + (int)hf * 8 + e < a.Cg ? pr[r][e] : 0.f;
      u32x4* dst = reinterpret_cast<u32x4*>(smem + kTables + stage + POS * (u - hf * (uint32_t)a.PSZ) + 16u * hf);
      if constexpr (KIND != BF16) {
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = scale_by(pr[r][e], left_out.x_scale);
        range.add(v);
        if constexpr (KIND == HALF) {
          const SplitHalf8 s = split_half8(v);
          if (u < 2u * (uint32_t)a.PSZ) {
            dst[0] = s.h;
            dst[2] = s.m;
          }
        }
      }
      if constexpr (KIND != HALF) {
        const Split8 s = split8(pr[r], sel);
        if (u < 2u * (uint32_t)a.PSZ) {
          dst[0] = s.h;
          dst[2] = s.m;
          dst[4] = s.l;
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // one unit's terms in registers at a time
    }
    if (KIND != BF16 && range.unheld()) unheld[chunk & 1] = (uint32_t)chunk + 1u;
  };

  // ---- dy: lane l takes run l/16 of a step and row l%16 of each of its wave's row blocks ----
  uint32_t arow[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    uint32_t m = m_tile * BM + (uint32_t)((wm * MB + i) * 16 + (lane & 15));
    if (m > (uint32_t)a.Kg - 1) m = (uint32_t)a.Kg - 1;  // rows past the edge are never stored
    arow[i] = 4u * (g * (uint32_t)a.Kg + m) * (uint32_t)a.P;
  }
  float raw[MB][8];
  int valid = 0;  // real pixels of the run in `raw`
  const uint32_t run_end = (uint32_t)a.N * (uint32_t)a.runs;
  auto load_dy = [&](int step) {  // step counted from chunk 0
    const uint32_t q = (uint32_t)step * kStepRuns + (uint32_t)(lane >> 4);
    uint32_t n, p;
    run_pos(q, n, p);
    valid = q < run_end ? a.P - (int)p : 0;
    const uint32_t base = q < run_end ? 4u * (n * (uint32_t)(a.Ktot * a.P) + p) : 0x80000000u;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const uint32_t off = base + arow[i];
      const u32x4 v0 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(dy_rsrc, off, 0, 0));
      const u32x4 v1 = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(dy_rsrc, off + 16u, 0, 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        raw[i][e] = __builtin_bit_cast(float, (uint32_t)v0[e]);
        raw[i][4 + e] = __builtin_bit_cast(float, (uint32_t)v1[e]);
      }
    }
  };

  M::Acc acc[MB][NB], lo[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < M::NR; ++r) acc[i][j][r] = lo[i][j][r] = 0.f;

  // uniform byte offset of each of this wave's taps inside the patch
  uint32_t tap_off[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    int tp = tap0 + j;
    if (tp > a.khw - 1) tp = a.khw - 1;  // blocks past the last tap are never stored
    const int ti = tp / a.kw, tj = tp - ti * a.kw;
    tap_off[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)POS * (ti * a.dh * a.PWID + tj * a.dw));
  }

  // ---- bias gradient from the same read of dy: every wave sums its rows over the chunks ch with
  // ch % (n_tiles*WN) == n_tile*WN + wn (see wgrad_kernel) ----
  const bool row_sums = a.bias_part != nullptr && KIND != AGAIN;
  const uint32_t turn = (uint32_t)(n_tile * WN + wn), turns = (uint32_t)(a.n_tiles * WN);
  float bsum[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) bsum[i] = 0.f;

  const bool two = a.patch_stages == 2 && KIND != AGAIN;
  // f16: the powers of two, from 2048 values of each blob, four neighbours at a time: those images' that the slice's runs belong to,
  // from anywhere in the image, a quarter of the slice a wave.  Images need not be of one size: a quarter alone 2^6 above the others
  // does not decide.
  auto sample_scales = [&]() {
    uint32_t top[2] = {0, 0};
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint32_t image = (uint32_t)(b ? a.Ktot * a.P : a.C * a.H * a.W), all = (b ? a.dy_bytes : a.x_bytes) / 4u;
      float v[8];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const uint32_t j = 2u * (uint32_t)t + i;
        uint32_t n, p;
        run_pos((uint32_t)chunk_first * kChunkRuns + (uint32_t)((uint64_t)j * (uint32_t)((chunk_end - chunk_first) * kChunkRuns) / (2 * kThreads)), n, p);
        if (n > (uint32_t)a.N - 1) n = (uint32_t)a.N - 1;
        uint32_t off = n * image + __umulhi(j * 2654435769u, image);
        if (off > all - 4u) off = all - 4u;
        const float* const at = (b ? a.dy : a.x) + off;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * i + e] = at[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const uint32_t u = sample_bits(v[e]);
        top[b] = u > top[b] ? u : top[b];
      }
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = (uint32_t)__shfl_xor((int)top[b], d);
        top[b] = u > top[b] ? u : top[b];
      }
    }
    uint32_t* const red = reinterpret_cast<uint32_t*>(smem);
    if (lane == 0) red[2 * wv] = top[0], red[2 * wv + 1] = top[1];
    __syncthreads();
    uint32_t best[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      uint32_t first = 0, second = 0;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t u = red[2 * w + b], below = u < first ? u : first;
        second = below > second ? below : second;
        first = u > first ? u : first;
      }
      best[b] = second != 0 && first - second > 6u << 23 ? second : first;
    }
    left_out.x_scale = __builtin_amdgcn_readfirstlane(half_scale(best[0]));
    left_out.dy_scale = __builtin_amdgcn_readfirstlane(half_scale(best[1]));
    __syncthreads();
  };
  // f16: every a.lead_chunks chunks the large sums' leading bits move to LDS, a place of its own for every lane.
  const Leading16 leading;
  bool led = false;
  uint2* const lead = reinterpret_cast<uint2*>(behind) + t;  // four sums, a block's, in eight bytes
  auto move_leading = [&]() {
#pragma unroll
    for (int b = 0; b < MB * NB; ++b) {
      M::Acc& c = acc[b / NB][b % NB];
      uint2 w = {0, 0};
      if (led) w = lead[b * kThreads];
      float v[4] = {c[0], c[1], c[2], c[3]};
      leading.give(w.x, v[0], v[1]);
      leading.give(w.y, v[2], v[3]);
      w.x = leading.take(v[0], v[1]);
      w.y = leading.take(v[2], v[3]);
#pragma unroll
      for (int r = 0; r < 4; ++r) c[r] = v[r];
      lead[b * kThreads] = w;
    }
    led = true;
  };
  int since = 0;
  auto following = [&](int i) {  // the next chunk
    do ++i;
    while (KIND == AGAIN && i < chunk_end && !left_out.has((i - chunk_first) >> coarse));
    return i;
  };
  int ch = following(chunk_first - 1);
  if (KIND != BF16 && t < (int)kUnheldWgradBytes / 4) unheld[t] = 0;
  if (KIND == AGAIN) __syncthreads();  // HALF's next barrier comes with the samples
  if (ch < chunk_end) {
    patch_load(ch);
    load_dy(ch * kChunkSteps);
    if constexpr (KIND == HALF) sample_scales();
    patch_store(0, 0, ch);
  }
  __syncthreads();

  const int last_step = chunk_end * kChunkSteps - 1;
  uint32_t stage = 0, table = 0;
  while (ch < chunk_end) {
    const int next = following(ch);
    const bool more = next < chunk_end;
    // a patch that is not held leaves out (HALF) or brings in (AGAIN) all steps of its chunk
    const bool patch_out = KIND != BF16 && __builtin_amdgcn_readfirstlane(unheld[ch & 1]) == (uint32_t)ch + 1u;
    if (more) patch_load(next);
    const bool my_turn = row_sums && (uint32_t)(ch - chunk_first) % turns == turn;
#pragma unroll 1
    for (int s = 0; s < kChunkSteps; ++s) {
      // positions of the two quads of pixels this lane names in the transposing reads, with its channel quad
      const uint32_t px = (uint32_t)s * 32u + (uint32_t)(lane >> 4) * 8u + (uint32_t)((lane & 15) >> 2);
      const uint32_t fix = kTables + stage + 8u * (uint32_t)(lane & 3);
      const uint32_t b0 = *reinterpret_cast<const uint32_t*>(smem + table + 4u * px) + fix;
      const uint32_t b1 = *reinterpret_cast<const uint32_t*>(smem + table + 4u * px + 16u) + fix;
      u32x4 bv[2][TERMS];
      auto load_b = [&](int j, u32x4(&b)[TERMS]) {
        const uint32_t o0 = b0 + tap_off[j], o1 = b1 + tap_off[j];
#pragma unroll
        for (int q = 0; q < TERMS; ++q) {
          const s16x4 x0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTrPtr)((LdsChar)smem + o0 + 32 * q));
          const s16x4 x1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LdsTrPtr)((LdsChar)smem + o1 + 32 * q));
          const uint2 y0 = __builtin_bit_cast(uint2, x0), y1 = __builtin_bit_cast(uint2, x1);
          b[q][0] = y0.x;
          b[q][1] = y0.y;
          b[q][2] = y1.x;
          b[q][3] = y1.y;
        }
      };
      // this step's dy operands: masked, summed, split; then the next step's loads.  Only an image's last run has anything to
      // mask: a test for the wave instead of a select per value, which the two multiplications of a split pair cost.
      u32x4 av[MB][TERMS];
      HalfRange range;
      if (__any(valid < 8)) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 8; ++e) raw[i][e] = e < valid ? raw[i][e] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const float(&v)[8] = raw[i];
        if (my_turn) bsum[i] += ((v[0] + v[1]) + (v[2] + v[3])) + ((v[4] + v[5]) + (v[6] + v[7]));
        if constexpr (KIND != BF16) {
          float scaled[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) scaled[e] = scale_by(v[e], left_out.dy_scale);
          if constexpr (KIND == HALF) {
            const SplitHalf8 sp = split_half8(scaled);
            av[i][0] = sp.h;
            av[i][1] = sp.m;
            asm volatile("" : "+v"(av[i][1]));  // here, or the operands stay in registers until the test below is decided
          }
          range.add(scaled);
        }
        if constexpr (KIND != HALF) {
          const Split8 sp = split8(v, sel);
          av[i][0] = sp.h;
          av[i][1] = sp.m;
          av[i][2] = sp.l;
        }
      }
      const int step = ch * kChunkSteps + s;
      load_dy(s + 1 < kChunkSteps ? step + 1 : more ? next * kChunkSteps : step);
      if constexpr (KIND != BF16) {
        const bool left = patch_out || __any(range.unheld());
        if (KIND == HALF && left && lane == 0)
          atomicOr(unheld + 2 + ((ch - chunk_first) >> coarse >> 5), 1u << ((ch - chunk_first) >> coarse & 31));
        if (left == (KIND == HALF)) continue;
      }
      load_b(0, bv[0]);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if (j + 1 < NB) load_b(j + 1, bv[(j + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);  // the next block's reads before this block's products, not behind them
        if constexpr (KIND == HALF) {
#pragma unroll
          for (int i = 0; i < MB; ++i) mfma_f16<16>(av[i][1], bv[j & 1][0], lo[i][j]);
#pragma unroll
          for (int i = 0; i < MB; ++i) mfma_f16<16>(av[i][0], bv[j & 1][0], acc[i][j]);
#pragma unroll
          for (int i = 0; i < MB; ++i) mfma_f16<16>(av[i][0], bv[j & 1][1], lo[i][j]);
        } else {
          constexpr int pa[5] = {2, 0, 1, 1, 0}, pb[5] = {0, 2, 1, 0, 1};
#pragma unroll
          for (int q = 0; q < 5; ++q)
#pragma unroll
            for (int i = 0; i < MB; ++i) mfma_bf16<16>(av[i][pa[q]], bv[j & 1][pb[q]], lo[i][j]);
#pragma unroll
          for (int i = 0; i < MB; ++i) mfma_bf16<16>(av[i][0], bv[j & 1][0], acc[i][j]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (KIND == HALF && ++since == a.lead_chunks && more) {
      move_leading();
      since = 0;
    }
    table ^= 4u * kChunkPix;
    if (two)
      stage = stage ? 0 : stage_bytes;
    else
      __syncthreads();
    if (more) patch_store(table, stage, next);
    ch = next;
    __syncthreads();
  }

  if (row_sums) {  // uniform over the grid; LDS is free after the loop's last barrier
    float* red = reinterpret_cast<float*>(smem);  // [WN][BM]
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      float v = bsum[i];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (lane < 16) red[wn * BM + (wm * MB + i) * 16 + lane] = v;
    }
    __syncthreads();
    for (int row = t; row < BM; row += kThreads) {
      float total = red[row];
#pragma unroll
      for (int v = 1; v < WN; ++v) total += red[v * BM + row];
      const uint32_t k = m_tile * BM + (uint32_t)row;
      if (k < (uint32_t)a.Kg) a.bias_part[((size_t)split * a.n_tiles + n_tile) * a.Ktot + g * a.Kg + k] = total;
    }
  }

  if constexpr (KIND == HALF) {
    const int back = -(left_out.x_scale + left_out.dy_scale);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      left_out.bits[i] = (uint64_t)__builtin_amdgcn_readfirstlane(unheld[2 * i + 3]) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane(unheld[2 * i + 2]);
#pragma unroll
    for (int b = 0; b < MB * NB; ++b) {
      M::Acc& c = acc[b / NB][b % NB];
      const M::Acc& l = lo[b / NB][b % NB];
      uint2 w = {0, 0};
      if (led) w = lead[b * kThreads];
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = __builtin_fmaf(l[r], kHalfDown, c[r]);
      leading.give(w.x, v[0], v[1]);
      leading.give(w.y, v[2], v[3]);
#pragma unroll
      for (int r = 0; r < 4; ++r) c[r] = scale_by(v[r], back);
    }
  } else {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int r = 0; r < M::NR; ++r) acc[i][j][r] = (acc[i][j][r] + lo[i][j][r]) * kSplitUnscale;
  }

  const int c = c16 * 16 + (lane & 15);
  // ---- sums that are not finite once more on the fp32 matrix instructions (see corr_split_kernel), behind f16 sums the whole slice's;
  // channels past the group's last are the next group's and never stored ----
  bool bad = false;
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < M::NR; ++r) bad |= not_finite(acc[i][j][r]);
  const bool redo = KIND != HALF && __any(bad && c < channels);
  if (redo) {
    int th[NB], tw[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) {
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int r = 0; r < M::NR; ++r) acc[i][j][r] = 0.f;
      int tp = tap0 + j;
      if (tp > a.khw - 1) tp = a.khw - 1;
      th[j] = __builtin_amdgcn_readfirstlane(tp / a.kw * a.dh);
      tw[j] = __builtin_amdgcn_readfirstlane(tp % a.kw * a.dw);
    }
#pragma unroll 1
    for (int step = chunk_first * kChunkSteps; step <= last_step; ++step) {
      load_dy(step);
      uint32_t n, p;
      run_pos((uint32_t)step * kStepRuns + (uint32_t)(lane >> 4), n, p);
      int ci = c, ir = 0, jr = 0;  // the channel and the tap within its fold
      if (FOLD) {
        ci = c / a.fold.ff;
        ir = (c - ci * a.fold.ff) / a.fold.fw;
        jr = c - ci * a.fold.ff - ir * a.fold.fw;
      }
      const uint32_t image = n * (uint32_t)(a.C * a.H * a.W) + (g * (uint32_t)a.Cg + (uint32_t)ci) * (uint32_t)(a.H * a.W);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const bool real = e < valid && c < channels;
        const uint32_t pix = p + e, pa = mdiv(pix, a.mPW), pb = pix - pa * a.PW;
        const int ih0 = (int)pa * a.sh - (FOLD ? 0 : a.ph), iw0 = (int)pb * a.sw - (FOLD ? 0 : a.pw);
        float b[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          int ih = ih0 + th[j], iw = iw0 + tw[j];
          if (FOLD) {
            ih = ih * a.fold.Uh + ir * a.fold.dh - a.ph;
            iw = iw * a.fold.Uw + jr * a.fold.dw - a.pw;
          }
          const bool ok = real && (uint32_t)ih < (uint32_t)a.H && (uint32_t)iw < (uint32_t)a.W;
          b[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                               x_rsrc, ok ? 4u * (image + (uint32_t)ih * (uint32_t)a.W + (uint32_t)iw) : 0x80000000u, 0, 0));
        }
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const float v = e < valid ? raw[i][e] : 0.f;
#pragma unroll
          for (int j = 0; j < NB; ++j) M::run(v, b[j], acc[i][j]);
        }
      }
    }
  }

  // ---- partial block -> workspace [split][g][k][tap][c], the order in which the lanes of a store are neighbours (16
  // channels, 64 bytes; as [k][c][tap] every lane of a store opened a line of its own, and a 32-row layer with 20 MB
  // of partials took 42 us instead of 20); the reduce kernel puts them into the weight blob's order.  Rows, channels and
  // taps past the edge carry offsets beyond the slice (at most 2^30 bytes): the range check of the store drops them. ----
  float* dst = a.part + (size_t)split * a.part_stride + (size_t)g * ((size_t)a.Kg * a.Kred);
  const __amdgpu_buffer_rsrc_t out_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(dst, 0, (int)(4u * (uint32_t)a.Kg * (uint32_t)a.Kred), 0x00020000);
  auto each = [&](auto&& act) {
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int r = 0; r < M::NR; ++r) {
        const uint32_t k = m_tile * BM + (uint32_t)((wm * MB + i) * 16 + M::row(r, lane));
        const uint32_t ro = k < (uint32_t)a.Kg && c < channels ? 4u * (k * (uint32_t)a.Kred + (uint32_t)c) : 0x80000000u;
#pragma unroll
        for (int j = 0; j < NB; ++j) act(i, j, r, ro + (tap0 + j < a.khw ? 4u * (uint32_t)((tap0 + j) * channels) : 0x40000000u));
      }
  };
  if (KIND == AGAIN && !redo)  // all loads before the stores, which they would wait for one by one
    each([&](int i, int j, int r, uint32_t off) {
      acc[i][j][r] += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(out_rsrc, off, 0, 0));
    });
  each([&](int i, int j, int r, uint32_t off) {
    const float v = acc[i][j][r];
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(int, v), out_rsrc, off, 0, 0);
  });
}

template <int WM, int WN, int MB, int NB, int EPT, SplitTerms KIND, bool FOLD>
__global__ __launch_bounds__(kThreads, 2) void wgrad_split_kernel(const WgradSplitArgs a) {
  LeftOut left_out = {0, 0, {0, 0}};
  wgrad_split<WM, WN, MB, NB, EPT, KIND, FOLD>(a, left_out);
  if constexpr (KIND == HALF)
    if (left_out.bits[0] | left_out.bits[1]) {
      __syncthreads();  // LDS is free
      wgrad_split<WM, WN, MB, NB, EPT, AGAIN, FOLD>(a, left_out);
    }
}

template <int WM, int WN, int MB, int NB, int EPT, SplitTerms KIND, bool FOLD = false>
int launch_k(const WgradSplitArgs& a, hipStream_t s) {
  constexpr int BM = WM * MB * 16;
  const size_t tables = 2 * 4 * kChunkPix, red = 4 * WN * BM;
  const size_t behind = (KIND == HALF ? kUnheldWgradBytes : 0) + (FOLD ? (a.n_tiles / a.tap_tiles) * 16 * sizeof(FoldEntry) : 0);
  size_t lds = tables + (KIND == HALF ? 64 : 96) * (size_t)a.PSZ * a.patch_stages + (KIND == HALF ? split_half_lead(BM, WN * NB * 16) : 0) + behind;
  const size_t again = tables + 96 * (size_t)a.PSZ + behind;  // one stage for what HALF leaves out
  if (lds < again) lds = again;
  static LdsOptIn opt_in;  // more than 64 KB of LDS needs an explicit opt-in, once per process
  if (const int e = lds_opt_in(opt_in, &wgrad_split_kernel<WM, WN, MB, NB, EPT, KIND, FOLD>, 160 * 1024)) return e;
  const uint32_t blocks = (uint32_t)a.G * a.S * a.m_tiles * a.n_tiles;
  hipLaunchKernelGGL((wgrad_split_kernel<WM, WN, MB, NB, EPT, KIND, FOLD>), dim3(blocks), dim3(kThreads), lds > red ? lds : red, s, a);
  return (int)hipGetLastError();
}

template <int WM, int WN, int MB, int NB, int EPT>
int launch_e(const WgradSplitArgs& a, hipStream_t s) {
  return a.half ? launch_k<WM, WN, MB, NB, EPT, HALF>(a, s) : launch_k<WM, WN, MB, NB, EPT, BF16>(a, s);
}

template <int WM, int WN, int MB, int NB>
int launch_t(const WgradSplitArgs& a, hipStream_t s) {
  if (split_patch_units(a.PSZ) == 2) return launch_e<WM, WN, MB, NB, 2>(a, s);
  if (split_patch_units(a.PSZ) == 3) return launch_e<WM, WN, MB, NB, 3>(a, s);
  return launch_e<WM, WN, MB, NB, 4>(a, s);
}

// The folded form, f16 terms only.
template <int WM, int WN, int MB, int NB>
int launch_f(const WgradSplitArgs& a, hipStream_t s) {
  if (split_patch_units(a.PSZ) <= 3) return launch_k<WM, WN, MB, NB, 3, HALF, true>(a, s);
  return launch_k<WM, WN, MB, NB, 4, HALF, true>(a, s);
}

}  // namespace

void wgrad_split_shape(int32_t tile, int32_t* rows, int32_t* taps) {
  static const int32_t shapes[WSPLIT_TILE_COUNT][2] = {{128, 9}, {128, 8}, {64, 16}, {32, 28}, {32, 12}, {96, 8}};
  *rows = shapes[tile][0];
  *taps = shapes[tile][1];
}

void wgrad_fold_shape(int32_t tile, int32_t* rows, int32_t* taps) {
  static const int32_t shapes[WFOLD_TILE_COUNT][2] = {{96, 10}, {128, 9}, {64, 16}, {32, 12}};
  *rows = shapes[tile][0];
  *taps = shapes[tile][1];
}

int launch_wgrad_fold(int32_t tile, const WgradSplitArgs& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (tile) {  //                      WM WN MB NB
    case WFOLD_96x10: return launch_f<2, 2, 3, 5>(a, s);
    case WFOLD_128x9: return launch_f<4, 1, 2, 9>(a, s);
    case WFOLD_64x16: return launch_f<2, 2, 2, 8>(a, s);
    case WFOLD_32x12: return launch_f<1, 4, 2, 3>(a, s);
    default: return (int)hipErrorInvalidValue;
  }
}

int32_t wgrad_split_chunk_runs() { return kChunkRuns; }

int launch_wgrad_split(int32_t tile, const WgradSplitArgs& a, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (tile) {  //                     WM WN MB NB
    case WSPLIT_128x9: return launch_t<4, 1, 2, 9>(a, s);
    case WSPLIT_128x8: return launch_t<4, 1, 2, 8>(a, s);
    case WSPLIT_64x16: return launch_t<2, 2, 2, 8>(a, s);
    case WSPLIT_32x28: return launch_t<1, 4, 2, 7>(a, s);
    case WSPLIT_32x12: return launch_t<1, 4, 2, 3>(a, s);
    case WSPLIT_96x8:  return launch_t<2, 2, 3, 4>(a, s);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace mi355conv
