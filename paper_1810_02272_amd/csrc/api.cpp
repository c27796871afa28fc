// Host side of the C boundary: parameter validation, shape arithmetic, kernel-variant choice,
// workspace sizing and the five entry points.  No device memory is allocated anywhere here, and
// conv_desc_create touches no device at all (it also runs on machines without a GPU).
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <new>

#include "internal.h"

using namespace mi355conv;

namespace {

thread_local int g_last_hip_error = 0;

constexpr int64_t kMaxElems = (int64_t)1 << 30;  // 32-bit byte offsets in the kernels

int64_t floor_div(int64_t a, int64_t b) {
  int64_t q = a / b;
  if ((a % b) != 0 && ((a < 0) != (b < 0))) --q;
  return q;
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t round_up(int64_t a, int64_t b) { return ceil_div(a, b) * b; }
// For the loops over tiles and slices, which a descriptor runs by the hundred: a 64-bit division takes several times as long.
uint32_t parts_of(int64_t a, uint32_t b) { return ((uint32_t)a + b - 1) / b; }

// Row tile: the smallest padded row count wins; a taller tile is taken over a shorter one when it
// pads at most 3 % more rows (the 32-row MFMA tiles it brings are worth that).  Column tile, among
// the variants of that height: the one with the smallest estimated makespan on 256 compute
// units -- rounds of workgroups times tile width -- with a 6 % handicap per halving of the
// width (narrow tiles re-read the packed weights more often per FLOP).  A mid-sized grid of a large
// problem may split its reduction (configure_ksplit): the estimate then takes the best split of each
// width, so that a wide tile in three slices can beat a narrow one that leaves the last round a third
// full (256 -> 384 channels, 3x3 at 13x13, backward data: 128x128 in 3 slices 325-334 us, 128x64
// unsplit 341).  Tiles that the patch-staged kernel may take (may_patch: the gather is one it can
// stage) are left out: that kernel does not split.
int32_t pick_corr_tile(int32_t rows, int64_t groups, int64_t ncols, int64_t kred, int64_t taps, bool may_patch) {
  int64_t best_pad = 0, best_bm = 0;
  for (int32_t t = 0; t < CORR_TILE_COUNT; ++t) {
    int32_t bm, bn, bk;
    corr_tile_shape(t, &bm, &bn, &bk);
    const int64_t pad = round_up(rows, bm);
    if (best_bm == 0 || pad < best_pad || (pad == best_pad && bm > best_bm)) {
      best_pad = pad;
      best_bm = bm;
    }
  }
  const int64_t min_pad = best_pad;
  for (int32_t t = 0; t < CORR_TILE_COUNT; ++t) {
    int32_t bm, bn, bk;
    corr_tile_shape(t, &bm, &bn, &bk);
    const int64_t pad = round_up(rows, bm);
    if (bm > best_bm && pad * 100 <= min_pad * 103) {
      best_pad = pad;
      best_bm = bm;
    }
  }
  int32_t best = -1;
  double best_cost = 0;
  for (int32_t t = 0; t < CORR_TILE_COUNT; ++t) {
    int32_t bm, bn, bk;
    corr_tile_shape(t, &bm, &bn, &bk);
    if (bm != best_bm) continue;
    const int64_t units = groups * (best_pad / bm) * ceil_div(ncols > 0 ? ncols : 1, bn);
    double cost = (double)ceil_div(units, 256) * bn;
    const int64_t chunks = ceil_div(kred, bk);
    const bool patch_tile = may_patch && ((bn == 256 && bm <= 48) || (taps >= 25 && bn == 128 && (bm == 128 || bm == 32)));
    if (units > 160 && units < 512 && !patch_tile && 2.0 * rows * (double)kred * (double)ncols * (double)groups >= 5e9)
      for (int64_t c = 2; c <= 8 && chunks / c >= 16; ++c) {  // the splits configure_ksplit may take
        const double split_cost = (double)ceil_div(units * c, 256) * bn / (double)c * (1.0 + 0.01 * (double)c);
        if (split_cost < cost) cost = split_cost;
      }
    for (int32_t w = bn; w < 256; w *= 2) cost *= 1.06;
    if (best < 0 || cost < best_cost) {
      best = t;
      best_cost = cost;
    }
  }
  return best;
}

// Thin groups.  The GEMM path pads a group's rows to 16 and its reduction to 16, so its cost per
// group is that of 16 x round_up(Cg*taps, 16) however few of them are real; the direct kernels cost
// Kg*Cg*taps multiply-adds per position at roughly a fifth of the matrix unit's rate for the 3x3 and
// 5x5 forms and a tenth for the general one (measured: 3x3 with 4 channels in and out per group is
// 1.8x faster direct, with 8 in and out 2x slower).
bool direct_is_faster(int64_t cg, int64_t kg, int64_t kh, int64_t kw) {
  const int64_t taps = kh * kw;
  const int64_t gemm = round_up(kg, 16) * round_up(cg * taps, 16);
  const bool rows_form = (kh == 3 && kw == 3) || (kh == 5 && kw == 5);
  return kg * cg * taps * (rows_form ? 5 : 10) <= gemm;
}

int32_t pick_wgrad_tile(int32_t rows, int32_t kred) {
  int32_t best = -1;
  int64_t best_work = 0, best_area = 0;
  for (int32_t t = 0; t < WGRAD_TILE_COUNT; ++t) {
    int32_t bm, bn, bk;
    wgrad_tile_shape(t, &bm, &bn, &bk);
    int64_t work = round_up(rows, bm) * round_up(kred, bn);
    const int64_t area = (int64_t)bm * bn;
    // a narrower tile must save at least 8 % of the padded work to be worth its extra LDS traffic
    if (best < 0 || work * 100 < best_work * 92 || (work <= best_work && area > best_area)) {
      best = t;
      best_work = work;
      best_area = area;
    }
  }
  return best;
}

// How the gather zeroes out-of-image elements (see corr_kernel): 0 = no padding at all and the blob
// below 2^31 bytes; 2 = at most 32 taps and the blob at most 2^29 bytes; 1 = anything else.
// `reach` = how far (bytes) a tap of a real column can point outside the blob: mode 2 adds
// 2^30 / 2^31 to such offsets and must neither wrap nor come back inside.
int32_t bounds_mode(bool no_padding, int64_t taps, int64_t bytes, int64_t reach) {
  if (no_padding && bytes < ((int64_t)1 << 31) - 4) return 0;
  if (taps <= 32 && bytes <= ((int64_t)1 << 29) && reach < ((int64_t)1 << 28)) return 2;
  return 1;
}

// One spatial dimension of the backward-data rewriting.  Input position x + pad = stride*a + r
// collects the taps i with i*dilation = stride*q + r from dy position a - q.
//  - Only the phases r in { i*dilation mod stride : i < kernel } are reached by any tap; when that
//    is a proper subset of 0 .. stride-1 of at most kMaxPhases values, the row space keeps only
//    those (a 1x1 stride-2 layer: one phase of four) and the rest of dx is zero-filled.
//  - When the stride divides the dilation (stride 1 included) the only phase is 0 and the taps sit
//    e = dilation/stride positions apart: kernel slots instead of (kernel-1)*dilation/stride + 1.
struct PhaseDim {
  int64_t Q, e, nv;
  int32_t tab;
  int32_t phase[kMaxPhases];
};

PhaseDim phase_dim(int64_t kernel, int64_t stride, int64_t dilation) {
  PhaseDim r = {};
  if (dilation % stride == 0) {
    r.Q = kernel;
    r.e = dilation / stride;
  } else {
    r.Q = (kernel - 1) * dilation / stride + 1;
    r.e = 1;
  }
  int64_t found = 0;
  int32_t vals[kMaxPhases];
  for (int64_t i = 0; i < kernel && found <= kMaxPhases; ++i) {
    const int32_t v = (int32_t)((i * dilation) % stride);
    bool seen = false;
    for (int64_t j = 0; j < found && j < kMaxPhases; ++j) seen = seen || vals[j] == v;
    if (!seen) {
      if (found < kMaxPhases) vals[found] = v;
      ++found;
    }
  }
  if (found >= stride || found > kMaxPhases) {  // every phase reached, or too many to tabulate
    r.nv = stride;
    r.tab = 0;
    return r;
  }
  for (int64_t i = 1; i < found; ++i)  // ascending order
    for (int64_t j = i; j > 0 && vals[j - 1] > vals[j]; --j) {
      const int32_t t = vals[j];
      vals[j] = vals[j - 1];
      vals[j - 1] = t;
    }
  r.nv = found;
  r.tab = 1;
  for (int64_t i = 0; i < found; ++i) r.phase[i] = vals[i];
  return r;
}

// "tile[m<bounds mode>,e<epilogue form>](S=<splits>,L=<launches>)", or "tile_patch[e.](S=1,L=2)" for the
// patch-staged kernel.
// Epilogue forms: s = separable byte offsets, r = range-checked stores with a compare per element,
// p = plain pointers (output of 2^31 bytes or more).
// L = kernel launches of the pass: the pack kernel, a zero fill (backward data with unreached
// phases), the main kernel, the reduce kernel of a split launch.
void corr_variant_name(char* buf, size_t len, int32_t tile, const CorrArgs& a, int zero_fill, int thin) {
  const char e = a.simple_epilogue ? 's' : ((uint32_t)a.out_elems < (1u << 29) ? 'r' : 'p');
  const int launches = 2 + (a.ksplit > 1) + (zero_fill != 0);
  if (thin && a.use_patch)  // rows staged in LDS, TW x TW taps unrolled, weights read in place: no pack kernel
    snprintf(buf, len, "corr_thin_r%d_lds%d[e%c](S=1,L=%d)", a.Mrows, a.TW, e, launches - 1);
  else if (thin)
    snprintf(buf, len, "corr_thin_r%d[m%d,e%c](S=1,L=%d)", a.Mrows, a.bounds_mode, e, launches);
  else if (a.use_patch)
    snprintf(buf, len, "%s_patch[e%c](S=%d,L=%d)", corr_tile_name(tile), e, a.ksplit, launches);
  else
    snprintf(buf, len, "%s[m%d,e%c](S=%d,L=%d)", corr_tile_name(tile), a.bounds_mode, e, a.ksplit, launches);
}

// "corrsplit_<tile>[p<patch units per thread>, fold<taps per channel>, cols or rows<channel groups>,e<epilogue form>](S,L)",
// with "half" before L for the f16 split
void split_variant_name(char* buf, size_t len, int32_t tile, const CorrSplitArgs& a, int zero_fill) {
  int32_t bm, bn, mt;
  split_tile_shape(tile, &bm, &bn, &mt);
  const char e = a.simple_epilogue ? 's' : ((uint32_t)a.out_elems < (1u << 29) ? 'r' : 'p');
  snprintf(buf, len, "corrsplit_m%d_%dx%d[%s%d,e%c](S=%d,%sL=%d)", mt, bm, bn, a.fold.subs ? a.fold.pixels ? "rows" : "cols" : a.fold.ff > 1 ? "fold" : "p",
           a.fold.subs ? a.fold.subs : a.fold.ff > 1 ? a.fold.ff : split_patch_units(a.PSZ + a.half, bn), e,
           a.ksplit, a.half ? "half," : "", 2 + (a.ksplit > 1) + (zero_fill != 0));
}

// "<kernel>_<rows>x<columns>x<waves>[w<how the weights are read>, or v<16-byte loads of x>](S,L)"
void small_variant_name(char* buf, size_t len, const char* kernel, const SmallTile& t, int32_t mode, int32_t S, int32_t launches) {
  snprintf(buf, len, "%s_%dx%dx%d[%c%d](S=%d,L=%d)", kernel, 16 * t.mb, 16 * t.nb, t.waves, kernel[0] == 'c' ? 'w' : 'v', mode, S, launches);
}

// Puts the names of the passes that the one-launch kernels take in place of the others' (which: 0 floats, 1 doubles).
void small_names(const conv_desc* d, int which, char* fwd, char* bwd, char* wg, size_t len) {
  const char* const corr = which ? "corrsmall64" : "corrsmall";
  if (d->fwd_small[which] >= 0)
    small_variant_name(fwd, len, corr, kCorrSmallTiles[d->fwd_small[which]], d->fwd_sm[which].wmode, 1, 1);
  if (d->bwd_small[which] >= 0)
    small_variant_name(bwd, len, corr, kCorrSmallTiles[d->bwd_small[which]], d->bwd_sm[which].wmode, 1, 1 + (d->bwd_zero_fill != 0));
  if (d->wg_small[which] >= 0)
    small_variant_name(wg, len, which ? "smallwgrad64" : "smallwgrad", kWgradSmallTiles[d->wg_small[which]], d->wg_sm[which].xvec,
                       d->wg_sm[which].S, 1 + (d->wg_sm[which].S > 1));
}

// Places of a channel up to which one workgroup sums them and finishes db of doubles: 2.6 to 3.5 us up to 6000 places where the
// two launches took 4.1 to 9.2, 5.1 to 12.8 against 5.8 to 17.2 at 21632, no longer ahead at 25088 (5.6 and 5.3, 32 channels).
constexpr int64_t kBias64Direct = 24576;

uint32_t koff_invalid(int32_t mode) { return mode == 0 ? 0x7FFFFFFCu : mode == 2 ? 0x40000000u : 0u; }

// Decides whether the patch-staged kernel runs this correlation and, if so, fills its fields.
// Used where the gather kernel's per-element work is largest: the 256-column tiles of at most 48 rows
// (measured: 5x5 grouped backward-data +9 %), and two 128-column tiles for kernels of 25 taps or more.
// Needs a stride-1, dilation-1 gather, 8-aligned channels per group, at least 3 taps, a blob of at
// most 2^30 bytes, and a patch that fits kPatchEPT*256 floats per channel and the LDS.
void configure_patch(CorrArgs& a, PackArgs& k, int64_t cg_in, int64_t n_img, int32_t bm, int32_t bn) {
  a.use_patch = 0;
  k.kperm_T = 0;
  const int64_t T = a.THW, TH = a.THW / a.TW;
  if (a.sh != 1 || a.sw != 1 || a.dh != 1 || a.dw != 1 || cg_in % 8 != 0 || T < 3) return;
  // 256-column tiles of at most 48 rows; with 25 taps or more also the 128x128 and 32x128 tiles, on grids
  // that the gather kernel would not split (measured with 5x5 kernels: 128x128 forward 451 -> 443 us,
  // 32x128 38 -> 34 us; with 3x3 kernels the gather kernel stays ahead, 298 -> 305 us)
  const bool wide = bn == 256 && bm <= 48;
  const bool many_taps = T >= 25 && bn == 128 && (bm == 128 || bm == 32) &&
                         (int64_t)a.G * a.m_tiles * a.col_tiles > 160;
  if (!wide && !many_taps) return;
  if ((int64_t)a.in_bytes > ((int64_t)1 << 30) || a.ncols < 1) return;
  const int64_t PH = a.P / a.PW, PWID = a.PW + a.TW - 1, RS = PH + TH - 1;
  // largest patch over all column tiles
  int64_t max_rows = 0;
  for (int64_t c0 = 0; c0 < a.ncols; c0 += bn) {
    const int64_t c1 = (c0 + bn < a.ncols ? c0 + bn : a.ncols) - 1;
    const int64_t n0 = c0 / a.P, a0 = (c0 % a.P) / a.PW, n1 = c1 / a.P, a1 = (c1 % a.P) / a.PW;
    const int64_t R0 = PH - a0 + TH - 1;
    const int64_t rows = (n1 == n0 ? a1 - a0 : R0 + (n1 - n0 - 1) * RS + a1) + TH;
    if (rows > max_rows) max_rows = rows;
  }
  // Channel stride of the patch in LDS.  At one MFMA step the four lane groups of a wave read four
  // channels 2*psz floats apart, 16 consecutive positions each: a stride of 8 mod 16 puts those
  // four runs on different banks.
  int64_t psz = max_rows * PWID;
  psz += (8 - psz % 16 + 16) % 16;
  const int64_t lds = (2 * (int64_t)bm * 20 + 16 * psz) * 4;
  if (psz > kPatchEPT * 256 || lds > 80 * 1024 || lds < 16 * ((int64_t)bm + bn)) return;
  a.use_patch = 1;
  a.Cg_in = (int32_t)cg_in;
  a.NS = (int32_t)(cg_in / 8 * T);
  a.PH = (int32_t)PH;
  a.Nimg = (int32_t)n_img;
  a.PWID = (int32_t)PWID;
  a.PSZ = (int32_t)psz;
  a.mPWID = make_magic((uint32_t)PWID);
  a.mRSEG = make_magic((uint32_t)RS);
  k.kperm_T = (int32_t)T;
}

// Split of the reduction: with few workgroups and a long chunk loop the chip idles while each
// workgroup walks its chunks one barrier at a time; S slices run side by side and a reduce kernel
// adds them.  Worth an extra launch when the grid is well under one workgroup per compute unit,
// or when a large problem leaves the compute units unevenly loaded.
// bm x bn: the tile; elem_bytes: 4 or 8 (the double path runs the same rule on its own tiles).
void configure_ksplit(CorrArgs& a, int64_t out_elems, int32_t bm, int32_t bn, int32_t elem_bytes = 4) {
  a.ksplit = 1;
  a.chunks_per_split = a.KP / 16;
  a.out_elems = (int32_t)out_elems;
  a.simple_epilogue = a.RShw == 1 && a.tab_h == 0 && a.tab_w == 0 && 4 * out_elems <= ((int64_t)1 << 30);
  const int64_t units = (int64_t)a.G * a.m_tiles * a.col_tiles, chunks = a.KP / 16;
  if (a.use_patch || chunks < 8 || a.ncols < 1) return;
  int64_t S = 1;
  const double flops = 2.0 * a.Mrows * a.Kred * (double)a.ncols * a.G;
  if (units <= 160 && flops < 2e9) {
    // Small grid of a small problem: the number of slices with the smallest modelled time.  A
    // workgroup that has its compute unit to itself walks its chunks at the latency of one chunk --
    // 0.18 us plus 0.30 us per 4096 tile elements (twice that in doubles) -- and S slices cost the
    // reduce kernel's launch, 1.6 us, plus their partial sums written and read once at 2.4 TB/s
    // (0.83 us per MB).  Constants fitted to split sweeps of the nine such passes of the benchmark's
    // small layers (rms error 1 us; the model picks the fastest or second fastest S on each: 2.a
    // forward, 32 chunks on 64 tiles of 64x64, 0.8 MB out: 4 slices 13.4 us against 14.6 with 8 and
    // 21.7 unsplit; 3.a forward, 16 chunks on 100 tiles, 1.6 MB out: unsplit 14.4 us against 18.0
    // with 4).  At most 16 slices of at least two chunks, at most 1024 workgroups.
    const double t_chunk = 0.18 + 0.30 * (elem_bytes == 8 ? 2.0 : 1.0) * (double)(bm * bn) / 4096.0;
    const double out_mb = (double)out_elems * elem_bytes / 1e6;
    double best_t = (double)chunks * t_chunk;
    for (int64_t c = 2; c <= 16 && c <= chunks / 2 && units * c <= 1024; ++c) {
      const double t = (double)ceil_div(chunks, c) * t_chunk + 1.6 + 0.83 * (double)c * out_mb;
      if (t < best_t) {
        best_t = t;
        S = c;
      }
    }
  } else if (units <= 160) {
    // Small grid of a larger problem (the matrix pipes, not latency, set the pace once the slices
    // fill the chip): two workgroups per compute unit, at least four chunks per slice
    S = ceil_div(512, units);
    if (S > chunks / 4) S = chunks / 4;
    if (S > 16) S = 16;
    // a long reduction carries twice as many slices as long as each keeps 32 chunks (the 9216 -> 4096
    // InnerProduct backward-data pass: 144 tiles, 256 chunks, 4 -> 8 slices, 118 -> 105 us)
    int64_t S2 = ceil_div(1024, units);
    if (S2 > chunks / 32) S2 = chunks / 32;
    if (S2 > 16) S2 = 16;
    if (S2 > S) S = S2;
  } else if (units < 512 && flops >= 5e9) {
    // Mid-sized grids of a large problem (a 14x14 or 7x7 layer with hundreds of channels): one or
    // two workgroups per compute unit with some units idle.  Take the split that brings the load
    // of the busiest unit, relative to the unsplit grid, down by at least 15 % (20 % when the
    // unsplit grid already has two workgroups on some units; 1 % per slice charged for the partial
    // sums); every slice keeps at least 16 chunks.
    const double base = (double)ceil_div(units, 256);
    double best = base > 1.0 ? 0.80 : 0.85;
    for (int64_t c = 2; c <= 8 && chunks / c >= 16; ++c) {
      const double ratio = (double)ceil_div(units * c, 256) / ((double)c * base) * (1.0 + 0.01 * (double)c);
      if (ratio < best) {
        best = ratio;
        S = c;
      }
    }
  }
  if (S < 2) return;
  a.chunks_per_split = (int32_t)ceil_div(chunks, S);
  a.ksplit = (int32_t)ceil_div(chunks, a.chunks_per_split);
}

// GEMMs of at most four rows per group (backward data of a layer with one to four input channels
// per group at stride 1, forward with that few outputs) with the offset-only epilogue take
// corr_thin_kernel: one lane per column, scalar A operands, no matrix unit -- the 16-row tiles
// spend three quarters or more of their matrix instructions on padding there.  The packed operand
// and the k table stay as they are (natural k order); the reduction is not split.
int32_t configure_thin(CorrArgs& a, PackArgs& k, int64_t cg_in, int64_t n_img, bool backward) {
  if (a.Mrows > 4 || !a.simple_epilogue || a.ncols < 1) return 0;
  a.use_patch = 0;
  k.kperm_T = 0;
  a.ksplit = 1;
  a.chunks_per_split = a.KP / 16;
  // A stride-1, dilation-1 gather with 3x3 or 5x5 taps whose rows fit LDS takes the staged form: 128
  // columns per workgroup, all channels of the group at once, the patch of the largest tile (geometry
  // of configure_patch) at most 512 floats per channel and 64 KB in all.  It reads its A operands
  // from the weight blob (output channel, input channel, tap): forward rows are output channels and
  // the gathered channels inputs; backward data the other way round with the taps reversed.
  const int64_t T = a.THW, w_grp = (int64_t)a.Mrows * cg_in * T;
  if (a.sh == 1 && a.sw == 1 && a.dh == 1 && a.dw == 1 && (a.TW == 3 || a.TW == 5) && T == a.TW * a.TW &&
      (int64_t)a.in_bytes <= ((int64_t)1 << 30) && w_grp * a.G < ((int64_t)1 << 31)) {
    const int64_t bn = 128, TH = a.TW;
    const int64_t PH = a.P / a.PW, PWID = a.PW + a.TW - 1, RS = PH + TH - 1;
    int64_t max_rows = 0;
    for (int64_t c0 = 0; c0 < a.ncols; c0 += bn) {
      const int64_t c1 = (c0 + bn < a.ncols ? c0 + bn : a.ncols) - 1;
      const int64_t n0 = c0 / a.P, a0 = (c0 % a.P) / a.PW, n1 = c1 / a.P, a1 = (c1 % a.P) / a.PW;
      const int64_t R0 = PH - a0 + TH - 1;
      const int64_t rows = (n1 == n0 ? a1 - a0 : R0 + (n1 - n0 - 1) * RS + a1) + TH;
      if (rows > max_rows) max_rows = rows;
    }
    const int64_t psz = max_rows * PWID;
    if (psz <= 512 && cg_in * psz * 4 <= 64 * 1024) {
      a.use_patch = 1;
      a.Cg_in = (int32_t)cg_in;
      a.NS = 0;
      a.PH = (int32_t)PH;
      a.Nimg = (int32_t)n_img;
      a.PWID = (int32_t)PWID;
      a.PSZ = (int32_t)psz;
      a.mPWID = make_magic((uint32_t)PWID);
      a.mRSEG = make_magic((uint32_t)RS);
      a.w_grp_stride = (int32_t)w_grp;
      a.w_row_stride = (int32_t)(backward ? T : cg_in * T);
      a.w_chan_stride = (int32_t)(backward ? a.Mrows * T : T);
      a.w_reversed = backward ? 1 : 0;
    }
  }
  return 1;
}

// One dimension of an LDS patch (corr_split_kernel, wgrad_split_kernel): `out` positions `stride` apart with windows of
// `ext` positions over an image of `size` positions behind `pad` zeros.  `share` of the zeros behind the image, which
// some window reads, are the same ones as those before the next row (image): `pitch` positions from row to row.  At most a
// window's worth: a tile that starts in an image's last row owns ext - share rows of that image.
struct PatchDim {
  int64_t pitch, share;
};

PatchDim patch_dim(int64_t out, int64_t stride, int64_t ext, int64_t pad, int64_t size) {
  const int64_t reach = (out - 1) * stride + ext, behind = reach - pad - size;
  PatchDim r;
  r.share = behind <= 0 || pad <= 0 ? 0 : behind < pad ? behind : pad;
  if (r.share > ext) r.share = ext;
  r.pitch = reach - r.share;
  return r;
}

// The most patch rows that any tile needs: tiles of `tile` units -- `unit` output positions of an image of P -- over `total`
// units, `per_image` to an image (its last unit may be short).  Ends where the tiles' starts repeat, where `enough` rows are
// passed and where no tile can need more: walking all 3025 tiles of 128 images of 55x55 took 40 us for each tile shape.
int64_t max_patch_rows(int64_t total, int64_t per_image, int64_t tile, int64_t unit, int64_t P, int64_t PW, int64_t stride,
                       int64_t ext, int64_t pitch, int64_t enough) {
  const int64_t PH = P / PW, extra = pitch - PH * stride, crossed = (per_image + tile - 2) / per_image;
  const int64_t bound = (PW - 1 + tile * unit - 1) / PW * stride + (extra > 0 ? extra * crossed : 0) + ext;
  int64_t most = 0, rest = total;
  uint32_t r = 0;  // the tile's first unit within its image
  do {
    const uint32_t last = r + (uint32_t)(rest < tile ? rest : tile) - 1, images = last / (uint32_t)per_image;
    const int64_t end = (int64_t)(last - images * (uint32_t)per_image) * unit + unit - 1;
    const int64_t a0 = r * (uint32_t)unit / (uint32_t)PW, a1 = (uint32_t)(end < P ? end : P - 1) / (uint32_t)PW;
    const int64_t rows = images * pitch + (a1 - a0) * stride + ext;
    if (rows > most) most = rows;
    r = (r + (uint32_t)tile) % (uint32_t)per_image;
    rest -= tile;
  } while (rest > 0 && r != 0 && most < bound && most <= enough);
  return most;
}

// The grid that corr_split_kernel walks (SplitFold in internal.h).
struct SplitGrid {
  SplitFold f;
  int64_t sh, sw, dh, dw, TH, TW;  // strides, dilations and taps on the grid
};

void plain_grid(int64_t cg, int64_t kh, int64_t kw, int64_t sh, int64_t sw, int64_t dh, int64_t dw, SplitGrid& g) {
  g = SplitGrid();
  g.f.fh = g.f.fw = g.f.ff = g.f.Uh = g.f.Uw = 1;
  g.f.dh = (int32_t)dh;
  g.f.dw = (int32_t)dw;
  g.f.kh = (int32_t)kh;
  g.f.kw = (int32_t)kw;
  g.f.V = (int32_t)cg;
  g.f.mFF = g.f.mFw = make_magic(1);
  g.sh = sh;
  g.sw = sw;
  g.dh = dh;
  g.dw = dw;
  g.TH = kh;
  g.TW = kw;
}

// The tile's columns, for 1x1 kernels.
void column_grid(int64_t cg, int64_t sh, int64_t sw, SplitGrid& g) {
  plain_grid(cg, 1, 1, 1, 1, 1, 1, g);
  g.f.subs = 4;
  g.f.Uh = (int32_t)sh;
  g.f.Uw = (int32_t)sw;
  g.TH = 4;  // the groups of 16 channels
}

// Layers whose few channels would leave the 16-channel chunks mostly empty.  Per dimension the taps stay, or the `stride`
// taps between two positions of a grid of every stride-th pixel are folded (undilated layers), or all of them are; of the
// nine combinations with at least three taps left (a patch is staged per 16 channels and read once per tap) the one that
// pads the reduction least.  Only where four channels are one 16-byte load -- 3 channels, 11x11, stride 4: 48 channels and
// 3x3 taps, 432 reduction indices for 363, 241 -> 195 us; with single loads the patch costs more than the matrix unit
// gains (3 channels, 5x5 at 64x64: 36 us fp32, 44 folded) -- and up to 1.25 times the reduction.
bool folded_grid(int64_t cg, int64_t kh, int64_t kw, int64_t sh, int64_t sw, int64_t dh, int64_t dw, int64_t pw,
                 SplitGrid& g) {
  plain_grid(cg, kh, kw, sh, sw, dh, dw, g);
  struct Dim {
    int64_t f, U, taps, s, d;
  };
  auto options = [](int64_t k, int64_t s, int64_t d, Dim* o) {
    int n = 0;
    o[n++] = {1, 1, k, s, d};
    if (s > 1 && d == 1) o[n++] = {s, s, ceil_div(k, s), 1, 1};
    o[n++] = {k, s, 1, 1, 1};
    return n;
  };
  Dim oh[3], ow[3];
  const int nh = options(kh, sh, dh, oh), nw = options(kw, sw, dw, ow);
  int64_t best = 0;
  for (int i = 0; i < nh; ++i)
    for (int j = 0; j < nw; ++j) {
      const int64_t V = cg * oh[i].f * ow[j].f, T = oh[i].taps * ow[j].taps, padded = round_up(V, 16) * T;
      if (oh[i].f * ow[j].f == 1 || T < 3 || (best && padded >= best)) continue;
      best = padded;
      g.f.fh = (int32_t)oh[i].f;
      g.f.fw = (int32_t)ow[j].f;
      g.f.Uh = (int32_t)oh[i].U;
      g.f.Uw = (int32_t)ow[j].U;
      g.f.V = (int32_t)V;
      g.sh = oh[i].s;
      g.sw = ow[j].s;
      g.dh = oh[i].d;
      g.dw = ow[j].d;
      g.TH = oh[i].taps;
      g.TW = ow[j].taps;
    }
  if (!best || best * 4 > cg * kh * kw * 5 || g.f.V > 512 || kh * dh > 16384 || kw * dw > 16384) return false;
  g.f.ff = g.f.fh * g.f.fw;
  g.f.mFF = make_magic((uint32_t)g.f.ff);
  g.f.mFw = make_magic((uint32_t)g.f.fw);
  return g.f.fw % 4 == 0 && g.f.Uw % 4 == 0 && dw == 1 && pw % 4 == 0;
}

// Whether sums of K products take f16 terms: where their error (squares of 2-norms in units of 2^-24) can be brought to `most`.  Returns
// the steps (of `step` indices, in whole `unit`s) between two moves of the sums' leading bits, or 0 for bf16 terms.  A move costs time
// (every 128 indices instead of 400: 57.3 GFLOP 160 -> 176 us), so the stretches are as long as `aim` allows.  The f16 terms' error
// is the operands', which zeros among the inputs leave as it is, the rounding of the sums within a stretch, and that of the moves.
int32_t half_interval(double K, double most, double aim, double step, int32_t unit) {
  auto error = [&](int32_t steps) {
    const double part = (double)steps * step < K ? (double)steps * step : K;
    return 2.4 + 0.0085 * part + 0.04 * K / part;
  };
  int32_t steps = unit;
  while ((double)steps * step < 112) steps += unit;
  if (error(steps) > most) return 0;
  while ((double)steps * step < K && error(steps + unit) < aim) steps += unit;
  return steps;
}

// The bf16 terms' error an index: without zeros, with a blob of half zeros, as behind a ReLU, and with two (a filter gradient whose dy
// came back through one).  Zeros add no rounding to a sum.  f16 terms are taken where they are no further off without zeros, those of
// a layer's own padding apart, and about a tenth further off at most with a blob of half zeros; an InnerProduct layer's data gradient,
// whose dz came back through its ReLU, takes them where they are no further off then.  The stretches are such that sums of about 750
// indices and more are no further off with half zeros, in the filter gradient of 2000 and more with half zeros in both blobs.
// Measured, bf16 -> f16 terms, without zeros, with half of both blobs zero, and with nine tenths:
//   3x3 forward, K = 648: 2.38 -> 1.99, 1.83 -> 1.98, 0.94 -> 1.80; 864: 2.81 -> 2.08, 2.17 -> 2.07, 1.06 -> 1.83;
//   1152: 3.26 -> 2.38, 2.53 -> 2.38, 1.20 -> 1.99; 2304: 4.79 -> 3.31, 3.77 -> 3.31, 1.68 -> 2.59;
//   filter gradient, 759 a slice: 2.90 -> 2.34, 1.90 -> 2.30, 1.29 -> 1.92; 1024: 3.25 -> 2.54, 2.03 -> 2.44, 1.22 -> 1.88;
//   896: 3.05 -> 2.33, 1.95 -> 2.28, 1.24 -> 1.89;
//   2404: 4.89 -> 2.92, 2.80 -> 2.76, 1.06 -> 1.80; 3584: 6.13 -> 3.68, 3.59 -> 3.50, 1.17 -> 1.91.
// None of these is above what the bf16 terms lose without zeros.  70 layers drawn like those of perf/cases.py, 114 outputs that differ: f16
// terms 0.76 of the bf16 terms' error in the geometric mean, 0.96 at most (biases, whose sums only changed their order, 1.03).
constexpr double kBf16Full = 0.0085, kBf16Half = 0.0052, kBf16BothHalf = 0.0035, kHalfMost = 1.15 * kBf16Half;

// Share of positions x taps that lie inside the image: the others are zeros.
double inside_image(int64_t positions, int64_t stride, int64_t taps, int64_t dilation, int64_t pad, int64_t size) {
  int64_t inside = 0;
  for (int64_t t = 0; t < taps; ++t)
    for (int64_t p = 0; p < positions; ++p) {
      const int64_t at = p * stride + t * dilation - pad;
      inside += at >= 0 && at < size;
    }
  return (double)inside / (double)(positions * taps);
}

// half_interval for corr_split_kernel: `cps` of `chunks` chunks of T taps in a slice, where bf16 terms would add up `bf16_cps`.  The
// tiles that hold several steps' weights move the leading bits between chunks only.
int32_t corr_half_interval(const CorrArgs& base, int32_t tile, int32_t mt, int64_t T, int64_t chunks, int64_t cps, int64_t bf16_cps,
                           double inside) {
  if (cps > kUnheldChunks) return 0;
  const int32_t step = mt == 32 ? 16 : 32;
  const bool by_chunk = tile == SPLIT_64x128 || tile == SPLIT_32x256 || tile == SPLIT_32x128;
  const double chunk = (double)base.Kred / (double)chunks;
  const bool inner_product = base.THW == 1 && base.IH == 1 && base.ncols == base.P;  // one image of one row: its data gradient's form
  const double bf16_K = chunk * (double)bf16_cps, most = inner_product ? kBf16Half : std::min(kHalfMost, kBf16Full * inside);
  return half_interval(chunk * (double)cps, most * bf16_K, 0.9 * kBf16Half * bf16_K, step, by_chunk ? (int32_t)ceil_div(16 * T, step) : 2);
}

// Tile and split count of corr_split_kernel on one grid by modelled time (us); tile < 0: the patch fits none.
// The workgroup that finishes last walks its steps alone on its compute unit (kAlone per step) or shares it with others
// (kShared per step and workgroup); a chunk costs its patch by units per thread; S slices cost the reduce kernel and their
// partial sums written and read.  The constants are a least-squares fit to 888 timings -- all tiles, 1 to 12 slices, 38
// layers of 0.3 to 57 GFLOP (rms error 8 %); the choice is 2 % behind the best of each layer on average, 13 % at worst.  Those of
// the f16 terms to 1072 timings of 40 passes of 1 to 57 GFLOP (7 %; 2 % and 12 %).
struct SplitPlan {
  int32_t tile, half;
  int64_t psz, S, units;  // units: output tiles
  int64_t bf16_cps;       // chunks of a slice on bf16 terms
  double inside;          // share of the products that are none of padding
  double cost;  // modelled time without the launches and the prologue, about 10 us
  PatchDim w, h;
};

SplitPlan plan_split(const CorrArgs& base, const SplitGrid& grid, int64_t out_elems, bool half, int64_t bf16_S) {
  struct Costs {
    double alone[SPLIT_TILE_COUNT], shared[SPLIT_TILE_COUNT], patch_alone, patch_shared, slices, slice_mb;
  };
  static const Costs kCosts[2] = {{{0.457, 0.444, 0.414, 0.376, 0.400, 0.298, 0.664}, {0.423, 0.424, 0.250, 0.340, 0.248, 0.166, 0.613}, 0.39, 0.25, 3.3, 0.46},
                                  {{0.356, 0.358, 0.309, 0.301, 0.300, 0.250, 0.494}, {0.260, 0.265, 0.165, 0.227, 0.175, 0.118, 0.387}, 0.19, 0.154, 1.8, 0.472}};
  const Costs& c = kCosts[half];
  SplitPlan plan = {};
  plan.tile = -1;
  plan.half = half;
  const bool columns = grid.f.subs != 0, image = grid.f.ff == 1 && !columns;
  const int64_t chunks = ceil_div(grid.f.V, columns ? 64 : 16);
  const int64_t T = grid.TH * grid.TW, PH = base.P / base.PW, ext = (grid.TH - 1) * grid.dh + 1;
  if (!columns) {
    plan.w = patch_dim(base.PW, grid.sw, (grid.TW - 1) * grid.dw + 1, image ? base.pw : 0, base.IW);
    plan.h = patch_dim(PH, grid.sh, ext, image ? base.ph : 0, base.IH);
  }
  plan.bf16_cps = bf16_S ? ceil_div(chunks, bf16_S) : 0;
  plan.inside = half && image ? inside_image(base.PW, grid.sw, grid.TW, grid.dw, base.pw, base.IW) *
                                    inside_image(PH, grid.sh, grid.TH, grid.dh, base.ph, base.IH)
                              : 1;
  const double out_mb = 4e-6 * (double)out_elems;
  double best = 0;
  for (int32_t t = 0; t < SPLIT_TILE_COUNT; ++t) {
    int32_t bm, bn, mt;
    split_tile_shape(t, &bm, &bn, &mt);
    if (!image && (bn > 128 || (columns && bm < 64))) continue;  // the folded and column forms are built for these
    int64_t psz = 4 * bn;
    if (!columns) {
      const int64_t max_rows = max_patch_rows(base.ncols, base.P, bn, 1, base.P, base.PW, grid.sh, ext, plan.h.pitch,
                                              512 / plan.w.pitch);
      psz = max_rows * plan.w.pitch + plan.w.share;
    }
    if (psz + (half && image) > 512) continue;  // with kUnheldBytes
    const int64_t units = (int64_t)base.G * ceil_div(base.Mrows, bm) * ceil_div(base.ncols, bn);
    const int64_t spc = ceil_div(T, mt == 32 ? 1 : 2);
    const double units_per_thread = image ? (double)split_patch_units(psz + half, bn) : 4.0;
    for (int64_t S = 1; S <= 16 && S <= chunks; ++S) {
      // Of grids that fill the chip, f16 terms take the least number of slices of at most kUnheldChunks (4096 -> 4096, 3x3 at 13x13,
      // batch 16, forward: 5258 us on bf16 terms, 3647 in two slices).
      if (S > 1 && (units * S > 2048 || units > 512) && !(half && ceil_div(chunks, S - 1) > kUnheldChunks)) break;
      const int64_t per_cu = ceil_div(units * S, 256), cps = ceil_div(chunks, S);
      if (half && !corr_half_interval(base, t, mt, T, chunks, cps, plan.bf16_cps, plan.inside)) continue;
      const double steps = (double)(cps * spc);
      double cost = per_cu == 1 ? steps * c.alone[t] + c.patch_alone * (double)cps * units_per_thread
                                : (double)per_cu * (steps * c.shared[t] + c.patch_shared * (double)cps * units_per_thread);
      if (S > 1) cost += c.slices + c.slice_mb * (double)S * out_mb;
      if (plan.tile < 0 || cost < best) {
        best = plan.cost = cost;
        plan.tile = t;
        plan.psz = psz;
        plan.S = S;
        plan.units = units;
      }
    }
  }
  return plan;
}

// Fragments of packed weights of a plan (row blocks x steps), and what they take in the workspace: three KB each on bf16 terms, on
// f16 terms five, a word, and the samples.
int64_t split_fragments(const CorrArgs& base, const SplitGrid& grid, int32_t tile) {
  int32_t bm, bn, mt;
  split_tile_shape(tile, &bm, &bn, &mt);
  return base.G * ceil_div(base.Mrows, bm) * (bm / mt) * ceil_div(grid.f.V, grid.f.subs ? 64 : 16) *
         ceil_div(grid.TH * grid.TW, mt == 32 ? 1 : 2);
}

int64_t split_pack_bytes(int64_t fragments, bool half) {
  return half ? fragments * 5120 + round_up(4 * fragments, 512) + kSampleBytes : fragments * 3072;
}

// The cheaper of the two splits.  The f16 one's pack kernel samples both blobs: 3 us more, and 0.26 us a MB of weights.
SplitPlan plan_split(const CorrArgs& base, const SplitGrid& grid, int64_t out_elems) {
  const SplitPlan bf16 = plan_split(base, grid, out_elems, false, 0);
  if (bf16.tile < 0 || grid.f.ff > 1) return bf16;
  SplitPlan f16 = plan_split(base, grid, out_elems, true, bf16.S);
  if (f16.tile < 0) return bf16;
  if (split_pack_bytes(split_fragments(base, grid, f16.tile), true) + (f16.S > 1 ? 4 * f16.S * out_elems : 0) >= 4 * kMaxElems) return bf16;
  f16.cost += 3 + 0.26 * 4e-6 * (double)base.G * base.Mrows * base.Kred;
  return f16.cost < bf16.cost ? f16 : bf16;
}

// Decides whether corr_split_kernel runs this correlation; fills a, k and the tile.  Returns the bytes of packed
// weights, 0 if it does not.
size_t configure_split(const CorrArgs& base, const PackArgs& pbase, int64_t cg_in, int64_t n_img, int64_t out_elems,
                       CorrSplitArgs& a, PackSplitArgs& k, int32_t& tile) {
  tile = -1;
  const double flops = 2.0 * base.Mrows * base.Kred * (double)base.ncols * base.G;
  if (base.ncols < 1 || (int64_t)base.in_bytes > ((int64_t)1 << 30)) return 0;
  // Below a GFLOP the two paths are level (100 x 32 -> 64 at 8x8, 5x5, 0.66 GFLOP: 19.4 us fp32, 20.8 split; one image of
  // 96 -> 256 in two groups at 27x27, 0.45 GFLOP: 22.2 and 20.8), the patch-staged fp32 kernel keeps reductions under 512,
  // and so do the 16-row fp32 tiles what fits them (8 rows on 32-row instructions: 36 us fp32, 66 split; 12 rows: 51 and 64).
  if (flops < 1e9 || base.Mrows <= 16 || base.Kred < (base.use_patch ? 512 : 128)) return 0;
  const int64_t kh = base.THW / base.TW, kw = base.TW;
  SplitGrid grid;
  SplitPlan plan = {};
  plan.tile = -1;
  if (base.THW == 1) {
    // 256 -> 256 at 14x14, batch 64, 1.6 GFLOP: level; 344 -> 347 at 43x38, batch 23, 9 GFLOP: 94 -> 83 us.  Shorter reductions
    // want more tiles: 307 -> 314 at 98x98, 5.6 GFLOP: 60 -> 65; the filter gradient of a 128 x 9216 -> 4096 inner product,
    // whose reduction are the 128 rows, 9.7 GFLOP: 106 -> 79.  64 rows: 54 and 57, 4.8 GFLOP
    column_grid(cg_in, base.sh, base.sw, grid);
    if (base.Mrows > 64 && flops >= (base.Kred < 320 ? 6e9 : 2.5e9)) plan = plan_split(base, grid, out_elems);
  } else if (cg_in * 100 >= round_up(cg_in, 16) * 70) {
    plain_grid(cg_in, kh, kw, base.sh, base.sw, base.dh, base.dw, grid);
    if (base.THW >= 3 && base.Kred >= 256) plan = plan_split(base, grid, out_elems);
  } else if (pbase.mode == 0 &&  // forward: a backward-data gather has the layer's output channels and stride 1
             folded_grid(cg_in, kh, kw, base.sh, base.sw, base.dh, base.dw, base.pw, grid)) {
    plan = plan_split(base, grid, out_elems);
  }
  if (plan.tile < 0) return 0;
  // Against the fp32 kernels, modelled as 85 TFLOP/s of rows padded to 16 and 12 us of launches: keeps what the split form is
  // too coarse for (16 channels to gather, 11x11, are one chunk that no slice can share: 42 us fp32, 53 split).  Reductions
  // under 800 that the fp32 kernel need not slice are closer: it has no reduce launch there, and what the modelled steps
  // leave out of a split workgroup (prologue, epilogue, patch of a kernel of 1 to 3 taps) weighs more.  Of 329 passes drawn
  // over 1 to 30 GFLOP, 305 take the split form, at worst 3 % slower, 48 % faster in the mean; without the second line of
  // constants 15 were up to 16 % slower (1x1, 141 -> 279 at 103x119: 57 and 67 us; 3x3, 80 -> 229 at 78x84: 31 and 36).  Of
  // 2640 that take it in a wider draw (0.4 to 20 GFLOP, images from 1x1 on) 24 are more than 3 % slower, at worst 21 %, with
  // the lines on weights below, 53 % faster in the mean.
  // Small strided backward passes stay: their scattered stores cost the gain (17 channels at 43x43, stride 2: 29 and 38).
  const double flops16 = 2.0 * (double)round_up(base.Mrows, 16) * base.Kred * (double)base.ncols * base.G;
  double here = plan.cost + 10, fp32 = flops16 / 85e6 + 12;
  if (base.ksplit == 1 && base.Kred < 800) {
    const int64_t per_cu = ceil_div(plan.units * plan.S, 256);
    here += (base.THW <= 3 ? 2.5 : 1.5) * (double)per_cu + (plan.S > 1 ? 4 : 0) + (base.simple_epilogue ? 0 : 6);
    fp32 = flops16 / 90e6 + 8;
  }
  // The model leaves out what packing six bytes a weight costs.  With many taps and few columns that decides (forward, one
  // image of 14x14, 3x3, 1024 -> 1024, 38 MB of weights: 67 us fp32, 97 split; 2048 -> 1024 on 200 columns: 119 and 182; on 784:
  // 329 and 293; data gradient, 2048 -> 1024 on 98 columns: 97 and 139); 1x1 weights are packed as they lie.
  const double weight_mb = 4e-6 * (double)base.G * base.Mrows * base.Kred;
  if (base.THW > 1 && pbase.mode == 0 && weight_mb > 6) here += 1.5 * (weight_mb - 6);
  if (base.THW > 1 && pbase.mode != 0 && weight_mb > 16) here += weight_mb - 16;
  if (here > fp32 || (!base.simple_epilogue && flops < 3e9)) return 0;
  tile = plan.tile;
  int32_t bm, bn, mt;
  split_tile_shape(tile, &bm, &bn, &mt);
  const bool columns = grid.f.subs != 0;
  const int64_t chunks = ceil_div(grid.f.V, columns ? 64 : 16);
  a = CorrSplitArgs();
  k = PackSplitArgs();
  static_cast<CorrArgs&>(a) = base;
  static_cast<PackArgs&>(k) = pbase;
  a.use_patch = 0;
  a.fold = k.fold = grid.f;
  a.sh = (int32_t)grid.sh;
  a.sw = (int32_t)grid.sw;
  a.dh = (int32_t)grid.dh;
  a.dw = (int32_t)grid.dw;
  a.TW = k.tTW = (int32_t)grid.TW;
  a.THW = k.tTHW = (int32_t)(grid.TH * grid.TW);
  a.Cg_in = (int32_t)cg_in;
  a.NS = (int32_t)chunks;
  a.PH = base.P / base.PW;
  a.Nimg = (int32_t)n_img;
  const bool pixels = columns && base.IHW == 1 && base.P == 1 && base.ph == 0 && base.pw == 0;
  a.fold.pixels = pixels;
  a.PWID = pixels ? bn + 1 : columns ? bn : (int32_t)plan.w.pitch;  // columns: from one group of 16 channels to the next
  a.share_w = (int32_t)plan.w.share;
  a.share_h = (int32_t)plan.h.share;
  a.PSZ = pixels ? 4 * a.PWID : (int32_t)plan.psz;
  const int64_t table = grid.f.ff > 1 ? 128 * chunks : 0;  // the folded form's, behind the stages
  a.patch_stages = plan.psz <= 416 && 192 * plan.psz + table <= 80 * 1024 ? 2 : 1;  // two workgroups per compute unit either way
  a.mPWID = make_magic((uint32_t)a.PWID);
  a.mRSEG = make_magic((uint32_t)(columns ? 1 : plan.h.pitch));
  a.m_tiles = (int32_t)ceil_div(a.Mrows, bm);
  a.MP = a.m_tiles * bm;
  a.col_tiles = (int32_t)ceil_div(a.ncols, bn);
  a.out_elems = (int32_t)out_elems;
  a.chunks_per_split = (int32_t)ceil_div(chunks, plan.S);
  a.ksplit = (int32_t)ceil_div(chunks, a.chunks_per_split);
  k.split_chunks = a.NS;
  // Six bytes a packed weight and the slices: a workspace beyond the boundary's 2^30 elements stays with the fp32 kernel (four).
  const int64_t fragments = split_fragments(base, grid, tile), bytes = split_pack_bytes(fragments, plan.half);
  if (plan.half) {
    a.half = k.half = 1;
    a.lead_steps = corr_half_interval(base, tile, mt, a.THW, chunks, a.chunks_per_split, plan.bf16_cps, plan.inside);
    const uint32_t stage = pixels ? split_half_stage(4, bn) : split_half_stage(columns ? 4 : split_patch_units(a.PSZ + 1, bn), 0);
    const uint32_t behind = split_half_lead(bm, bn) + (columns && !pixels ? kUnheldBytes : 0);
    a.patch_stages = 2 * stage + behind <= 80 * 1024 ? 2 : 1;  // two workgroups per compute unit
    const int64_t per_sample = ceil_div(n_img, kSamples);
    a.mSample = make_magic((uint32_t)per_sample);
    k.in_elems = a.in_bytes / 4;
    k.sample_elems = (uint32_t)(per_sample * a.in_img_stride);
    k.fragments = (uint32_t)fragments;
    k.w_elems = (uint32_t)(pbase.G * pbase.Kg * pbase.Cg * pbase.kh * pbase.kw);
  }
  if (bytes + (a.ksplit > 1 ? 4 * a.ksplit * out_elems : 0) >= 4 * kMaxElems) {
    tile = -1;
    return 0;
  }
  return (size_t)bytes;
}

// The layer's own part of the arguments.
void wgrad_split_args(const WgradArgs& w, int64_t N, WgradSplitArgs& a) {
  a = WgradSplitArgs();
  a.dy_bytes = w.dy_bytes;
  a.x_bytes = w.x_bytes;
  a.N = (int32_t)N;
  a.P = w.P;
  a.PW = w.PW;
  a.PH = w.P / w.PW;
  a.mPW = w.mPW;
  a.runs = (int32_t)ceil_div(w.P, 8);
  a.mRuns = make_magic((uint32_t)a.runs);
  a.Kg = w.Kg;
  a.Ktot = w.Ktot;
  a.Cg = w.Cg;
  a.C = w.C;
  a.H = w.H;
  a.W = w.W;
  a.kw = w.kw;
  a.khw = w.khw;
  a.sh = w.sh;
  a.sw = w.sw;
  a.dh = w.dh;
  a.dw = w.dw;
  a.ph = w.ph;
  a.pw = w.pw;
  a.Kred = w.Kred;
}

// Modelled time (us) of the fp32 filter gradient, see configure_wgrad_split.
double wgrad_fp32_time(const WgradArgs& w, int32_t fp32_tile, double w_mb) {
  int32_t bm, bn, bk;
  wgrad_tile_shape(fp32_tile, &bm, &bn, &bk);
  static const double kFp32Step[WGRAD_TILE_COUNT] = {1.74, 1.45, 1.04, 0.634, 0.978};
  const double bounds = (double)(bm * bn) / 16384.0 * (w.bounds_mode == 1 ? 0.51 : w.bounds_mode == 2 ? 0.29 : 0.0);
  const int64_t per_cu = ceil_div((int64_t)w.G * w.m_tiles * w.n_tiles * w.S, 256);
  return 13.2 + 0.375 * (double)w.S * w_mb + (double)(per_cu * ceil_div(w.cols_per_split, 32)) * (kFp32Step[fp32_tile] + bounds);
}

// Decides whether wgrad_split_kernel runs the backward filter instead of the fp32 kernel on its tile and split; fills a and
// returns its own tile, -1 if it does not.
int32_t configure_wgrad_split(const WgradArgs& w, int32_t fp32_tile, int64_t N, int64_t K, int64_t w_elems, WgradSplitArgs& a) {
  const double flops = 2.0 * w.Kg * w.Kred * (double)w.ncols * w.G;
  if (w.ncols < 1 || flops < 4e8 || w.x_bytes > (1u << 30) || w.dy_bytes > (1u << 31) - 32) return -1;
  if (4 * (int64_t)w.Kg * w.Kred > ((int64_t)1 << 30)) return -1;
  const int64_t TH = w.khw / w.kw, PH = w.P / w.PW;
  const int64_t ext = (TH - 1) * w.dh + 1;
  const PatchDim dim_w = patch_dim(w.PW, w.sw, (int64_t)(w.kw - 1) * w.dw + 1, w.pw, w.W);
  const PatchDim dim_h = patch_dim(PH, w.sh, ext, w.ph, w.H);
  const int64_t PWID = dim_w.pitch, RS = dim_h.pitch;
  const int64_t runs = ceil_div(w.P, 8), total_runs = N * runs, chunk_runs = wgrad_split_chunk_runs();
  const int64_t max_rows = max_patch_rows(total_runs, runs, chunk_runs, 8, w.P, w.PW, w.sh, ext, RS, 512 / PWID);
  const int64_t psz = max_rows * PWID + dim_w.share;
  if (psz > 512) return -1;
  const int64_t c16 = ceil_div(w.Cg, 16);
  // Splits: the whole grid resident at once (two workgroups per compute unit) or half of that, partials at most 32 MiB.
  // Tile and splits by modelled time (us), as in configure_split: a chunk is four steps; a fit to 580 timings of
  // all tiles and 1 to 12 quarters of a resident grid on the same layers (rms error 5 %; the choice is 1 % behind the
  // best on average, 12 % at worst).
  // The second line, for the f16 terms, is a fit to 589 timings of 20 layers of 1 to 57 GFLOP (6 %; 1 % and 7 %); their samples
  // cost 3 us.  They take sums of one slice long enough for them.
  struct Costs {
    double alone[WSPLIT_TILE_COUNT], shared[WSPLIT_TILE_COUNT], patch_alone, patch_shared, slice_mb, workgroup, fixed;
  };
  static const Costs kCosts[2] = {{{1.40, 1.19, 1.18, 1.06, 0.64, 1.04}, {1.09, 0.985, 0.97, 0.90, 0.52, 0.89}, 0.37, 0.16, 0.66, 0.73, 0},
                                  {{0.973, 0.854, 0.866, 0.785, 0.525, 0.819}, {0.708, 0.650, 0.622, 0.566, 0.380, 0.633}, 0.339, 0.187, 0.556, 2.07, 3.2}};
  const int64_t chunks = ceil_div(total_runs, chunk_runs), max_by_ws = ((int64_t)8 << 20) / w_elems;
  const double units_per_thread = (double)split_patch_units(psz), w_mb = 4e-6 * (double)w_elems;
  int32_t best = -1, best_lead = 0;
  int64_t best_cps = 0;
  double best_cost = 0, least_work = 0;
  const double chunk_pix = (double)w.ncols / (double)chunks;
  // The samples are of four neighbours.  Blocks and runs that hold less than 45 % of real work stay with what the bf16 terms are
  // compared with (20 -> 320, 5x5 at 2x3, 42 %: 137 us fp32, 142 bf16 terms, 118 f16 terms).
  const auto half_fits = [&](double work) {
    return w.x_bytes >= 16 && w.dy_bytes >= 16 && work * 8.0 * (double)total_runs <= 2.2 * (double)w.Kg * w.Kred * (double)w.ncols;
  };
  int64_t bf16_cps = 0;  // of the best plan on bf16 terms
  const double inside = inside_image(w.PW, w.sw, w.kw, w.dw, w.pw, w.W) * inside_image(PH, w.sh, w.khw / w.kw, w.dh, w.ph, w.H);
  for (int half = 0; half < 2; ++half) {
    const Costs& c = kCosts[half];
    // Half zeros in both blobs count from sums on that two chunks a stretch are enough for: a move every chunk costs what the
    // instructions save (45 -> 77, 3x5 at 51x67, batch 37, 758 a slice: 57 -> 70 us, 67 on bf16 terms).
    const double bf16_pix = chunk_pix * (double)bf16_cps, aim = (bf16_pix < 1500 ? kHalfMost : 0.9 * kBf16BothHalf) * bf16_pix;
    for (int32_t t = 0; t < WSPLIT_TILE_COUNT; ++t) {
      int32_t rows, taps;
      wgrad_split_shape(t, &rows, &taps);
      const double work = (double)round_up(w.Kg, rows) * (double)round_up(w.khw, taps) * (double)(16 * c16);
      if (least_work == 0 || work < least_work) least_work = work;
      if (half && !half_fits(work)) continue;
      const int64_t tiles = (int64_t)w.G * ceil_div(w.Kg, rows) * ceil_div(w.khw, taps) * c16;
      for (int64_t places = 256; places <= 512; places += 256) {
        int64_t S = places / tiles;
        if (S > max_by_ws) S = max_by_ws;
        if (S > 256) S = 256;
        if (S > chunks) S = chunks;
        if (S < 1) S = 1;
        const int64_t cps = ceil_div(chunks, S), per_cu = ceil_div(tiles * ceil_div(chunks, cps), 256);
        const int32_t lead = half ? half_interval(chunk_pix * (double)cps, std::min(kHalfMost, kBf16Full * inside) * bf16_pix, aim, chunk_pix, 1) : 0;
        if (half && !lead) continue;
        const double cost = c.fixed + c.slice_mb * (double)S * w_mb + c.workgroup * (double)per_cu +
                            (per_cu == 1 ? (double)cps * (4 * c.alone[t] + c.patch_alone * units_per_thread)
                                         : (double)(per_cu * cps) * (4 * c.shared[t] + c.patch_shared * units_per_thread));
        if (best < 0 || cost < best_cost) {
          best = t;
          best_cost = cost;
          best_cps = cps;
          best_lead = lead;
        }
      }
    }
    bf16_cps = best_cps;
  }
  // Fewer chunks than that cannot be shared out (4 chunks, 0.5 GFLOP: 18.8 us fp32, 21.2 split; 5, 2.4 GFLOP: 58.6, 62.9).
  if (chunks < 8) return -1;
  // What the blocks pad more than the fp32 tile costs the advantage: up to twice its work on a large problem (202 -> 14
  // channels, 5x3: 1.6 times the work, 186 -> 156 us), 1.45 times under 4.5 GFLOP (54 -> 74, 3x3 at 75x60, 1.5 times: 57 ->
  // 61 us) and 1.12 times under 2.5 GFLOP (64 -> 96 channels, 3x1 at 28x28, twice the work: 38 -> 42 us; 300 -> 200, 3x3
  // at 12x12, 1.11 times: 38 -> 33 us).
  int32_t bm, bn, bk;
  wgrad_tile_shape(pick_wgrad_tile(w.Kg, w.Kred), &bm, &bn, &bk);
  if (least_work > (flops < 2.5e9 ? 1.12 : flops < 4.5e9 ? 1.45 : 2.0) * (double)round_up(w.Kg, bm) * (double)round_up(w.Kred, bn)) return -1;
  // The rest by modelled times (us).  The fp32 kernel's: workgroups of a compute unit times the 32-column steps of one, by
  // tile and by what the bounds test costs it, and its slices; a fit to 825 filter gradients of 0.4 to 20 GFLOP (rms error
  // 5 %; 7 % on 1288, the split kernel's 8 %).  A run holds pixels of one image, so best_cost counts the zeros that fill an
  // image's last run.  Of those 1288 the lines above let through, 139 were more than 3 % slower than fp32 (one pixel, 512 -> 512,
  // 3x3, batch 2048: 134 us fp32, 390 split; 48 x 249 -> 266, 2x2 taps on tiles of eight: 62 and 78), with this line 16, at
  // worst 11 %; 26 that gained more than 3 % stay behind with them, at best 434 -> 293 us.
  if (8.4 + 0.99 * best_cost > wgrad_fp32_time(w, fp32_tile, w_mb)) return -1;
  int32_t rows, taps;
  wgrad_split_shape(best, &rows, &taps);
  wgrad_split_args(w, N, a);
  a.part_stride = (int32_t)w_elems;
  a.G = w.G;
  a.m_tiles = (int32_t)ceil_div(w.Kg, rows);
  a.tap_tiles = (int32_t)ceil_div(w.khw, taps);
  a.n_tiles = (int32_t)(c16 * a.tap_tiles);
  a.PWID = (int32_t)PWID;
  a.PSZ = (int32_t)psz;
  a.ext = (int32_t)ext;
  a.share_h = (int32_t)dim_h.share;
  a.patch_stages = psz <= 416 ? 2 : 1;  // two workgroups per compute unit either way
  a.mPWID = make_magic((uint32_t)PWID);
  a.mRSEG = make_magic((uint32_t)RS);
  a.chunks = (int32_t)chunks;
  a.chunks_per_split = (int32_t)best_cps;
  a.S = (int32_t)ceil_div(chunks, best_cps);
  if (best_lead) {
    a.half = 1;
    a.lead_chunks = best_lead;
    const uint32_t rest = 2 * 4 * 8 * (uint32_t)chunk_runs + split_half_lead(rows, 16 * taps) + kUnheldWgradBytes;
    a.patch_stages = 128 * (uint32_t)a.PSZ + rest <= 80 * 1024 ? 2 : 1;  // two workgroups per compute unit
  }
  const int64_t tiles = (int64_t)a.G * a.m_tiles * a.n_tiles;
  if (a.S * (w_elems + a.n_tiles * K) >= kMaxElems || tiles * a.S >= ((int64_t)1 << 31)) return -1;
  return best;
}

// The same on the folded grid of a layer with few channels, f16 terms only: its tile, or -1.
int32_t configure_wgrad_fold(const WgradArgs& w, int32_t fp32_tile, int64_t N, int64_t K, int64_t w_elems, WgradSplitArgs& a) {
  const double flops = 2.0 * w.Kg * w.Kred * (double)w.ncols * w.G;
  if (w.ncols < 1 || flops < 1e9 || w.x_bytes > (1u << 30) || w.dy_bytes > (1u << 31) - 32 || w.x_bytes < 16 || w.dy_bytes < 16) return -1;
  SplitGrid grid;
  if ((int64_t)w.Cg * 100 >= round_up(w.Cg, 16) * 70 ||
      !folded_grid(w.Cg, w.khw / w.kw, w.kw, w.sh, w.sw, w.dh, w.dw, w.pw, grid))
    return -1;
  const int64_t T = grid.TH * grid.TW, V = grid.f.V, part = K * T * V;
  if (part > ((int64_t)8 << 20)) return -1;  // one slice is within the fixed scratch array
  const int64_t ext = (grid.TH - 1) * grid.dh + 1;
  const PatchDim dim_w = patch_dim(w.PW, grid.sw, (grid.TW - 1) * grid.dw + 1, 0, w.W);
  const PatchDim dim_h = patch_dim(w.P / w.PW, grid.sh, ext, 0, w.H);
  const int64_t runs = ceil_div(w.P, 8), total_runs = N * runs, chunk_runs = wgrad_split_chunk_runs();
  const int64_t max_rows = max_patch_rows(total_runs, runs, chunk_runs, 8, w.P, w.PW, grid.sh, ext, dim_h.pitch, 512 / dim_w.pitch);
  const int64_t psz = max_rows * dim_w.pitch + dim_w.share;
  if (psz > 512) return -1;
  const int64_t c16 = ceil_div(V, 16), chunks = ceil_div(total_runs, chunk_runs);
  if (chunks < 8) return -1;
  // A fit to 135 timings of 16 layers (rms error 5 %).  A patch unit is dearer than the image's: its table entries, and two loads with
  // a test of every element's column.
  static const double kAlone[WFOLD_TILE_COUNT] = {0.834, 0.849, 0.747, 0.325}, kShared[WFOLD_TILE_COUNT] = {0.459, 0.466, 0.396, 0.088};
  const double units_per_thread = psz <= 384 ? 3 : 4, chunk_pix = (double)w.ncols / (double)chunks, part_mb = 4e-6 * (double)part;
  int32_t best = -1, best_lead = 0;
  int64_t best_cps = 0;
  double best_cost = 0;
  for (int32_t t = 0; t < WFOLD_TILE_COUNT; ++t) {
    int32_t rows, taps;
    wgrad_fold_shape(t, &rows, &taps);
    const int64_t tiles = (int64_t)w.G * ceil_div(w.Kg, rows) * ceil_div(T, taps) * c16;
    for (int64_t places = 256; places <= 512; places += 256) {
      int64_t S = places / tiles;
      if (S > ((int64_t)8 << 20) / part) S = ((int64_t)8 << 20) / part;
      if (S > 256) S = 256;
      if (S > chunks) S = chunks;
      if (S < 1) S = 1;
      const int64_t cps = ceil_div(chunks, S), per_cu = ceil_div(tiles * ceil_div(chunks, cps), 256);
      const double pix = chunk_pix * (double)cps;
      // what runs otherwise are the fp32 kernels, further off than the bf16 terms without zeros
      const int32_t lead = half_interval(pix, kHalfMost * pix, 0.9 * kBf16Half * pix, chunk_pix, 1);
      if (!lead) continue;
      const double cost = 6.9 + 0.604 * (double)S * part_mb + 3.43 * (double)per_cu +
                          (per_cu == 1 ? (double)cps * (4 * kAlone[t] + 0.669 * units_per_thread)
                                       : (double)(per_cu * cps) * (4 * kShared[t] + 0.580 * units_per_thread));
      if (best < 0 || cost < best_cost) {
        best = t;
        best_cost = cost;
        best_cps = cps;
        best_lead = lead;
      }
    }
  }
  if (best < 0 || 1.08 * best_cost > wgrad_fp32_time(w, fp32_tile, 4e-6 * (double)w_elems)) return -1;
  int32_t rows, taps;
  wgrad_fold_shape(best, &rows, &taps);
  wgrad_split_args(w, N, a);
  a.fold = grid.f;
  a.kw = (int32_t)grid.TW;
  a.khw = (int32_t)T;
  a.sh = (int32_t)grid.sh;
  a.sw = (int32_t)grid.sw;
  a.dh = (int32_t)grid.dh;
  a.dw = (int32_t)grid.dw;
  a.Kred = (int32_t)(T * V);
  a.part_stride = (int32_t)part;
  a.G = w.G;
  a.m_tiles = (int32_t)ceil_div(w.Kg, rows);
  a.tap_tiles = (int32_t)ceil_div(T, taps);
  a.n_tiles = (int32_t)(c16 * a.tap_tiles);
  a.PWID = (int32_t)dim_w.pitch;
  a.PSZ = (int32_t)psz;
  a.ext = (int32_t)ext;
  a.share_h = 0;
  a.mPWID = make_magic((uint32_t)dim_w.pitch);
  a.mRSEG = make_magic((uint32_t)dim_h.pitch);
  a.chunks = (int32_t)chunks;
  a.chunks_per_split = (int32_t)best_cps;
  a.S = (int32_t)ceil_div(chunks, best_cps);
  a.half = 1;
  a.lead_chunks = best_lead;
  const uint32_t rest = 2 * 4 * 8 * (uint32_t)chunk_runs + split_half_lead(rows, 16 * taps) + kUnheldWgradBytes + 128 * (uint32_t)c16;
  a.patch_stages = 128 * (uint32_t)a.PSZ + rest <= 80 * 1024 ? 2 : 1;  // two workgroups per compute unit
  return best;
}

// The launch that clears dx where no tap reaches some of it, whatever kernel runs the rest (us; dx in MB): a fit to 1300 such passes.
double zero_fill_model(bool zero_fill, double out_mb) { return zero_fill ? 2.7 + 0.15 * out_mb : 0.0; }

// Modelled time (us) of a forward or backward-data pass on the tiled fp32 kernels: the launches, packed weights (MB), partial
// sums and output (MB), then per tile the chunks of 16 reduction indices that one workgroup walks alone and those that the
// workgroups of a compute unit share, dearer where the gather compares or masks.  A fit to 8653 timings -- every tile, 1 to 16
// slices, 240 passes of 0.15 to 20 GFLOP (rms error 14 to 16 %, most of it in configurations far from the best).
struct CorrModel {
  CorrModel(const CorrArgs& a, int32_t tile, int64_t out_elems, bool zero_fill) {
    static const double kCost[CORR_TILE_COUNT][4] = {  // alone, shared, with compares, with masks
        {0.243, 0.802, 0.151, 0.075}, {0.208, 0.386, 0.081, 0.045}, {0.263, 0.564, 0.191, 0.099}, {0.296, 0.327, 0.152, 0.078},
        {0.250, 0.168, 0.074, 0.035}, {0.317, 0.379, 0.233, 0.104}, {0.281, 0.184, 0.107, 0.043}, {0.253, 0.615, 0.280, 0.136},
        {0.238, 0.263, 0.137, 0.065}, {0.250, 0.307, 0.134, 0.028}, {0.208, 0.080, 0.021, 0.003}};
    int32_t bm, bn, bk;
    corr_tile_shape(tile, &bm, &bn, &bk);
    const double* const c = kCost[tile];
    all = (uint32_t)ceil_div(a.Kred, 16);
    const int64_t m_tiles = parts_of(a.Mrows, (uint32_t)bm);
    units = (int64_t)a.G * m_tiles * parts_of(a.ncols, (uint32_t)bn);
    out_mb = 4e-6 * (double)out_elems;
    const double pack_mb = 4e-6 * (double)a.G * (double)(m_tiles * bm) * (double)(16 * (int64_t)all);
    launches = 5.5 + 0.3 * pack_mb + 0.25 * out_mb + zero_fill_model(zero_fill, out_mb);
    alone = c[0];
    shared = c[1] + (a.bounds_mode == 1 ? c[2] : a.bounds_mode == 2 ? c[3] : 0.0);
    workgroup = tile == CORR_16x64 ? 0.09 : 0.0;
  }
  double time(int64_t S) const {  // in S slices
    const uint32_t chunks = parts_of(all, (uint32_t)S), slices = parts_of(all, chunks);
    const double per_cu = (double)((units * slices + 255) >> 8);
    return launches + (slices > 1 ? 2.2 + 0.7 * (double)slices * out_mb : 0.0) + (double)chunks * (alone + per_cu * shared) + per_cu * workgroup;
  }
  uint32_t all;
  int64_t units;
  double out_mb, launches, alone, shared, workgroup;
};

// Tile and slices of a pass on the tiled fp32 kernels by that model, for passes of 0.2 GFLOP and more: the row count that pads
// least says little about the time.  73 -> 2 channels 8x8, stride 2, at 26x32, batch 73, backward data: 16x64 unsplit 128 us, in
// 12 slices 61; 236 -> 300 in four groups, 3x5, stride 2: 16x64 162, 32x128 94.  Of 152 passes of the fit that these kernels
// took, none was on the tiles of at most 48 rows by 256 columns that the patch-staged kernel takes (left alone); the
// choice is 11 % faster than the rules' in the geometric mean, up to twice, and 2 % behind the best.  Smaller passes keep the
// rules (pick_corr_tile, configure_ksplit): where the tiles run them at all, the times of the choice differ by 3 % (4 from 0.05 GFLOP on).
void plan_corr(CorrArgs& a, PackArgs& k, int64_t out_elems, bool zero_fill, int32_t& tile) {
  const double flops = 2.0 * a.Mrows * a.Kred * (double)a.ncols * a.G;
  if (a.use_patch || a.ncols < 1 || flops < 2e8) return;
  static const int32_t kSlices[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16};
  const int64_t all = ceil_div(a.Kred, 16);
  int32_t best = tile;
  int64_t best_S = a.ksplit;
  double cost = 0.92 * CorrModel(a, tile, out_elems, zero_fill).time(a.ksplit);  // nearer than that is within the model's error
  for (int32_t t = 0; t < CORR_TILE_COUNT; ++t) {
    int32_t bm, bn, bk;
    corr_tile_shape(t, &bm, &bn, &bk);
    if ((int64_t)a.G * a.KP * round_up(a.Mrows, bm) >= kMaxElems) continue;
    const CorrModel model(a, t, out_elems, zero_fill);
    for (const int64_t S : kSlices) {
      if (S > 1 && (2 * S > all || S * out_elems > ((int64_t)16 << 20))) break;  // slices of two chunks, 64 MiB of partial sums
      const double c = model.time(S);
      if (c < cost) {
        best = t;
        best_S = S;
        cost = c;
      }
    }
  }
  if (best == tile && best_S == a.ksplit) return;
  int32_t bm, bn, bk;
  corr_tile_shape(best, &bm, &bn, &bk);
  tile = best;
  a.MP = k.MP = (int32_t)round_up(a.Mrows, bm);
  a.m_tiles = a.MP / bm;
  a.col_tiles = (int32_t)ceil_div(a.ncols, bn);
  a.chunks_per_split = (int32_t)ceil_div(all, best_S);
  a.ksplit = (int32_t)ceil_div(all, a.chunks_per_split);
}

// The time of a pass on the tiled fp32 kernels, as planned, against which the one-launch kernel is held.  Below 0.7 GFLOP CorrModel is 8
// to 17 % short of it; a fit of its own to 51740 timings -- every tile, 1 to 16 slices -- is 5 to 10 % off (rms) on 19000 others.  20 -> 50
// channels, 5x5 at 12x12, batch 64, backward data: 23.7 us on the tiles, 24.8 here, 21.7 by CorrModel; 19.5 in one launch.
double tiled_time(const CorrArgs& a, int32_t tile, int64_t out_elems, bool backward, bool zero_fill) {
  static const double kCost[CORR_TILE_COUNT][5] = {  // alone, shared, with compares, with masks, workgroup
      {0.397, 0.599, 0.186, 0.145, 2.023}, {0.294, 0.263, 0.108, 0.111, 1.164}, {0.448, 0.334, 0.234, 0.167, 2.082},
      {0.338, 0.261, 0.155, 0.114, 1.092}, {0.286, 0.105, 0.104, 0.093, 0.532}, {0.426, 0.151, 0.357, 0.219, 1.605},
      {0.319, 0.078, 0.186, 0.135, 0.617}, {0.311, 0.458, 0.355, 0.229, 2.052}, {0.262, 0.142, 0.217, 0.154, 0.946},
      {0.267, 0.142, 0.286, 0.165, 1.037}, {0.236, 0.012, 0.067, 0.056, 0.255}};
  if (2.0 * a.Mrows * a.Kred * (double)a.ncols * a.G >= 0.7e9) return CorrModel(a, tile, out_elems, zero_fill).time(a.ksplit);
  const double* const c = kCost[tile];
  const double per_cu = (double)ceil_div((int64_t)a.G * a.m_tiles * a.col_tiles * a.ksplit, 256);
  const double out_mb = 4e-6 * (double)out_elems, pack_mb = 4e-6 * (double)a.G * (double)a.MP * (double)a.KP;
  const double shared = c[1] + (a.bounds_mode == 1 ? c[2] : a.bounds_mode == 2 ? c[3] : 0.0);
  const double rest = 6.07 + 0.787 * pack_mb + 0.096 * out_mb + (a.ksplit > 1 ? 2.33 + 0.608 * a.ksplit * out_mb : 0.0) +
                      (double)a.chunks_per_split * (c[0] + per_cu * shared) + per_cu * c[4];
  return (backward ? 1.05 : 0.98) * rest + zero_fill_model(zero_fill, out_mb);
}

// The time of a pass on the tiled kernels of doubles, as planned, on tiles of `rows`: launches, packed weights, partial sums and output
// (MB), then per tile the chunks that one workgroup walks alone, those that the workgroups of a compute unit share, and these
// workgroups; a forward pass 3 % less, backward data 4 % more.  A fit to 12665 timings of up to 6 GFLOP -- every tile, 1 to 16 slices; 6
// to 8 % off (rms) from the smallest to the largest, on 16796 others as well.
double corr64_model(const CorrArgs& a, int32_t rows, int64_t out_elems, bool backward, bool zero_fill) {
  static const struct {
    int32_t rows;
    double alone, shared, workgroup;
  } kCost[] = {{16, 0.266, 0.138, 0.494}, {32, 0.318, 0.222, 0.666}, {48, 0.360, 0.326, 0.866}, {64, 0.405, 0.444, 1.062}, {96, 0.497, 0.679, 1.683}};
  int t = 0;
  while (kCost[t].rows != rows) ++t;
  const double per_cu = (double)ceil_div((int64_t)a.G * a.m_tiles * a.col_tiles * a.ksplit, 256);
  const double out_mb = 8e-6 * (double)out_elems, pack_mb = 8e-6 * (double)a.G * (double)a.MP * (double)a.KP;
  const double rest = 5.97 + 0.544 * pack_mb + 0.073 * out_mb + (a.ksplit > 1 ? 2.27 + 0.363 * a.ksplit * out_mb : 0.0) +
                      (double)a.chunks_per_split * (kCost[t].alone + kCost[t].shared * per_cu) + kCost[t].workgroup * per_cu;
  return (backward ? 1.04 : 0.97) * rest + zero_fill_model(zero_fill, out_mb);
}

// Tile and slices of the fp64 kernel where another choice is modelled at least 8 % ahead, from 0.05 to 6 GFLOP.  The model is a fit
// to 130 layers of those sizes on every tile and slice count (260 passes, rms error 8 %).  Of the 260, 55 change, 1.26 times as
// fast in the geometric mean, two 6 % slower; one of 0.18 GFLOP took 268 us unsplit on the 16-row tile and 86 in sixteen
// slices, one of 4.5 GFLOP 335 on it and 124 on 48 rows.
void plan_corr64(CorrArgs& a, int64_t out_elems, int32_t& rows) {
  const double flops = 2.0 * a.Mrows * a.Kred * (double)a.ncols * a.G;
  if (a.ncols < 1 || flops < 5e7 || flops > 6e9) return;
  static const int32_t kSlices[] = {1, 2, 3, 4, 6, 8, 12, 16};
  static const struct {
    int32_t rows;
    double chain, chunk, workgroup;
  } kTiles[] = {{16, 0.270, 0.146, 0.44}, {32, 0.285, 0.239, 0.54}, {48, 0.325, 0.349, 0.70}, {64, 0.363, 0.471, 0.88}, {96, 0.446, 0.724, 1.47}};
  const int64_t all = ceil_div(a.Kred, kF64TileK);
  const double out_mb = 8e-6 * (double)out_elems;
  int32_t best = rows;
  int64_t best_S = a.ksplit;
  double cost = 0, here = 0;
  for (const auto& t : kTiles) {
    const int64_t m_tiles = parts_of(a.Mrows, (uint32_t)t.rows), units = (int64_t)a.G * m_tiles * a.col_tiles;
    const double launches = 5.0 + 0.21 * out_mb + 0.27 * 8e-6 * (double)(a.G * m_tiles * t.rows) * (double)a.KP;
    auto model = [&](int64_t S) {
      const uint32_t chunks = parts_of(all, (uint32_t)S), slices = parts_of(all, chunks);
      const double per_cu = (double)((units * slices + 255) >> 8);
      return launches + (S > 1 ? 4.0 + 0.288 * (double)S * out_mb : 0.0) + (double)chunks * (t.chain + t.chunk * per_cu) + t.workgroup * per_cu;
    };
    if (t.rows == rows) here = 0.92 * model(a.ksplit);  // nearer than that is within the model's error
    for (const int64_t S : kSlices) {
      if (S > 1 && (2 * S > all || S * out_elems > ((int64_t)8 << 20))) break;  // slices of two chunks, 64 MiB of partial sums
      const double c = model(S);
      if (cost == 0 || c < cost) {
        best = t.rows;
        best_S = S;
        cost = c;
      }
    }
  }
  if (cost >= here) return;
  rows = best;
  a.MP = (int32_t)round_up(a.Mrows, best);
  a.m_tiles = a.MP / best;
  a.chunks_per_split = (int32_t)ceil_div(all, best_S);
  a.ksplit = (int32_t)ceil_div(all, a.chunks_per_split);
}

// Modelled times (us) of the one-launch kernels: a launch; then per tile the wave's chain of reduction groups (blocks of 64
// places in the filter gradient), the groups that a compute unit's workgroups share, and those workgroups.
struct SmallCost {
  double chain, shared, workgroup;
};

// Decides whether corr_small_kernel runs this correlation instead of the launches of `base`, which are modelled to take `old`
// us; fills a and returns its tile, -1 if it does not.
int32_t configure_corr_small(const CorrArgs& base, const PackArgs& k, int64_t w_elems, int64_t out_elems, bool zero_fill,
                             int32_t elem_bytes, double old, CorrSmallArgs& a) {
  const int64_t limit = (int64_t)1 << 30, TH = base.THW / base.TW;
  // Not measured: forward passes of layers with a stride and a dilation, and what the patch-staged kernel takes.
  if (base.use_patch || (base.sh * base.sw > 1 && base.dh * base.dw > 1)) return -1;
  const double flops = 2.0 * base.Mrows * base.Kred * (double)base.ncols * base.G;
  if (flops > (elem_bytes == 8 ? 1e9 : 1.5e9)) return -1;
  if (base.ncols < 1 || (int64_t)base.in_bytes > limit || elem_bytes * w_elems > limit || elem_bytes * out_elems > limit) return -1;
  // the kernel's packed displacements, and the row that stands for "past the reduction"
  if (base.IH > 16384 || base.IW > 16384 || base.ph > 4096 || base.pw > 4096) return -1;
  if ((TH - 1) * base.dh > 8192 || (int64_t)(base.TW - 1) * base.dw > 8192 || k.kh > 8192 || k.kw > 8192) return -1;
  a = CorrSmallArgs();
  static_cast<CorrArgs&>(a) = base;
  a.w_bytes = (uint32_t)(elem_bytes * w_elems);
  a.use_patch = 0;
  a.ksplit = 1;
  a.tap_pitch = a.THW;
  a.Qh = (int32_t)TH;
  a.kh = k.kh;
  a.kw = k.kw;
  const int32_t T = k.kh * k.kw;
  a.pad = base.ph > 0 || base.pw > 0 ||
          ((int64_t)base.P / base.PW - 1) * base.sh - base.ph + (TH - 1) * base.dh >= base.IH ||
          ((int64_t)base.PW - 1) * base.sw - base.pw + (int64_t)(base.TW - 1) * base.dw >= base.IW;
  a.w_grp_stride = k.Kg * k.Cg * T;
  if (k.mode == 0) {
    a.wmode = 0;
    a.w_row_stride = k.Cg * T;
    a.w_chan_stride = T;
  } else {
    a.w_row_stride = T;
    a.w_chan_stride = k.Cg * T;
    // tap slot q of a row phase r stands for the tap (stride*q + r) / dilation (see phase_dim): the same tap for every row
    // where the stride divides the dilation, stride*q + r in an undilated layer, and not linear in q otherwise
    const bool same_h = k.dh % k.sh == 0, same_w = k.dw % k.sw == 0;
    if ((!same_h && k.dh != 1) || (!same_w && k.dw != 1)) return -1;
    a.step_h = same_h ? 1 : k.sh;
    a.step_w = same_w ? 1 : k.sw;
    a.wmode = !same_h || !same_w ? 2 : T < 3 ? 1 : 3;
    a.Cg_in = k.Kg;
    if (a.wmode == 3) a.tap_pitch = (int32_t)round_up(T, 4);
  }
  const int64_t KT = round_up((int64_t)a.Kred / a.THW * a.tap_pitch, 16);
  if (KT * (a.wmode == 3 ? 9 : 4 * (2 + a.wmode)) > 56 * 1024) return -1;  // the tables
  a.KT = (int32_t)KT;
  a.mPitch = make_magic((uint32_t)a.tap_pitch);
  // [doubles][weights by single loads][tile]: fits to every tile on 203 (doubles: 123) passes of up to 3 (1) GFLOP, rms errors
  // 10 to 19 %; the choice is 2 % behind the best tile on average, 1.5 times at worst
  static const SmallCost kCost[2][2][CORR_SMALL_COUNT] = {
      {{{0.129, 0.035, 0.32}, {0.110, 0.037, 0.58}, {0.123, 0.048, 0.53}, {0.216, 0.054, 0.67}, {0.228, 0.082, 1.05}, {0.148, 0.060, 0.80}, {0.274, 0.103, 1.22}},
       {{0.151, 0.047, 0.32}, {0.193, 0.050, 0.43}, {0.224, 0.061, 0.54}, {0.224, 0.062, 0.73}, {0.259, 0.094, 1.18}, {0.309, 0.081, 0.72}, {0.390, 0.117, 1.45}}},
      {{{0.072, 0.059, 0.42}, {0.000, 0.066, 0.72}, {0.091, 0.089, 0.68}, {0.139, 0.092, 0.78}, {0.149, 0.153, 1.21}, {0.119, 0.114, 1.01}, {}},
       {{0.151, 0.063, 0.39}, {0.000, 0.079, 0.69}, {0.156, 0.107, 0.59}, {0.214, 0.102, 0.65}, {0.242, 0.175, 0.99}, {0.151, 0.159, 0.88}, {}}}};
  // a forward gather that strides over columns takes more cache lines a load; one that stays in the image no bounds tests
  const double strided = (base.sw == 1 ? 1.0 : base.sw < 4 ? 1.1 : 1.3) * (a.pad ? 1.0 : elem_bytes == 8 ? 0.95 : 0.88);
  const double launches = 3.0 + zero_fill_model(zero_fill, 1e-6 * elem_bytes * (double)out_elems);
  const int64_t groups = KT / 16;
  int32_t best = -1;
  double here = 0;
  for (int32_t t = 0; t < CORR_SMALL_COUNT; ++t) {
    const SmallCost& c = kCost[elem_bytes == 8][a.wmode == 1 || a.wmode == 2][t];
    const SmallTile& s = kCorrSmallTiles[t];
    if (c.shared == 0) continue;  // no instance
    const int64_t units = (int64_t)a.G * parts_of(a.Mrows, 16 * (uint32_t)s.mb) * parts_of(a.ncols, 16 * (uint32_t)s.nb);
    const double per_cu = (double)((units + 255) >> 8);
    const double cost = launches + strided * (c.chain * (double)parts_of(groups, (uint32_t)s.waves) + (c.shared * (double)groups + c.workgroup) * per_cu);
    if (best < 0 || cost < here) {
      best = t;
      here = cost;
    }
  }
  // Nearer to the time of the tile chosen: rows past the last load no weights, and rows of 64 taps, or 16, meet in the caches where they are
  // read by single loads (rms errors 9 to 11 %, floats with such loads 14; without this 10 to 17).
  static const double kNear[2][4][2] = {{{0.86, 0.22}, {0.71, 0.17}, {0.88, 0.27}, {0.93, 0.07}}, {{0.79, 0.28}, {0.90, 0.17}, {0.90, 0.17}, {0.94, 0.15}}};
  const double* const near = kNear[elem_bytes == 8][a.wmode];
  const double fill = (double)a.Mrows / (double)round_up(a.Mrows, 16 * kCorrSmallTiles[best].mb);
  double meet = elem_bytes == 4 && a.wmode == 2 ? (T % 64 == 0 ? 0.19 : T % 16 == 0 ? 0.07 : 0.0) : 0.0;
  // Outputs of up to nine pixels gather from an image for every one or two columns.  Over long reductions that is 0 to 60 % dearer: of 123
  // such forward passes 28 were over 1.1 times the tiles' time, 9 of the 84 still taken so are.
  if (elem_bytes == 4 && a.wmode == 0 && a.P <= 9 && groups >= 80) meet = 0.12;
  here = launches + 0.15 + (here - launches) * (near[0] + near[1] * fill + meet);
  const double margin = elem_bytes == 4 && flops >= 0.7e9 ? 0.9 : 0.95;
  if (here > margin * old) return -1;
  a.m_tiles = (int32_t)ceil_div(a.Mrows, 16 * kCorrSmallTiles[best].mb);
  a.col_tiles = (int32_t)ceil_div(a.ncols, 16 * kCorrSmallTiles[best].nb);
  if ((int64_t)a.G * a.m_tiles * a.col_tiles >= ((int64_t)1 << 31)) return -1;
  return best;
}

// The kernel of a forward or backward-data pass of floats: thin rows, split bf16, one launch, or the tiles.
struct CorrChoice {
  int32_t thin, split, small;
  size_t pack_bytes;  // 0: a blob too large for the boundary
};

CorrChoice choose_corr(CorrArgs& a, PackArgs& k, int32_t& tile, int64_t cg_in, int64_t n_img, bool backward, int64_t out_elems,
                       int64_t w_elems, bool zero_fill, bool one_launch, CorrSplitArgs& sp, PackSplitArgs& sp_pack, CorrSmallArgs& small) {
  CorrChoice c = {0, -1, -1, 0};
  CorrArgs tiled = a;
  PackArgs tiled_pack = k;
  c.thin = configure_thin(a, k, cg_in, n_img, backward);
  const int64_t pack_elems = (int64_t)a.G * a.KP * a.MP;
  if (pack_elems >= kMaxElems || (int64_t)a.G * a.m_tiles * a.col_tiles >= ((int64_t)1 << 31)) return c;
  if (c.thin && !a.use_patch && one_launch) {
    // Without LDS staging a thin-row workgroup walks its reduction in dependent steps of eight indices a wave: 4 -> 384
    // channels, 5x3 at 15x15, batch 4, 118 us, in one launch 15; 2 -> 30, 11x11 at 24x24, 128 and 14; 1 -> 82, 7x7, batch 8,
    // 127 and 32 on 16-row tiles in 16 slices.  And its weights are packed by a launch of their own: of 1600 passes under 5 MFLOP nearly
    // all are ahead in one launch, 1.8 times in the geometric mean.  A fit to 4800 passes (rms error 13 to 16 %).
    const int64_t steps = ceil_div(2 * ceil_div(a.Kred, 16), 4), per_cu = ceil_div((int64_t)a.G * ceil_div(a.ncols, 64), 256);
    int32_t t = tile;
    plan_corr(tiled, tiled_pack, out_elems, zero_fill, t);
    const double thin = 5.7 + 4e-6 * 0.75 * (double)out_elems +
                        (double)steps * (0.383 + (a.bounds_mode == 1 ? 0.619 : 0.0) + 0.0389 * (double)per_cu * a.Mrows);
    const double here = tiled_time(tiled, t, out_elems, backward, zero_fill);
    c.small = configure_corr_small(tiled, tiled_pack, w_elems, out_elems, zero_fill, 4, here < thin ? here : thin, small);
    if (c.small >= 0 || here < 0.9 * thin) {
      c.thin = 0;
      a = tiled;
      k = tiled_pack;
      tile = t;
    }
  }
  c.pack_bytes = (size_t)pack_elems * 4 + (size_t)a.KP * sizeof(KTabEntry);
  if (c.thin || c.small >= 0) return c;
  if (const size_t bytes = configure_split(a, k, cg_in, n_img, out_elems, sp, sp_pack, c.split)) {
    c.pack_bytes = bytes;
    return c;
  }
  plan_corr(a, k, out_elems, zero_fill, tile);
  if (one_launch) c.small = configure_corr_small(a, k, w_elems, out_elems, zero_fill, 4, tiled_time(a, tile, out_elems, backward, zero_fill), small);
  // one launch uses no workspace; what it asks for stays within what the rules' tile would
  if (c.small < 0) c.pack_bytes = (size_t)a.G * (size_t)a.KP * (size_t)a.MP * 4 + (size_t)a.KP * sizeof(KTabEntry);
  return c;
}

// Decides whether wgrad_small_kernel runs the backward filter instead of the launches of `w` (tiles of bm x bn, steps of
// 32 columns); fills a and returns its tile, -1 if it does not.
int32_t configure_wgrad_small(const WgradArgs& w, int64_t N, int32_t elem_bytes, int32_t bm, int32_t bn, WgradSmallArgs& a) {
  const int64_t limit = (int64_t)1 << 30, TH = w.khw / w.kw;
  if (w.sh * w.sw > 1 && w.dh * w.dw > 1) return -1;  // not measured: layers with a stride and a dilation
  const double flops = 2.0 * w.Kg * w.Kred * (double)w.ncols * w.G;
  if (flops > 1e9) return -1;
  // Doubles over fewer than 64 places: what a workgroup costs beside its one block is dearer than the fit has it.  0.71 of the tiles' time
  // with one 16x16 tile a compute unit, 0.78 with two, 1.02 with more (up to 1.35; floats 0.73).
  if (elem_bytes == 8 && w.ncols < 64 && (int64_t)w.G * parts_of(w.Kg, 16) * parts_of(w.Kred, 16) > 512) return -1;
  if (w.ncols < 1 || (int64_t)w.x_bytes > limit || (int64_t)w.dy_bytes > limit) return -1;
  if (w.H > 16384 || w.W > 16384 || w.ph > 4096 || w.pw > 4096) return -1;  // packed into 16 bits
  if ((TH - 1) * w.dh > 8192 || (int64_t)(w.kw - 1) * w.dw > 8192) return -1;
  a = WgradSmallArgs();
  static_cast<WgradArgs&>(a) = w;
  a.N = (int32_t)N;
  a.xvec = w.khw == 1 && w.sh == 1 && w.sw == 1 && w.ph == 0 && w.pw == 0;
  auto set_runs = [&](WgradSmallArgs& r) {
    r.row_runs = (int32_t)ceil_div(w.PW, 4);
    r.runs = r.xvec == 2 ? (int32_t)(w.P / w.PW) * r.row_runs : (int32_t)ceil_div(w.P, 4);
    r.mRuns = make_magic((uint32_t)r.runs);
    r.mRowRuns = make_magic((uint32_t)r.row_runs);
    r.blocks = (int32_t)ceil_div(N * r.runs, 16);
  };
  a.pad = w.ph > 0 || w.pw > 0;
  // [doubles][xvec][tile], and what a reduce launch costs: fits to every tile and 1 to 128 slices on 182 (doubles: 64) filter
  // gradients, rms errors 10 to 25 %; the choice is 3 (doubles: 5) % behind the best on average.  Runs within rows of doubles
  // are two loads each and took 1.09 times as long as single ones: no instance.
  static const SmallCost kCost[2][3][WGRAD_SMALL_COUNT] = {
      {{{0.453, 0.190, 0.41}, {0.476, 0.321, 0.97}, {0.598, 0.268, 0.91}, {0.883, 0.412, 1.30}, {1.422, 0.365, 0.36}},
       {{0.000, 0.154, 0.36}, {0.093, 0.211, 0.86}, {0.129, 0.227, 0.59}, {0.599, 0.289, 1.21}, {0.986, 0.221, 0.60}},
       {{0.341, 0.124, 0.75}, {0.585, 0.200, 1.13}, {0.653, 0.194, 1.04}, {1.058, 0.311, 1.45}, {1.593, 0.268, 0.47}}},
      {{{0.000, 0.329, 0.93}, {0.000, 0.488, 2.37}, {0.000, 0.494, 2.18}, {}, {0.780, 0.682, 2.28}},
       {{0.000, 0.438, 0.00}, {0.000, 0.681, 0.00}, {0.000, 0.635, 0.00}, {}, {1.190, 0.801, 0.00}},
       {}}};
  const double w_mb = 1e-6 * elem_bytes * (double)w.part_stride;
  const int32_t first = a.xvec, last = elem_bytes == 4 && w.sw == 1 && first == 0 ? 2 : first;
  int32_t best = -1, best_xvec = 0;
  int64_t best_bps = 0;
  double here = 0;
  for (a.xvec = first; a.xvec <= last; a.xvec += 2) {
    set_runs(a);
    for (int32_t t = 0; t < WGRAD_SMALL_COUNT; ++t) {
      const SmallCost& c = kCost[elem_bytes == 8][a.xvec][t];
      const SmallTile& s = kWgradSmallTiles[t];
      if (c.shared == 0) continue;  // no instance
      const int64_t tiles = (int64_t)w.G * parts_of(w.Kg, 16 * (uint32_t)s.mb) * parts_of(w.Kred, 16 * (uint32_t)s.nb);
      // a running sum hardly longer than on the tiled kernel: one of 256 was up to 1.3 times as far off as the slices there
      const int64_t sums = s.waves * (elem_bytes == 8 ? 1 : 4 / (s.mb * s.nb)), free = elem_bytes == 8 ? 2048 : 192;
      const int64_t longest = sums * ((w.cols_per_split > free ? w.cols_per_split : free) + 1);
      for (uint32_t S = 1; S <= (uint32_t)w.S; S *= 2) {  // at most the slices that the workspace has room for
        const uint32_t bps = parts_of(a.blocks, S), slices = parts_of(a.blocks, bps);
        const int64_t per_cu = (tiles * slices + 255) >> 8;
        if ((int64_t)bps * 64 >= longest) continue;
        const double cost = 3.3 + c.chain * (double)parts_of(bps, (uint32_t)s.waves) + (c.shared * (double)bps + c.workgroup) * (double)per_cu +
                            (slices > 1 ? 2.0 + (elem_bytes == 8 ? 1.0 : 1.6) * (double)slices * w_mb : 0.0);
        if (best < 0 || cost < here) {
          best = t;
          best_xvec = a.xvec;
          best_bps = bps;
          here = cost;
        }
      }
    }
  }
  if (best < 0) return -1;
  a.xvec = best_xvec;
  set_runs(a);
  // The launches of `w`, a fit to as many layers (rms errors 7 and 16 %).  With the margins below 136 of 190 layers of floats up to 4
  // GFLOP are taken, 1.42 times as fast in the geometric mean over all, three more than 3 % slower; doubles 90 of 110, 1.20 times, six.
  static const double kOld[2][7] = {{3.2, 0.74, 0.236, 0.374, 0.115, 0.242, 2.9}, {4.7, 0.63, 1.46, 1.91, 0.0, 0.222, 1.9}};
  const double* const o = kOld[elem_bytes == 8];
  const double area = (double)(bm * bn) / 4096.0;
  const int64_t steps = ceil_div(w.cols_per_split, 32), per_cu = ceil_div((int64_t)w.G * w.m_tiles * w.n_tiles * w.S, 256);
  const double old = o[0] + o[1] * w.S * w_mb + (double)steps * (o[2] + o[3] * area) +
                     (double)(per_cu * steps) * (o[4] + o[5] * area + (elem_bytes == 4 && w.bounds_mode == 1 ? 0.32 : 0.0)) + o[6] * (double)per_cu;
  // Of other gradients, over fewer than 64 places, 430 of floats take 0.55 of the tiles' time and 400 of doubles 0.75, 23 over 1.1 times.
  // 1x1 layers and fully connected ones need another 1.2: rows of x far apart cost more than the fit knows (28 x 3090 -> 3506
  // outputs took 26.9 us here, 21.7 on the tiles).
  const double least = (flops < 0.5e9 ? 0.9 : 0.75) / (a.xvec == 1 && elem_bytes == 4 ? 1.2 : 1.0);
  if (here > least * old) return -1;
  a.m_tiles = (int32_t)ceil_div(a.Kg, 16 * kWgradSmallTiles[best].mb);
  a.n_tiles = (int32_t)ceil_div(a.Kred, 16 * kWgradSmallTiles[best].nb);
  a.blocks_per_split = (int32_t)best_bps;
  a.S = (int32_t)ceil_div(a.blocks, best_bps);
  if ((int64_t)a.S * a.G * a.m_tiles * a.n_tiles >= ((int64_t)1 << 31)) return -1;
  return best;
}

// The split kernel's launches; its partial sums, if any, lie behind the packed weights.
int launch_split(int32_t tile, const PackSplitArgs& pack, const CorrSplitArgs& plan, size_t pack_bytes, const float* in,
                 const float* w, const float* bias, float* out, bool accumulate, void* ws, void* stream) {
  PackSplitArgs k = pack;
  k.w = w;
  k.A = static_cast<float*>(ws);
  k.in = in;
  if (k.half) {
    k.unheld = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + (size_t)k.fragments * 5120);
    k.scale = reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + pack_bytes - kSampleBytes);
  }
  if (const int e = launch_pack_split(tile, k, stream)) return e;
  CorrSplitArgs a = plan;
  a.scale = k.scale;
  a.unheld = k.unheld;
  a.A = k.A;
  a.in = in;
  a.bias = bias;
  a.out = out;
  a.accumulate = accumulate;
  a.part = reinterpret_cast<float*>(static_cast<char*>(ws) + pack_bytes);
  return launch_corr_split(tile, a, stream);
}

}  // namespace

namespace mi355conv {

int record_hip_error(int e) {
  g_last_hip_error = e;
  return CONV_EHIP;
}

int conv_desc_backward_filter_workspace_bytes(const conv_desc* d, size_t* bytes) {
  if (!d || !bytes) return CONV_EINVAL;
  *bytes = d->wg_ws;
  return CONV_OK;
}

int run_forward(const conv_desc* d, const float* x, const float* w, const float* bias, float* y, void* ws,
                size_t ws_bytes, void* hip_stream) {
  if (!d || !w) return CONV_EINVAL;
  if ((d->p.bias_term != 0) != (bias != nullptr)) return CONV_EINVAL;
  if (d->p.n == 0) return CONV_OK;  // empty blobs: nothing to read or write
  if (!x || !y) return CONV_EINVAL;
  if (d->use_direct) {
    DirectArgs da = d->dir;
    da.in = x;
    da.w = w;
    da.bias = bias;
    da.out = y;
    const int ed = launch_direct(0, da, false, hip_stream);
    return ed ? record_hip_error(ed) : CONV_OK;
  }
  if (d->fwd_ws > 0 && (!ws || ws_bytes < d->fwd_ws)) return CONV_EWORKSPACE;
  if (d->fwd_small[0] >= 0) {
    CorrSmallArgs a = d->fwd_sm[0];
    a.A = w;
    a.in = x;
    a.bias = bias;
    a.out = y;
    const int es = launch_corr_small(d->fwd_small[0], a, false, hip_stream);
    return es ? record_hip_error(es) : CONV_OK;
  }
  float* const part = reinterpret_cast<float*>(static_cast<char*>(ws) + d->fwd_pack_bytes);
  const bool split = d->fwd_split >= 0;
  int e;
  if (split) {
    e = launch_split(d->fwd_split, d->fwd_sp_pack, d->fwd_sp, d->fwd_pack_bytes, x, w, bias, y, false, ws, hip_stream);
  } else {
    PackArgs k = d->fwd_pack;
    k.w = w;
    k.A = static_cast<float*>(ws);
    k.ktab = reinterpret_cast<KTabEntry*>(k.A + (size_t)k.G * k.KP * k.MP);
    const bool in_place = d->fwd_thin && d->fwd.use_patch;  // that kernel reads the weight blob itself
    e = in_place ? 0 : launch_pack(k, hip_stream);
    if (e) return record_hip_error(e);
    CorrArgs a = d->fwd;
    a.A = in_place ? w : k.A;
    a.ktab = k.ktab;
    a.in = x;
    a.bias = bias;
    a.out = y;
    a.part = part;
    e = d->fwd_thin  ? launch_corr_thin(a, hip_stream)
        : a.use_patch ? launch_corr_patch(d->fwd_tile, a, hip_stream)
                      : launch_corr(d->fwd_tile, a, hip_stream);
  }
  if (e) return record_hip_error(e);
  const int32_t ksplit = split ? d->fwd_sp.ksplit : d->fwd.ksplit;
  if (ksplit > 1) {  // add the split partials and the bias
    ReduceArgs r = {};
    r.part = part;
    r.dst = y;
    r.count = d->fwd.out_elems;
    r.S = ksplit;
    r.beta = 0.f;
    r.bias = bias;
    r.chan_elems = d->OH * d->OW;
    r.channels = d->p.num_output;
    r.mChanElems = make_magic(r.chan_elems);
    r.mChannels = make_magic(r.channels);
    e = launch_reduce(r, hip_stream);
  }
  return e ? record_hip_error(e) : CONV_OK;
}

int run_backward_data(const conv_desc* d, const float* w, const float* dy, float* dx, float beta, void* ws,
                      size_t ws_bytes, void* hip_stream) {
  if (!d || !w) return CONV_EINVAL;
  if (!(beta == 0.f || beta == 1.f)) return CONV_EINVAL;
  if (d->p.n == 0) return CONV_OK;
  if (!dy || !dx) return CONV_EINVAL;
  if (d->use_direct) {
    DirectArgs da = d->dir;
    da.in = dy;
    da.w = w;
    da.out = dx;
    if (beta != 0.f) return CONV_EINVAL;  // accumulation into dx is only used by the ungrouped InnerProduct passes
    const int ed = launch_direct(1, da, false, hip_stream);
    return ed ? record_hip_error(ed) : CONV_OK;
  }
  if (d->bwd_ws > 0 && (!ws || ws_bytes < d->bwd_ws)) return CONV_EWORKSPACE;
  if (d->bwd_small[0] >= 0) {
    int es = d->bwd_zero_fill && beta == 0.f ? launch_fill_zero(dx, (size_t)d->bwd.out_elems * 4, hip_stream) : 0;
    if (es) return record_hip_error(es);
    CorrSmallArgs a = d->bwd_sm[0];
    a.A = w;
    a.in = dy;
    a.out = dx;
    a.accumulate = beta != 0.f;
    es = launch_corr_small(d->bwd_small[0], a, false, hip_stream);
    return es ? record_hip_error(es) : CONV_OK;
  }
  float* const part = reinterpret_cast<float*>(static_cast<char*>(ws) + d->bwd_pack_bytes);
  const bool split = d->bwd_split >= 0;
  const int32_t ksplit = split ? d->bwd_sp.ksplit : d->bwd.ksplit, out_elems = d->bwd.out_elems;
  int e = 0;
  if (d->bwd_zero_fill) {  // positions no tap reaches: zero the split partials, or dx itself when it is overwritten
    if (ksplit > 1)
      e = launch_fill_zero(part, (size_t)ksplit * out_elems * 4, hip_stream);
    else if (beta == 0.f)
      e = launch_fill_zero(dx, (size_t)out_elems * 4, hip_stream);
    if (e) return record_hip_error(e);
  }
  if (split) {
    e = launch_split(d->bwd_split, d->bwd_sp_pack, d->bwd_sp, d->bwd_pack_bytes, dy, w, nullptr, dx, beta != 0.f, ws,
                     hip_stream);
  } else {
    PackArgs k = d->bwd_pack;
    k.w = w;
    k.A = static_cast<float*>(ws);
    k.ktab = reinterpret_cast<KTabEntry*>(k.A + (size_t)k.G * k.KP * k.MP);
    const bool in_place = d->bwd_thin && d->bwd.use_patch;  // that kernel reads the weight blob itself
    e = in_place ? 0 : launch_pack(k, hip_stream);
    if (e) return record_hip_error(e);
    CorrArgs a = d->bwd;
    a.A = in_place ? w : k.A;
    a.ktab = k.ktab;
    a.in = dy;
    a.bias = nullptr;
    a.out = dx;
    a.accumulate = beta != 0.f;
    a.part = part;
    e = d->bwd_thin  ? launch_corr_thin(a, hip_stream)
        : a.use_patch ? launch_corr_patch(d->bwd_tile, a, hip_stream)
                      : launch_corr(d->bwd_tile, a, hip_stream);
  }
  if (e) return record_hip_error(e);
  if (ksplit > 1) {
    ReduceArgs r = {};
    r.part = part;
    r.dst = dx;
    r.count = out_elems;
    r.S = ksplit;
    r.beta = beta;
    e = launch_reduce(r, hip_stream);
  }
  return e ? record_hip_error(e) : CONV_OK;
}

size_t forward_transposed_workspace_bytes(const conv_desc* d) {
  if (d->fwd_split < 0 || !d->fwd_sp.fold.pixels || !d->fwd_sp.simple_epilogue || d->p.group != 1) return 0;
  return d->fwd_pack_bytes + (size_t)d->fwd_sp.ksplit * (size_t)d->fwd_sp.out_elems * 4;
}

int run_forward_transposed(const conv_desc* d, const float* x, const float* w, float* y, void* ws, size_t ws_bytes,
                           void* hip_stream, const ReduceExtras& extras) {
  if (!ws || ws_bytes < forward_transposed_workspace_bytes(d)) return CONV_EWORKSPACE;
  float* const part = reinterpret_cast<float*>(static_cast<char*>(ws) + d->fwd_pack_bytes);
  CorrSplitArgs plan = d->fwd_sp;
  plan.OWd = d->p.n;  // a row of the output is one channel of all images
  plan.out_img_stride = 1;
  int e = launch_split(d->fwd_split, d->fwd_sp_pack, plan, d->fwd_pack_bytes, x, w, nullptr, part, false, ws, hip_stream);
  if (e) return record_hip_error(e);
  ReduceArgs r = {};
  r.part = part;
  r.dst = y;
  r.count = plan.out_elems;
  r.S = plan.ksplit;
  r.bias = extras.bias;
  r.chan_elems = extras.chan_elems;
  r.channels = extras.channels;
  r.mChanElems = make_magic(r.chan_elems);
  r.mChannels = make_magic(r.channels);
  r.relu = extras.relu;
  e = launch_reduce(r, hip_stream);
  return e ? record_hip_error(e) : CONV_OK;
}

int run_backward_filter(const conv_desc* d, const float* x, const float* dy, float* dw, float beta, void* ws,
                        size_t ws_bytes, void* hip_stream, const ReduceExtras& extras, float* db) {
  if (!d || !dw) return CONV_EINVAL;
  if (!(beta == 0.f || beta == 1.f)) return CONV_EINVAL;
  const bool empty = d->p.n == 0;  // the gradient sum is empty: dw = beta*dw
  if (!empty && (!x || !dy)) return CONV_EINVAL;
  const size_t need = db ? d->wgb_ws : d->wg_ws;
  if (!empty && need > 0 && (!ws || ws_bytes < need)) return CONV_EWORKSPACE;
  const int32_t w_elems = (int32_t)((int64_t)d->p.num_output * d->wg.Kred);
  WgradArgs a = d->wg;
  a.dy = dy;
  a.x = x;
  a.part = static_cast<float*>(ws);
  int e = 0;
  if (d->use_direct) {
    // thin groups: the direct filter-gradient kernel; its workgroups of a group's first input channel
    // also add up the dy values they read (S x K sums behind the filter partials)
    DirectArgs da = d->dir;
    da.in = x;
    da.w = dy;
    da.part = ws;
    a.S = da.S;
    a.n_tiles = 1;
    if (db) da.bias_part = a.bias_part = a.part + (size_t)da.S * w_elems;
    if (!empty) e = launch_direct(2, da, false, hip_stream);
  } else if (d->wg_small[0] >= 0 && !empty) {
    WgradSmallArgs sa = d->wg_sm[0];
    a.S = sa.S;
    a.n_tiles = 1;  // one share of the row sums per slice
    sa.dy = dy;
    sa.x = x;
    sa.part = a.part;
    sa.dw_out = dw;
    sa.beta = beta;
    if (db) sa.bias_part = a.bias_part = sa.S == 1 ? db : a.part + (size_t)sa.S * w_elems;
    if (sa.S == 1) {
      if (extras.bias) sa.col_bias = extras.bias;
      sa.relu = extras.relu;
    }
    e = launch_wgrad_small(d->wg_small[0], sa, false, hip_stream);
    if (e || sa.S == 1) return e ? record_hip_error(e) : CONV_OK;
  } else if (d->wg_split >= 0 || d->wg_fold >= 0) {
    WgradSplitArgs sa = d->wg_sp;
    a.S = sa.S;
    a.n_tiles = sa.n_tiles;
    if (db) a.bias_part = a.part + (size_t)a.S * sa.part_stride;
    sa.dy = dy;
    sa.x = x;
    sa.part = a.part;
    sa.bias_part = a.bias_part;
    if (!empty) e = d->wg_fold >= 0 ? launch_wgrad_fold(d->wg_fold, sa, hip_stream) : launch_wgrad_split(d->wg_split, sa, hip_stream);
  } else if (!empty) {
    if (db) a.bias_part = a.part + (size_t)a.S * w_elems;  // row sums of dy ride along, behind the filter partials
    e = launch_wgrad(d->wg_tile, a, hip_stream);
  }
  if (e) return record_hip_error(e);
  ReduceArgs r = {};
  r.part = a.part;
  r.dst = dw;
  r.count = w_elems;
  r.S = empty ? 0 : a.S;
  r.beta = beta;
  r.bias = extras.bias;
  r.chan_elems = extras.chan_elems;
  r.channels = extras.channels;
  r.mChanElems = make_magic(r.chan_elems);
  r.mChannels = make_magic(r.channels);
  r.relu = extras.relu;
  if (db) {  // the same launch finishes db from the S * n_tiles shares of the row sums
    r.part2 = empty ? nullptr : a.bias_part;
    r.dst2 = db;
    r.count2 = d->p.num_output;
    r.S2 = empty ? 0 : a.S * a.n_tiles;
  }
  if (d->wg_fold >= 0 && !d->use_direct) {
    ReduceFoldArgs rf;
    static_cast<ReduceArgs&>(rf) = r;
    rf.count = d->wg_sp.part_stride;
    rf.taps = d->wg_sp.khw;
    rf.tap_channels = d->wg_sp.fold.V;
    rf.mRow = make_magic((uint32_t)d->wg_sp.Kred);
    rf.mTapChannels = make_magic((uint32_t)rf.tap_channels);
    rf.fold = d->wg_sp.fold;
    rf.channels = d->wg_sp.Cg;
    rf.grid_w = d->wg_sp.kw;
    e = launch_reduce_fold(rf, hip_stream);
  } else if (d->wg_split >= 0 && !d->use_direct && d->wg_sp.khw > 1) {
    ReduceTapsArgs rt;
    static_cast<ReduceArgs&>(rt) = r;
    rt.taps = d->wg_sp.khw;
    rt.tap_channels = d->wg_sp.Cg;
    rt.mRow = make_magic((uint32_t)d->wg_sp.Kred);
    rt.mTapChannels = make_magic((uint32_t)d->wg_sp.Cg);
    e = launch_reduce_taps(rt, hip_stream);
  } else {
    e = launch_reduce(r, hip_stream);
  }
  return e ? record_hip_error(e) : CONV_OK;
}

}  // namespace mi355conv

extern "C" {

// one_launch: the kernels of small layers may be taken (conv_desc_create_tiled leaves them out)
static int create_desc(conv_desc_t** out, const conv_params_t* pp, bool one_launch) {
  if (!out || !pp) return CONV_EINVAL;
  const conv_params_t p = *pp;
  if (p.n < 0 || p.c < 1 || p.h < 1 || p.w < 1 || p.num_output < 1) return CONV_EINVAL;
  if (p.kernel_h < 1 || p.kernel_w < 1 || p.stride_h < 1 || p.stride_w < 1) return CONV_EINVAL;
  if (p.pad_h < 0 || p.pad_w < 0 || p.dilation_h < 1 || p.dilation_w < 1) return CONV_EINVAL;
  if (p.group < 1 || p.c % p.group != 0 || p.num_output % p.group != 0) return CONV_EINVAL;
  if (p.bias_term != 0 && p.bias_term != 1) return CONV_EINVAL;

  const int64_t ext_h = (int64_t)p.dilation_h * (p.kernel_h - 1) + 1;
  const int64_t ext_w = (int64_t)p.dilation_w * (p.kernel_w - 1) + 1;
  const int64_t OH = floor_div((int64_t)p.h + 2 * (int64_t)p.pad_h - ext_h, p.stride_h) + 1;
  const int64_t OW = floor_div((int64_t)p.w + 2 * (int64_t)p.pad_w - ext_w, p.stride_w) + 1;
  if (OH < 1 || OW < 1) return CONV_ESHAPE;
  // tap offsets are packed into 16 bits, coordinates into 28
  if (ext_h > 32768 || ext_w > 32768 || p.pad_h > (1 << 20) || p.pad_w > (1 << 20)) return CONV_ESHAPE;
  if (p.h > (1 << 24) || p.w > (1 << 24) || p.stride_h > (1 << 20) || p.stride_w > (1 << 20)) return CONV_ESHAPE;

  const int64_t N = p.n, C = p.c, H = p.h, W = p.w, K = p.num_output, G = p.group;
  const int64_t Cg = C / G, Kg = K / G;
  const int64_t kred = Cg * p.kernel_h * p.kernel_w;
  // sizes in 128-bit arithmetic first: four 31-bit factors do not fit 64 bits
  const __int128 big = kMaxElems;
  if ((__int128)C * H * W >= big || (__int128)K * OH * OW >= big || (__int128)N * C * H * W >= big ||
      (__int128)N * K * OH * OW >= big || (__int128)K * Cg * p.kernel_h * p.kernel_w >= big)
    return CONV_ESHAPE;
  const int64_t x_elems = N * C * H * W, y_elems = N * K * OH * OW, w_elems = K * kred;

  conv_desc* d = new (std::nothrow) conv_desc;
  if (!d) return CONV_EINVAL;
  memset(d, 0, sizeof(*d));
  d->p = p;
  d->OH = (int32_t)OH;
  d->OW = (int32_t)OW;
  d->Cg = (int32_t)Cg;
  d->Kg = (int32_t)Kg;

  int32_t bm, bn, bk;

  // ---- forward: rows = output channels of a group, k = (c, i, j), columns = (n, oh, ow) ----
  {
    d->fwd_tile = pick_corr_tile((int32_t)Kg, G, N * OH * OW, kred, (int64_t)p.kernel_h * p.kernel_w,
                                 p.stride_h == 1 && p.stride_w == 1 && p.dilation_h == 1 && p.dilation_w == 1 && Cg % 8 == 0);
    corr_tile_shape(d->fwd_tile, &bm, &bn, &bk);
    CorrArgs& a = d->fwd;
    a.ncols = (int32_t)(N * OH * OW);
    a.P = (int32_t)(OH * OW);
    a.PW = (int32_t)OW;
    a.mP = make_magic(a.P);
    a.mPW = make_magic(a.PW);
    a.IH = p.h;
    a.IW = p.w;
    a.IHW = p.h * p.w;
    a.in_img_stride = (int32_t)(C * H * W);
    a.in_grp_stride = (int32_t)(Cg * H * W);
    a.in_bytes = (uint32_t)(4 * x_elems);
    a.bounds_mode = bounds_mode(p.pad_h == 0 && p.pad_w == 0, (int64_t)p.kernel_h * p.kernel_w, 4 * x_elems,
                                4 * ((p.pad_h + ext_h) * W + p.pad_w + ext_w));
    a.TW = p.kernel_w;
    a.THW = p.kernel_h * p.kernel_w;
    a.mTW = make_magic(a.TW);
    a.mTHW = make_magic(a.THW);
    a.sh = p.stride_h;
    a.sw = p.stride_w;
    a.dh = p.dilation_h;
    a.dw = p.dilation_w;
    a.ph = p.pad_h;
    a.pw = p.pad_w;
    a.Kred = (int32_t)kred;
    a.KP = (int32_t)round_up(kred, bk);
    a.Mrows = (int32_t)Kg;
    a.MP = (int32_t)round_up(Kg, bm);
    a.RSh = a.RSw = a.RShw = 1;
    a.OSh = a.OSw = 1;
    a.mRSw = make_magic(1);
    a.mRShw = make_magic(1);
    a.opad_h = a.opad_w = 0;
    a.OHd = (int32_t)OH;
    a.OWd = (int32_t)OW;
    a.out_img_stride = (int32_t)(K * OH * OW);
    a.chan_per_grp = (int32_t)Kg;
    a.G = (int32_t)G;
    a.m_tiles = a.MP / bm;
    a.col_tiles = (int32_t)ceil_div(a.ncols, bn);
    PackArgs& k = d->fwd_pack;
    k.mode = 0;
    k.G = (int32_t)G;
    k.Kg = (int32_t)Kg;
    k.Cg = (int32_t)Cg;
    k.kh = p.kernel_h;
    k.kw = p.kernel_w;
    k.sh = k.sw = k.dh = k.dw = 1;
    k.Qh = k.Qw = 1;
    k.Kred = a.Kred;
    k.KP = a.KP;
    k.Mrows = a.Mrows;
    k.MP = a.MP;
    k.tTW = a.TW;
    k.tTHW = a.THW;
    k.tIW = a.IW;
    k.tIHW = a.IHW;
    k.tdh = a.dh;
    k.tdw = a.dw;
    k.koff_invalid = koff_invalid(a.bounds_mode);
    configure_patch(a, k, Cg, N, bm, bn);
    configure_ksplit(a, y_elems, bm, bn);
    const CorrChoice c = choose_corr(a, k, d->fwd_tile, Cg, N, false, y_elems, w_elems, false, one_launch, d->fwd_sp, d->fwd_sp_pack, d->fwd_sm[0]);
    if (c.pack_bytes == 0) {
      delete d;
      return CONV_ESHAPE;
    }
    d->fwd_thin = c.thin;
    d->fwd_split = c.split;
    d->fwd_small[0] = c.small;
    d->fwd_pack_bytes = c.pack_bytes;
    const int32_t S = c.small >= 0 ? 1 : c.split >= 0 ? d->fwd_sp.ksplit : a.ksplit;
    d->fwd_ws = d->fwd_pack_bytes + (S > 1 ? (size_t)S * y_elems * 4 : 0);
  }

  // ---- backward data: a stride-1 correlation over dy whose rows are (c, row phase, column
  // phase) of dx -- input position h + pad = stride*a + rh collects the taps i with
  // i*dilation = stride*q + rh from dy row a - q (see phase_dim for the tap slots and the phases
  // kept).  Positions with a < a0 = pad / stride lie wholly in the padding, so the column space
  // starts at a0. ----
  {
    const PhaseDim dim_h = phase_dim(p.kernel_h, p.stride_h, p.dilation_h);
    const PhaseDim dim_w = phase_dim(p.kernel_w, p.stride_w, p.dilation_w);
    const int64_t Qh = dim_h.Q, Qw = dim_w.Q;
    const int64_t a0h = p.pad_h / p.stride_h, a0w = p.pad_w / p.stride_w;
    const int64_t Ah = (H - 1 + p.pad_h) / p.stride_h + 1 - a0h;
    const int64_t Aw = (W - 1 + p.pad_w) / p.stride_w + 1 - a0w;
    const int64_t rows = Cg * dim_h.nv * dim_w.nv;
    const int64_t kred_b = Kg * Qh * Qw;
    d->bwd_zero_fill = dim_h.nv < p.stride_h || dim_w.nv < p.stride_w;
    if (rows >= ((int64_t)1 << 24) || N * Ah * Aw >= ((int64_t)1 << 31) || kred_b >= kMaxElems) {
      delete d;
      return CONV_ESHAPE;
    }
    d->bwd_tile = pick_corr_tile((int32_t)rows, G, N * Ah * Aw, kred_b, Qh * Qw, Kg % 8 == 0);
    corr_tile_shape(d->bwd_tile, &bm, &bn, &bk);
    CorrArgs& a = d->bwd;
    a.ncols = (int32_t)(N * Ah * Aw);
    a.P = (int32_t)(Ah * Aw);
    a.PW = (int32_t)Aw;
    a.mP = make_magic(a.P);
    a.mPW = make_magic(a.PW);
    a.IH = (int32_t)OH;
    a.IW = (int32_t)OW;
    a.IHW = (int32_t)(OH * OW);
    a.in_img_stride = (int32_t)(K * OH * OW);
    a.in_grp_stride = (int32_t)(Kg * OH * OW);
    a.in_bytes = (uint32_t)(4 * y_elems);
    a.bounds_mode = bounds_mode(false, Qh * Qw, 4 * y_elems,
                                4 * (2 * ((Qh - 1) * dim_h.e + 1) * OW + 2 * ((Qw - 1) * dim_w.e + 1)));
    a.TW = (int32_t)Qw;
    a.THW = (int32_t)(Qh * Qw);
    a.mTW = make_magic(a.TW);
    a.mTHW = make_magic(a.THW);
    a.sh = a.sw = 1;
    a.dh = (int32_t)dim_h.e;
    a.dw = (int32_t)dim_w.e;
    a.ph = (int32_t)((Qh - 1) * dim_h.e - a0h);
    a.pw = (int32_t)((Qw - 1) * dim_w.e - a0w);
    a.Kred = (int32_t)kred_b;
    a.KP = (int32_t)round_up(kred_b, bk);
    a.Mrows = (int32_t)rows;
    a.MP = (int32_t)round_up(rows, bm);
    a.RSh = (int32_t)dim_h.nv;
    a.RSw = (int32_t)dim_w.nv;
    a.RShw = a.RSh * a.RSw;
    a.mRSw = make_magic(a.RSw);
    a.mRShw = make_magic(a.RShw);
    a.OSh = p.stride_h;
    a.OSw = p.stride_w;
    a.tab_h = dim_h.tab;
    a.tab_w = dim_w.tab;
    for (int i = 0; i < kMaxPhases; ++i) {
      a.phase_h[i] = dim_h.phase[i];
      a.phase_w[i] = dim_w.phase[i];
    }
    a.opad_h = (int32_t)(p.pad_h - a0h * p.stride_h);
    a.opad_w = (int32_t)(p.pad_w - a0w * p.stride_w);
    a.OHd = p.h;
    a.OWd = p.w;
    a.out_img_stride = (int32_t)(C * H * W);
    a.chan_per_grp = (int32_t)Cg;
    a.G = (int32_t)G;
    a.m_tiles = a.MP / bm;
    a.col_tiles = (int32_t)ceil_div(a.ncols, bn);
    PackArgs& k = d->bwd_pack;
    k.mode = 1;
    k.G = (int32_t)G;
    k.Kg = (int32_t)Kg;
    k.Cg = (int32_t)Cg;
    k.kh = p.kernel_h;
    k.kw = p.kernel_w;
    k.sh = p.stride_h;
    k.sw = p.stride_w;
    k.dh = p.dilation_h;
    k.dw = p.dilation_w;
    k.Qh = (int32_t)Qh;
    k.Qw = (int32_t)Qw;
    k.nvh = a.RSh;
    k.nvw = a.RSw;
    k.eh = a.dh;
    k.ew = a.dw;
    k.tab_h = a.tab_h;
    k.tab_w = a.tab_w;
    for (int i = 0; i < kMaxPhases; ++i) {
      k.phase_h[i] = a.phase_h[i];
      k.phase_w[i] = a.phase_w[i];
    }
    k.Kred = a.Kred;
    k.KP = a.KP;
    k.Mrows = a.Mrows;
    k.MP = a.MP;
    k.tTW = a.TW;
    k.tTHW = a.THW;
    k.tIW = a.IW;
    k.tIHW = a.IHW;
    k.tdh = a.dh;
    k.tdw = a.dw;
    k.koff_invalid = koff_invalid(a.bounds_mode);
    configure_patch(a, k, Kg, N, bm, bn);
    configure_ksplit(a, x_elems, bm, bn);
    const CorrChoice c = choose_corr(a, k, d->bwd_tile, Kg, N, true, x_elems, w_elems, d->bwd_zero_fill != 0, one_launch, d->bwd_sp, d->bwd_sp_pack,
                                     d->bwd_sm[0]);
    if (c.pack_bytes == 0) {
      delete d;
      return CONV_ESHAPE;
    }
    d->bwd_thin = c.thin;
    d->bwd_split = c.split;
    d->bwd_small[0] = c.small;
    d->bwd_pack_bytes = c.pack_bytes;
    const int32_t S = c.small >= 0 ? 1 : c.split >= 0 ? d->bwd_sp.ksplit : a.ksplit;
    d->bwd_ws = d->bwd_pack_bytes + (S > 1 ? (size_t)S * x_elems * 4 : 0);
  }

  // ---- backward filter: rows = output channels, columns = (c, i, j), reduction over (n, oh, ow)
  {
    d->wg_tile = pick_wgrad_tile((int32_t)Kg, (int32_t)kred);
    wgrad_tile_shape(d->wg_tile, &bm, &bn, &bk);
    WgradArgs& a = d->wg;
    a.ncols = (int32_t)(N * OH * OW);
    a.P = (int32_t)(OH * OW);
    a.PW = (int32_t)OW;
    a.mP = make_magic(a.P);
    a.mPW = make_magic(a.PW);
    a.dy_bytes = (uint32_t)(4 * y_elems);
    a.x_bytes = (uint32_t)(4 * x_elems);
    // the dy base of a column past the split is 2^31: both blobs must stay below that for modes 0 and 2
    a.bounds_mode = 1;
    if (4 * y_elems < ((int64_t)1 << 31) - 4) {
      a.bounds_mode = bounds_mode(p.pad_h == 0 && p.pad_w == 0, (int64_t)p.kernel_h * p.kernel_w, 4 * x_elems,
                                  4 * ((p.pad_h + ext_h) * W + p.pad_w + ext_w));
      if (a.bounds_mode == 2 && (p.dilation_h != 1 || p.dilation_w != 1 || p.kernel_h * p.kernel_w > 31))
        a.bounds_mode = 1;
    }
    a.Kg = (int32_t)Kg;
    a.Ktot = (int32_t)K;
    a.Cg = (int32_t)Cg;
    a.C = p.c;
    a.H = p.h;
    a.W = p.w;
    a.HW = p.h * p.w;
    a.kw = p.kernel_w;
    a.khw = p.kernel_h * p.kernel_w;
    a.mKW = make_magic(a.kw);
    a.mKHW = make_magic(a.khw);
    a.sh = p.stride_h;
    a.sw = p.stride_w;
    a.dh = p.dilation_h;
    a.dw = p.dilation_w;
    a.ph = p.pad_h;
    a.pw = p.pad_w;
    a.Kred = (int32_t)kred;
    a.G = (int32_t)G;
    a.m_tiles = (int32_t)ceil_div(Kg, bm);
    a.n_tiles = (int32_t)ceil_div(kred, bn);
    // Split the reduction so that the whole grid is resident at once -- LDS holds two workgroups per
    // compute unit (three of the 32-row tile), and a grid of 1.4 times that many runs a second,
    // mostly empty round (5.a: 714 workgroups on 512 places took 255 us, 507 take 234) -- with each
    // split at least four k tiles long and the partials at most 32 MiB; a grid slightly above a
    // multiple of the 256 compute units is trimmed back to it (its last few workgroups would
    // otherwise share a compute unit while the others have one to themselves).
    const int64_t max_by_len = ceil_div((int64_t)a.ncols, 4 * bk);
    const int64_t max_by_ws = ((int64_t)8 << 20) / (w_elems > 0 ? w_elems : 1);
    auto splits_for = [&](int64_t tiles, int64_t places) {
      int64_t S = places / tiles;
      if (S > max_by_len) S = max_by_len;
      if (S > max_by_ws) S = max_by_ws;
      if (S > 256) S = 256;  // beyond one split per compute unit the reduce kernel only gets slower
      if (S < 1) S = 1;
      while (S > 1 && tiles * S > 256 && (tiles * S) % 256 != 0 && (tiles * S) % 256 < 64) --S;
      return S;
    };
    int64_t tiles = G * a.m_tiles * a.n_tiles;
    int64_t S = splits_for(tiles, 256 * (bm == 32 ? 3 : 2));
    // A grid that cannot fill the compute units because its splits are as short as they may get takes
    // the 32-row tile instead of the 64-row one when both pad the rows alike: twice the workgroups,
    // three resident per compute unit (2.a 12.9 -> 10.8 us, 3.b 13.2 -> 11.0, 3.c 12.3 -> 10.1).
    if (d->wg_tile == WGRAD_64x128 && tiles * S < 256 && round_up(Kg, 32) == round_up(Kg, 64)) {
      d->wg_tile = WGRAD_32x128;
      wgrad_tile_shape(d->wg_tile, &bm, &bn, &bk);
      a.m_tiles = (int32_t)ceil_div(Kg, bm);
      a.n_tiles = (int32_t)ceil_div(kred, bn);
      tiles = G * a.m_tiles * a.n_tiles;
      S = splits_for(tiles, 256 * 3);
    }
    a.cols_per_split = (int32_t)round_up(ceil_div((int64_t)a.ncols > 0 ? a.ncols : 1, S), bk);
    a.S = (int32_t)ceil_div((int64_t)a.ncols > 0 ? a.ncols : 1, a.cols_per_split);
    if (a.S * w_elems >= kMaxElems || tiles * a.S >= ((int64_t)1 << 31)) {
      delete d;
      return CONV_ESHAPE;
    }
    a.part_stride = (int32_t)w_elems;
    a.bias_part = nullptr;
    d->wg_ws = (size_t)a.S * (size_t)w_elems * 4;
    d->wgb_ws = (size_t)a.S * (size_t)(w_elems + a.n_tiles * K) * 4;
    if (a.S * (w_elems + a.n_tiles * K) >= kMaxElems) {
      delete d;
      return CONV_ESHAPE;
    }
    d->wg_split = configure_wgrad_split(a, d->wg_tile, N, K, w_elems, d->wg_sp);
    d->wg_fold = d->wg_split >= 0 ? -1 : configure_wgrad_fold(a, d->wg_tile, N, K, w_elems, d->wg_sp);
    d->wg_small[0] = d->wg_split >= 0 || d->wg_fold >= 0 || !one_launch ? -1 : configure_wgrad_small(a, N, 4, bm, bn, d->wg_sm[0]);
    if (d->wg_split >= 0 || d->wg_fold >= 0) {
      d->wg_ws = (size_t)d->wg_sp.S * (size_t)d->wg_sp.part_stride * 4;
      d->wgb_ws = (size_t)d->wg_sp.S * (size_t)(d->wg_sp.part_stride + d->wg_sp.n_tiles * K) * 4;
    }
  }

  // ---- backward bias ----
  char bias64[32];
  {
    BiasGradArgs& a = d->bg;
    a.N = p.n;
    a.K = p.num_output;
    a.P = (int32_t)(OH * OW);
    int64_t S = ceil_div(2048, K);
    if (S > N) S = N;
    if (S < 1) S = 1;
    // up to a megabyte: one workgroup per channel sums the whole batch and finishes db
    // itself -- the second launch would cost more than the lost parallelism
    d->bg_direct = y_elems * 4 <= ((int64_t)1 << 20);
    if (d->bg_direct) S = 1;
    a.n_per_split = (int32_t)ceil_div(N > 0 ? N : 1, S);
    a.S = (int32_t)ceil_div(N > 0 ? N : 1, a.n_per_split);
    d->bg_ws = p.bias_term ? (size_t)a.S * K * 4 : 0;
    a.mP = make_magic((uint32_t)a.P);
    d->bg64_direct = N * a.P <= kBias64Direct;
    snprintf(bias64, sizeof(bias64), "bias_grad64[%s](S=%d,L=%d)", d->bg64_direct ? "one" : "two", d->bg64_direct ? 1 : a.S,
             d->bg64_direct ? 1 : 2);
  }

  // ---- double base type: the same geometry on the fp64 tiles, compare-style bounds checks ----
  {
    const int32_t bn64 = kF64TileCols, bk64 = kF64TileK;
    const int64_t max64 = (int64_t)1 << 29;  // 32-bit byte offsets of 8-byte elements
    d->f64_ok = x_elems < max64 && y_elems < max64 && w_elems < max64;
    auto corr64 = [&](const CorrArgs& src, const PackArgs& psrc, CorrArgs& a, PackArgs& k, int64_t in_elems,
                      bool zero_fill, size_t& ws, int32_t& tile_rows, int32_t& small, CorrSmallArgs& sm) {
      a = src;
      const int32_t bm64 = tile_rows = f64_pick_rows(src.Mrows, false);
      a.in_bytes = (uint32_t)(8 * in_elems);
      a.bounds_mode = 1;
      a.KP = (int32_t)round_up(a.Kred, bk64);
      a.MP = (int32_t)round_up(a.Mrows, bm64);
      a.m_tiles = a.MP / bm64;
      a.col_tiles = (int32_t)ceil_div(a.ncols, bn64);
      a.use_patch = 0;
      a.accumulate = 0;
      configure_ksplit(a, src.out_elems, bm64, bn64, 8);  // the same rule on this tile's grid (chunks are 16 k rows here too)
      plan_corr64(a, src.out_elems, tile_rows);
      small = -1;
      if (one_launch)
        small = configure_corr_small(a, psrc, w_elems, src.out_elems, zero_fill, 8, corr64_model(a, tile_rows, src.out_elems, psrc.mode != 0, zero_fill), sm);
      a.simple_epilogue = src.simple_epilogue && 8 * (int64_t)src.out_elems <= ((int64_t)1 << 30);
      k = psrc;
      k.KP = a.KP;
      k.MP = a.MP;
      k.kperm_T = 0;
      k.koff_invalid = 0;
      const int64_t pack_elems = (int64_t)a.G * a.KP * a.MP;
      if (pack_elems >= max64 || (int64_t)a.G * a.m_tiles * a.col_tiles >= ((int64_t)1 << 31)) d->f64_ok = 0;
      ws = (size_t)pack_elems * 8 + (size_t)a.KP * sizeof(KTabEntry) +
           (a.ksplit > 1 && small < 0 ? (size_t)a.ksplit * (size_t)src.out_elems * 8 : 0);
    };
    corr64(d->fwd, d->fwd_pack, d->fwd64, d->fwd64_pack, x_elems, false, d->fwd64_ws, d->fwd64_rows, d->fwd_small[1], d->fwd_sm[1]);
    corr64(d->bwd, d->bwd_pack, d->bwd64, d->bwd64_pack, y_elems, d->bwd_zero_fill != 0, d->bwd64_ws, d->bwd64_rows, d->bwd_small[1], d->bwd_sm[1]);
    const int32_t bm64 = d->wg64_rows = f64_pick_rows(Kg, true);
    WgradArgs& a = d->wg64;
    a = d->wg;
    a.dy_bytes = (uint32_t)(8 * y_elems);
    a.x_bytes = (uint32_t)(8 * x_elems);
    a.bounds_mode = 1;
    a.m_tiles = (int32_t)ceil_div(Kg, bm64);
    a.n_tiles = (int32_t)ceil_div(kred, bn64);
    const int64_t tiles = G * a.m_tiles * a.n_tiles;
    int64_t S = 1024 / tiles;
    const int64_t max_by_len = ceil_div((int64_t)a.ncols, 4 * bk64);
    const int64_t max_by_ws = ((int64_t)8 << 20) / (w_elems > 0 ? w_elems : 1);
    if (S > max_by_len) S = max_by_len;
    if (S > max_by_ws) S = max_by_ws;
    if (S > 256) S = 256;
    if (S < 1) S = 1;
    a.cols_per_split = (int32_t)round_up(ceil_div((int64_t)a.ncols > 0 ? a.ncols : 1, S), bk64);
    a.S = (int32_t)ceil_div((int64_t)a.ncols > 0 ? a.ncols : 1, a.cols_per_split);
    if (a.S * w_elems >= max64 || tiles * a.S >= ((int64_t)1 << 31)) d->f64_ok = 0;
    d->wg64_ws = (size_t)a.S * (size_t)w_elems * 8;
    d->wg_small[1] = !one_launch ? -1 : configure_wgrad_small(a, N, 8, bm64, bn64, d->wg_sm[1]);
    d->bg64_ws = 2 * d->bg_ws;
    auto corr64_name = [](char* buf, size_t len, int32_t rows, const CorrArgs& c, int32_t zero_fill) {
      snprintf(buf, len, "corr64_%dx64x16[e%c](S=%d,L=%d)", rows, c.simple_epilogue ? 's' : 'p', c.ksplit, 2 + (c.ksplit > 1) + (zero_fill != 0));
    };
    char f[64], b[64], wg[64];
    if (d->fwd_small[1] < 0) corr64_name(f, sizeof(f), d->fwd64_rows, d->fwd64, 0);
    if (d->bwd_small[1] < 0) corr64_name(b, sizeof(b), d->bwd64_rows, d->bwd64, d->bwd_zero_fill);
    if (d->wg_small[1] < 0) snprintf(wg, sizeof(wg), "wgrad64_%dx64x16(S=%d,L=2)", d->wg64_rows, a.S);
    small_names(d, 1, f, b, wg, sizeof(f));
    snprintf(d->names64, sizeof(d->names64), "fwd=%s;bwd_data=%s;bwd_filter=%s;bwd_bias=%s", f, b, wg, bias64);
    d->ws_bytes64 = d->fwd64_ws;
    if (d->bwd64_ws > d->ws_bytes64) d->ws_bytes64 = d->bwd64_ws;
    if (d->wg64_ws > d->ws_bytes64) d->ws_bytes64 = d->wg64_ws;
    if (d->bg64_ws > d->ws_bytes64) d->ws_bytes64 = d->bg64_ws;
  }

  // ---- thin groups: direct kernels instead of the GEMM tiles ----
  {
    const int64_t taps = (int64_t)p.kernel_h * p.kernel_w;
    d->use_direct = G > 1 && taps <= 64 && direct_is_faster(Cg, Kg, p.kernel_h, p.kernel_w);
    DirectArgs& a = d->dir;
    a.bias_part = nullptr;
    a.N = p.n;
    a.C = p.c;
    a.H = p.h;
    a.W = p.w;
    a.K = p.num_output;
    a.OH = (int32_t)OH;
    a.OW = (int32_t)OW;
    a.kh = p.kernel_h;
    a.kw = p.kernel_w;
    a.sh = p.stride_h;
    a.sw = p.stride_w;
    a.ph = p.pad_h;
    a.pw = p.pad_w;
    a.dh = p.dilation_h;
    a.dw = p.dilation_w;
    a.Cg = (int32_t)Cg;
    a.Kg = (int32_t)Kg;
    a.x_elems = (uint32_t)x_elems;
    a.y_elems = (uint32_t)y_elems;
    a.w_elems = (uint32_t)w_elems;
    a.mOW = make_magic((uint32_t)OW);
    a.mOH = make_magic((uint32_t)OH);
    a.mK = make_magic((uint32_t)K);
    a.mKg = make_magic((uint32_t)Kg);
    a.mW = make_magic((uint32_t)W);
    a.mH = make_magic((uint32_t)H);
    a.mC = make_magic((uint32_t)C);
    a.mCg = make_magic((uint32_t)Cg);
    a.mSh = make_magic((uint32_t)p.stride_h);
    a.mSw = make_magic((uint32_t)p.stride_w);
    if (d->use_direct) {
      a.taps = (int32_t)taps;
      a.slots = (int32_t)(64 / taps);
      a.chunks_per_img = (int32_t)ceil_div(OH * OW, a.slots);
      a.mTaps = make_magic((uint32_t)taps);
      a.mKw = make_magic((uint32_t)p.kernel_w);
      a.mChunks = make_magic((uint32_t)a.chunks_per_img);
      // splits over the images: about a thousand workgroups, partial sums of at most 32 MiB
      int64_t S = ceil_div(1024, K * Cg);
      const int64_t max_by_ws = ((int64_t)8 << 20) / (w_elems > 0 ? w_elems : 1);
      if (S > max_by_ws) S = max_by_ws;
      if (S > N) S = N;
      if (S > 256) S = 256;
      if (S < 1) S = 1;
      a.imgs_per_split = (int32_t)ceil_div(N > 0 ? N : 1, S);
      a.S = (int32_t)ceil_div(N > 0 ? N : 1, a.imgs_per_split);
      if ((int64_t)N * a.chunks_per_img >= ((int64_t)1 << 31) || K * Cg >= ((int64_t)1 << 31) ||
          a.S * (w_elems + K) >= kMaxElems)
        d->use_direct = 0;
    }
    if (d->use_direct) {
      d->fwd_ws = d->bwd_ws = 0;
      d->wg_ws = (size_t)a.S * (size_t)w_elems * 4;
      d->wgb_ws = (size_t)a.S * (size_t)(w_elems + K) * 4;  // S x K sums of dy behind the filter partials
      d->fwd64_ws = d->bwd64_ws = 0;
      d->wg64_ws = 2 * d->wg_ws;
      d->ws_bytes64 = d->wg64_ws > d->bg64_ws ? d->wg64_ws : d->bg64_ws;
      char df[3][32];
      for (int pass = 0; pass < 3; ++pass) direct_form_name(pass, a, df[pass], sizeof(df[pass]));
      snprintf(d->names64, sizeof(d->names64),
               "fwd=direct64[%s](S=1,L=1);bwd_data=direct64[%s](S=1,L=1);bwd_filter=direct64[%s](S=%d,L=2);"
               "bwd_bias=%s",
               df[0], df[1], df[2], a.S, bias64);
    }
  }

  d->ws_bytes = d->fwd_ws;
  if (d->bwd_ws > d->ws_bytes) d->ws_bytes = d->bwd_ws;
  if (d->wg_ws > d->ws_bytes) d->ws_bytes = d->wg_ws;
  if (d->bg_ws > d->ws_bytes) d->ws_bytes = d->bg_ws;
  if (p.bias_term && d->wgb_ws > d->ws_bytes) d->ws_bytes = d->wgb_ws;
  {
    // every template parameter and run-time branch that selects different kernel code is spelled out:
    // tile, bounds mode (m0/m1/m2) or patch staging, epilogue form (es/er/ep: separable offsets, range-
    // checked stores with compares, plain pointers), staging of the filter gradient (lds/reg), one or
    // two launches of the bias gradient
    char f[64], b[64], wg[64];
    if (d->fwd_split >= 0)
      split_variant_name(f, sizeof(f), d->fwd_split, d->fwd_sp, 0);
    else if (d->fwd_small[0] < 0)
      corr_variant_name(f, sizeof(f), d->fwd_tile, d->fwd, 0, d->fwd_thin);
    if (d->bwd_split >= 0)
      split_variant_name(b, sizeof(b), d->bwd_split, d->bwd_sp, d->bwd_zero_fill);
    else if (d->bwd_small[0] < 0)
      corr_variant_name(b, sizeof(b), d->bwd_tile, d->bwd, d->bwd_zero_fill, d->bwd_thin);
    if (d->wg_split < 0 && d->wg_fold < 0 && d->wg_small[0] < 0) snprintf(wg, sizeof(wg), "%s[m%d,%s,e%c](S=%d,L=2)", wgrad_tile_name(d->wg_tile), d->wg.bounds_mode,
             d->wg_tile == WGRAD_128x128 ? "lds" : "reg", 4 * Kg * kred <= ((int64_t)1 << 30) ? 'r' : 'p', d->wg.S);
    if (d->wg_fold >= 0) {
      int32_t rows, taps;
      wgrad_fold_shape(d->wg_fold, &rows, &taps);
      snprintf(wg, sizeof(wg), "splitwgrad_fold%d_%dx%dx16[p%d,st%d](S=%d,half,L=2)", d->wg_sp.fold.ff, rows, taps,
               split_patch_units(d->wg_sp.PSZ), d->wg_sp.patch_stages, d->wg_sp.S);
    }
    if (d->wg_split >= 0) {
      int32_t rows, taps;
      wgrad_split_shape(d->wg_split, &rows, &taps);
      const int32_t psz = d->wg_sp.PSZ;
      snprintf(wg, sizeof(wg), "splitwgrad_%dx%dx16[p%d,st%d](S=%d,%sL=2)", rows, taps, split_patch_units(psz),
               d->wg_sp.patch_stages, d->wg_sp.S, d->wg_sp.half ? "half," : "");
    }
    small_names(d, 0, f, b, wg, sizeof(f));
    if (d->use_direct) {
      char df[3][32];
      for (int pass = 0; pass < 3; ++pass) direct_form_name(pass, d->dir, df[pass], sizeof(df[pass]));
      snprintf(f, sizeof(f), "direct[%s](S=1,L=1)", df[0]);
      snprintf(b, sizeof(b), "direct[%s](S=1,L=1)", df[1]);
      snprintf(wg, sizeof(wg), "direct[%s](S=%d,L=2)", df[2], d->dir.S);
    }
    snprintf(d->names, sizeof(d->names), "fwd=%s;bwd_data=%s;bwd_filter=%s;bwd_bias=bias_grad[%s](S=%d,L=%d)", f, b, wg,
             d->bg_direct ? "one" : "two", d->bg.S, d->bg_direct ? 1 : 2);
  }
  *out = d;
  return CONV_OK;
}

int conv_desc_create(conv_desc_t** out, const conv_params_t* pp) { return create_desc(out, pp, true); }

int conv_desc_create_tiled(conv_desc_t** out, const conv_params_t* pp) { return create_desc(out, pp, false); }

int conv_desc_destroy(conv_desc_t* d) {
  if (!d) return CONV_EINVAL;
  delete d;
  return CONV_OK;
}

int conv_desc_output_shape(const conv_desc_t* d, int32_t* n, int32_t* k, int32_t* oh, int32_t* ow) {
  if (!d) return CONV_EINVAL;
  if (n) *n = d->p.n;
  if (k) *k = d->p.num_output;
  if (oh) *oh = d->OH;
  if (ow) *ow = d->OW;
  return CONV_OK;
}

int conv_desc_workspace_bytes(const conv_desc_t* d, size_t* bytes) {
  if (!d || !bytes) return CONV_EINVAL;
  *bytes = d->ws_bytes;
  return CONV_OK;
}

const char* conv_desc_kernel_names(const conv_desc_t* d) { return d ? d->names : ""; }

int conv_forward(const conv_desc_t* d, const float* x, const float* w, const float* bias, float* y, void* ws,
                 size_t ws_bytes, void* hip_stream) {
  return run_forward(d, x, w, bias, y, ws, ws_bytes, hip_stream);
}

int conv_backward_data(const conv_desc_t* d, const float* w, const float* dy, float* dx, void* ws, size_t ws_bytes,
                       void* hip_stream) {
  return run_backward_data(d, w, dy, dx, 0.f, ws, ws_bytes, hip_stream);
}

int conv_backward_filter(const conv_desc_t* d, const float* x, const float* dy, float* dw, float beta, void* ws,
                         size_t ws_bytes, void* hip_stream) {
  return run_backward_filter(d, x, dy, dw, beta, ws, ws_bytes, hip_stream, ReduceExtras());
}

int conv_backward_filter_bias(const conv_desc_t* d, const float* x, const float* dy, float* dw, float* db, float beta,
                              void* ws, size_t ws_bytes, void* hip_stream) {
  if (!d || !db) return CONV_EINVAL;
  if (!d->p.bias_term) return CONV_EINVAL;
  return run_backward_filter(d, x, dy, dw, beta, ws, ws_bytes, hip_stream, ReduceExtras(), db);
}

int conv_backward_bias(const conv_desc_t* d, const float* dy, float* db, float beta, void* ws, size_t ws_bytes,
                       void* hip_stream) {
  if (!d || !db) return CONV_EINVAL;
  if (!d->p.bias_term) return CONV_EINVAL;
  if (!(beta == 0.f || beta == 1.f)) return CONV_EINVAL;
  const bool empty = d->p.n == 0;
  if (!empty && !dy) return CONV_EINVAL;
  if (!empty && (!ws || ws_bytes < d->bg_ws)) return CONV_EWORKSPACE;
  BiasGradArgs a = d->bg;
  a.dy = dy;
  a.part = static_cast<float*>(ws);
  if (!empty && d->bg_direct) {  // small blob: one launch writes db
    a.db = db;
    a.beta = beta;
    const int e1 = launch_bias_grad(a, hip_stream);
    return e1 ? record_hip_error(e1) : CONV_OK;
  }
  int e = empty ? 0 : launch_bias_grad(a, hip_stream);
  if (e) return record_hip_error(e);
  ReduceArgs r = {};
  r.part = a.part;
  r.dst = db;
  r.count = d->p.num_output;
  r.S = empty ? 0 : a.S;
  r.beta = beta;
  e = launch_reduce(r, hip_stream);
  return e ? record_hip_error(e) : CONV_OK;
}

// ---- double base type ----

const char* conv_desc_kernel_names_f64(const conv_desc_t* d) { return d && d->f64_ok ? d->names64 : ""; }

int conv_desc_workspace_bytes_f64(const conv_desc_t* d, size_t* bytes) {
  if (!d || !bytes) return CONV_EINVAL;
  if (!d->f64_ok) return CONV_ESHAPE;
  *bytes = d->ws_bytes64;
  return CONV_OK;
}

static int run_corr64(const conv_desc_t* d, int32_t small, const CorrSmallArgs& small_args, int32_t tile_rows, const CorrArgs& args, const PackArgs& pack, size_t need,
                      const double* w, const double* in, const double* bias, double* out, size_t zero_out_bytes,
                      void* ws, size_t ws_bytes, void* hip_stream) {
  if (!d->f64_ok) return CONV_ESHAPE;
  if (!ws || ws_bytes < need) return CONV_EWORKSPACE;
  if (small >= 0) {
    int es = zero_out_bytes ? launch_fill_zero(out, zero_out_bytes, hip_stream) : 0;
    if (es) return record_hip_error(es);
    CorrSmallArgs sa = small_args;
    sa.A = reinterpret_cast<const float*>(w);
    sa.in = reinterpret_cast<const float*>(in);
    sa.bias = reinterpret_cast<const float*>(bias);
    sa.out = reinterpret_cast<float*>(out);
    es = launch_corr_small(small, sa, true, hip_stream);
    return es ? record_hip_error(es) : CONV_OK;
  }
  PackArgs k = pack;
  const size_t pack_bytes = (size_t)k.G * k.KP * k.MP * 8 + (size_t)k.KP * sizeof(KTabEntry);
  double* const part = reinterpret_cast<double*>(static_cast<char*>(ws) + pack_bytes);
  if (zero_out_bytes) {  // backward data with row / column phases no tap reaches: clear dx, or the slices' partial sums
    const int ez = args.ksplit > 1 ? launch_fill_zero(part, (size_t)args.ksplit * zero_out_bytes, hip_stream)
                                   : launch_fill_zero(out, zero_out_bytes, hip_stream);
    if (ez) return record_hip_error(ez);
  }
  k.w = reinterpret_cast<const float*>(w);
  k.A = static_cast<float*>(ws);
  k.ktab = reinterpret_cast<KTabEntry*>(static_cast<double*>(ws) + (size_t)k.G * k.KP * k.MP);
  int e = launch_pack(k, hip_stream, true);
  if (e) return record_hip_error(e);
  CorrArgs a = args;
  a.A = k.A;
  a.ktab = k.ktab;
  a.in = reinterpret_cast<const float*>(in);
  a.bias = reinterpret_cast<const float*>(bias);
  a.out = reinterpret_cast<float*>(out);
  a.part = reinterpret_cast<float*>(part);
  e = launch_corr64(tile_rows, a, hip_stream);
  if (e) return record_hip_error(e);
  if (a.ksplit > 1) {  // add the slices and the bias
    ReduceArgs r = {};
    r.part = a.part;
    r.dst = a.out;
    r.count = a.out_elems;
    r.S = a.ksplit;
    r.beta = 0.f;
    r.bias = a.bias;
    r.chan_elems = d->OH * d->OW;
    r.channels = d->p.num_output;
    r.mChanElems = make_magic(r.chan_elems);
    r.mChannels = make_magic(r.channels);
    e = launch_reduce64(r, hip_stream);
  }
  return e ? record_hip_error(e) : CONV_OK;
}

int conv_forward_f64(const conv_desc_t* d, const double* x, const double* w, const double* bias, double* y, void* ws,
                     size_t ws_bytes, void* hip_stream) {
  if (!d || !w) return CONV_EINVAL;
  if ((d->p.bias_term != 0) != (bias != nullptr)) return CONV_EINVAL;
  if (d->p.n == 0) return CONV_OK;
  if (!x || !y) return CONV_EINVAL;
  if (d->use_direct && d->f64_ok) {
    DirectArgs da = d->dir;
    da.in = x;
    da.w = w;
    da.bias = bias;
    da.out = y;
    const int ed = launch_direct(0, da, true, hip_stream);
    return ed ? record_hip_error(ed) : CONV_OK;
  }
  return run_corr64(d, d->fwd_small[1], d->fwd_sm[1], d->fwd64_rows, d->fwd64, d->fwd64_pack, d->fwd64_ws, w, x, bias, y, 0, ws, ws_bytes,
                    hip_stream);
}

int conv_backward_data_f64(const conv_desc_t* d, const double* w, const double* dy, double* dx, void* ws,
                           size_t ws_bytes, void* hip_stream) {
  if (!d || !w) return CONV_EINVAL;
  if (d->p.n == 0) return CONV_OK;
  if (!dy || !dx) return CONV_EINVAL;
  if (d->use_direct && d->f64_ok) {
    DirectArgs da = d->dir;
    da.in = dy;
    da.w = w;
    da.out = dx;
    const int ed = launch_direct(1, da, true, hip_stream);
    return ed ? record_hip_error(ed) : CONV_OK;
  }
  const size_t zero = d->bwd_zero_fill ? (size_t)d->bwd64.out_elems * 8 : 0;
  return run_corr64(d, d->bwd_small[1], d->bwd_sm[1], d->bwd64_rows, d->bwd64, d->bwd64_pack, d->bwd64_ws, w, dy, nullptr, dx, zero, ws, ws_bytes,
                    hip_stream);
}

int conv_backward_filter_f64(const conv_desc_t* d, const double* x, const double* dy, double* dw, double beta,
                             void* ws, size_t ws_bytes, void* hip_stream) {
  if (!d || !dw) return CONV_EINVAL;
  if (!(beta == 0.0 || beta == 1.0)) return CONV_EINVAL;
  if (!d->f64_ok) return CONV_ESHAPE;
  const bool empty = d->p.n == 0;
  if (!empty && (!x || !dy)) return CONV_EINVAL;
  if (!empty && (!ws || ws_bytes < d->wg64_ws)) return CONV_EWORKSPACE;
  WgradArgs a = d->wg64;
  a.dy = reinterpret_cast<const float*>(dy);
  a.x = reinterpret_cast<const float*>(x);
  a.part = static_cast<float*>(ws);
  int e = 0;
  if (d->use_direct) {
    DirectArgs da = d->dir;
    da.in = x;
    da.w = dy;
    da.part = ws;
    a.S = da.S;
    if (!empty) e = launch_direct(2, da, true, hip_stream);
  } else if (!empty && d->wg_small[1] >= 0) {
    WgradSmallArgs sa = d->wg_sm[1];
    a.S = sa.S;
    sa.dy = a.dy;
    sa.x = a.x;
    sa.part = a.part;
    sa.dw_out = reinterpret_cast<float*>(dw);
    sa.beta = (float)beta;
    e = launch_wgrad_small(d->wg_small[1], sa, true, hip_stream);
    if (e || sa.S == 1) return e ? record_hip_error(e) : CONV_OK;
  } else if (!empty) {
    e = launch_wgrad64(d->wg64_rows, a, hip_stream);
  }
  if (e) return record_hip_error(e);
  ReduceArgs r = {};
  r.part = a.part;
  r.dst = reinterpret_cast<float*>(dw);
  r.count = (int32_t)((int64_t)d->p.num_output * d->wg64.Kred);
  r.S = empty ? 0 : a.S;
  r.beta = (float)beta;
  e = launch_reduce64(r, hip_stream);
  return e ? record_hip_error(e) : CONV_OK;
}

int conv_backward_bias_f64(const conv_desc_t* d, const double* dy, double* db, double beta, void* ws, size_t ws_bytes,
                           void* hip_stream) {
  if (!d || !db) return CONV_EINVAL;
  if (!d->p.bias_term) return CONV_EINVAL;
  if (!(beta == 0.0 || beta == 1.0)) return CONV_EINVAL;
  if (!d->f64_ok) return CONV_ESHAPE;
  const bool empty = d->p.n == 0;
  if (!empty && !dy) return CONV_EINVAL;
  if (!empty && (!ws || ws_bytes < d->bg64_ws)) return CONV_EWORKSPACE;
  BiasGradArgs a = d->bg;
  a.dy = reinterpret_cast<const float*>(dy);
  a.part = static_cast<float*>(ws);
  if (!empty && d->bg64_direct) {  // one launch writes db
    a.S = 1;
    a.n_per_split = d->p.n;
    a.db = reinterpret_cast<float*>(db);
    a.beta = (float)beta;
    const int e1 = launch_bias_grad64(a, hip_stream);
    return e1 ? record_hip_error(e1) : CONV_OK;
  }
  int e = empty ? 0 : launch_bias_grad64(a, hip_stream);
  if (e) return record_hip_error(e);
  ReduceArgs r = {};
  r.part = a.part;
  r.dst = reinterpret_cast<float*>(db);
  r.count = d->p.num_output;
  r.S = empty ? 0 : a.S;
  r.beta = (float)beta;
  e = launch_reduce64(r, hip_stream);
  return e ? record_hip_error(e) : CONV_OK;
}

const char* conv_status_string(int status) {
  switch (status) {
    case CONV_OK: return "success";
    case CONV_EINVAL: return "invalid argument";
    case CONV_ESHAPE: return "unsupported shape (empty output or a tensor too large for 32-bit offsets)";
    case CONV_EWORKSPACE: return "workspace missing or too small";
    case CONV_EHIP: return "HIP launch failed";
    default: return "unknown status";
  }
}

int conv_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
