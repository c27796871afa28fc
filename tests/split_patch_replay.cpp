// The index arithmetic of corr_split_kernel and wgrad_split_kernel on the host, from a descriptor's own kernel arguments:
// which image position every operand read of a tile finds in its LDS patch.  Same 32-bit unsigned arithmetic as the kernels.
// Counts go to out: [0] reads, [1] reads outside the patch, [2] reads that find another position than the definition's
// (any two positions outside the image are the same zero).
#include "internal.h"

using namespace mi355conv;

namespace {

struct Source {
  uint32_t n;
  int64_t row, col;
  bool zero;  // loaded from beyond the blob
};

bool outside(int64_t ih, int64_t iw, int64_t H, int64_t W) { return ih < 0 || ih >= H || iw < 0 || iw >= W; }

}  // namespace

extern "C" int replay_corr(const conv_desc* d, int backward, int64_t* out) {
  const int32_t tile = backward ? d->bwd_split : d->fwd_split;
  if (tile < 0) return 0;
  const CorrSplitArgs& a = backward ? d->bwd_sp : d->fwd_sp;
  static const int32_t widths[SPLIT_TILE_COUNT] = {128, 256, 128, 128, 256, 128, 256};  // columns, by SplitTile
  const int32_t bn = widths[tile];
  const bool cols = a.fold.subs != 0, fold = a.fold.ff > 1;
  if (a.fold.pixels) return 2;
  out[0] = out[1] = out[2] = 0;
  const uint32_t P = (uint32_t)a.P, PW = (uint32_t)a.PW, PSZ = (uint32_t)a.PSZ;
  const uint32_t ext = (uint32_t)((a.THW / a.TW - 1) * a.dh + 1);
  for (uint32_t col_tile = 0; col_tile < (uint32_t)a.col_tiles; ++col_tile) {
    const uint32_t col0 = col_tile * (uint32_t)bn, n0 = col0 / P, a0 = (col0 - n0 * P) / PW;
    const uint32_t R0 = ((uint32_t)a.PH - 1 - a0) * a.sh + ext - a.share_h, RS = ((uint32_t)a.PH - 1) * a.sh + ext - a.share_h;
    auto patch_row_base = [&](uint32_t n, uint32_t pa) {
      const uint32_t s = n - n0;
      return s == 0 ? (pa - a0) * a.sh : R0 + (s - 1) * RS + pa * a.sh;
    };
    uint32_t col_last = col0 + bn - 1;
    if (col_last > (uint32_t)a.ncols - 1) col_last = (uint32_t)a.ncols - 1;
    uint32_t patch_elems = PSZ;
    if (!cols) patch_elems = (patch_row_base(col_last / P, col_last % P / PW) + ext) * (uint32_t)a.PWID + a.share_w;
    auto source = [&](uint32_t e) {
      Source r = {0, 0, 0, true};
      if (e >= patch_elems) return r;
      const uint32_t prow = e / (uint32_t)a.PWID, pcol = e % (uint32_t)a.PWID;
      uint32_t n = n0, rin = prow, alo = a0;
      int gr, gc = (int)pcol;
      if (cols) {
        const uint32_t col = col0 + pcol;
        n = col > col_last ? (uint32_t)a.Nimg : col / P;
        gr = (int)(col % P / PW);
        gc = (int)(col % P % PW);
      } else {
        if (prow >= R0) {
          const uint32_t s1 = (prow - R0) / RS;
          n = n0 + 1 + s1;
          rin = prow - R0 - s1 * RS;
          alo = 0;
        }
        gr = (int)(alo * a.sh + rin);
      }
      r.n = n;
      r.row = (fold || cols ? gr * a.fold.Uh : gr) - a.ph;
      r.col = (fold || cols ? gc * a.fold.Uw : gc) - a.pw;
      r.zero = n >= (uint32_t)a.Nimg || (!fold && outside(r.row, r.col, a.IH, a.IW));
      return r;
    };
    for (uint32_t col = col0; col <= col_last; ++col) {
      const uint32_t n = col / P, pa = col % P / PW, pb = col % P % PW;
      const uint32_t base = cols ? col - col0 : patch_row_base(n, pa) * (uint32_t)a.PWID + pb * a.sw;
      for (int tap = 0; tap < a.THW; ++tap) {
        const int i = cols ? 0 : tap / a.TW, j = cols ? 0 : tap % a.TW;
        const uint32_t at = base + (cols ? (uint32_t)tap * a.PWID : (uint32_t)(i * a.dh * a.PWID + j * a.dw));
        ++out[0];
        if (at >= PSZ) {
          ++out[1];
          continue;
        }
        const int64_t gr = (int64_t)pa * a.sh + i * a.dh, gc = (int64_t)pb * a.sw + j * a.dw;
        const int64_t ih = (fold || cols ? gr * a.fold.Uh : gr) - a.ph, iw = (fold || cols ? gc * a.fold.Uw : gc) - a.pw;
        const Source s = source(at);
        const bool none = !fold && outside(ih, iw, a.IH, a.IW);
        out[2] += none ? !s.zero : s.zero || s.n != n || s.row != ih || s.col != iw;
      }
    }
  }
  return 1;
}

extern "C" int replay_wgrad(const conv_desc* d, int64_t* out) {
  if (d->wg_split < 0) return 0;
  const WgradSplitArgs& a = d->wg_sp;
  out[0] = out[1] = out[2] = 0;
  const uint32_t kRuns = 16, PW = (uint32_t)a.PW, runs = (uint32_t)a.runs;
  for (uint32_t chunk = 0; chunk < (uint32_t)a.chunks; ++chunk) {
    const uint32_t q0 = chunk * kRuns, n0 = q0 / runs, a0 = (q0 - n0 * runs) * 8u / PW;
    const uint32_t R0 = ((uint32_t)a.PH - 1 - a0) * a.sh + a.ext - a.share_h, RS = ((uint32_t)a.PH - 1) * a.sh + a.ext - a.share_h;
    for (uint32_t q = q0; q < q0 + kRuns && q < (uint32_t)a.N * runs; ++q)
      for (uint32_t e = 0; e < 8; ++e) {
        const uint32_t n = q / runs, p = q % runs * 8u + e;
        if (p >= (uint32_t)a.P) break;
        const uint32_t pa = p / PW, pb = p % PW, s = n - n0;
        const uint32_t base = (s == 0 ? (pa - a0) * a.sh : R0 + (s - 1) * RS + pa * a.sh) * (uint32_t)a.PWID + pb * a.sw;
        for (int tap = 0; tap < a.khw; ++tap) {
          const int i = tap / a.kw, j = tap % a.kw;
          const uint32_t at = base + (uint32_t)(i * a.dh * a.PWID + j * a.dw);
          ++out[0];
          if (at >= (uint32_t)a.PSZ) {
            ++out[1];
            continue;
          }
          const uint32_t prow = at / (uint32_t)a.PWID, pcol = at % (uint32_t)a.PWID;
          uint32_t m = n0, rin = prow, alo = a0;
          if (prow >= R0) {
            const uint32_t s1 = (prow - R0) / RS;
            m = n0 + 1 + s1;
            rin = prow - R0 - s1 * RS;
            alo = 0;
          }
          const int ih = (int)(alo * a.sh + rin) - a.ph, iw = (int)pcol - a.pw;
          const int want_h = (int)pa * a.sh - a.ph + i * a.dh, want_w = (int)pb * a.sw - a.pw + j * a.dw;
          const bool zero = m >= (uint32_t)a.N || outside(ih, iw, a.H, a.W);
          out[2] += outside(want_h, want_w, a.H, a.W) ? !zero : zero || m != n || ih != want_h || iw != want_w;
        }
      }
  }
  return 1;
}
