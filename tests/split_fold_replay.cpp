// The folded form of wgrad_split_kernel reads its patch as the image form does, on the grid of folded positions: an image without
// padding whose size is the grid's.
#include "split_patch_replay.cpp"

extern "C" int replay_fold(conv_desc* d, int64_t* out) {
  if (d->wg_fold < 0) return 0;
  const WgradSplitArgs kept = d->wg_sp;
  const int32_t tile = d->wg_split;
  WgradSplitArgs& a = d->wg_sp;
  a.H = (a.PH - 1) * a.sh + a.ext;
  a.W = (a.PW - 1) * a.sw + (a.kw - 1) * a.dw + 1;
  a.ph = a.pw = 0;
  d->wg_split = 0;
  const int replayed = replay_wgrad(d, out);
  d->wg_sp = kept;
  d->wg_split = tile;
  return replayed;
}
