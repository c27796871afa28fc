// Small layers in one launch per pass: correlation (forward, backward data) and filter gradient for both base types.
//
// A pass of a few hundred MFLOP on the tiled kernels is a chain of launches -- pack, main, reduce -- each of which costs the
// host 2.3 us and the device 2 to 4 us whatever it does.  Here a workgroup owns one small output tile and ALL of its
// reduction: its waves take the groups of 16 reduction indices in turn, feed the matrix unit straight from the blobs (no
// packed copy, no LDS staging, so no barrier inside the loop), and add their sums through LDS in wave order at the end.
// The weights are read where they lie; a ring of three register sets per wave keeps loads in flight.
//
// Bound by latency on the smallest layers: table build, one ring of loads, the wave's chain of matrix instructions, the
// exchange and the stores are 3.5 us, which is what an empty launch takes.  From some 0.1 GFLOP on the single-element gathers
// bind it (four cache accesses per group and column block), at up to 60 % of the matrix unit.  Device time with all launches,
// tiled kernels -> here: 20 -> 50, 5x5 at 12x12, batch 64, forward 14.0 -> 7.0 us, backward data 23.7 -> 19.5; one image of
// 96 -> 256 in two groups, 5x5 at 27x27, forward 22.7 -> 14.8; 12 -> 187, 5x5, stride 2 at 7x7, batch 14: 13.6 -> 4.6, 13.7 ->
// 10.8, filter gradient 14.1 -> 4.7; 84 -> 40, 3x1 at 7x7, batch 71: 10.8 -> 5.3, 15.4 -> 6.0, 10.2 -> 7.7.
#include <hip/hip_runtime.h>

#include "device_utils.h"
#include "internal.h"

namespace mi355conv {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 16x16x4 matrix instruction of either base type: lane l feeds A[l%16][l/16] and B[l/16][l%16]; accumulator register r of
// lane l is row `row(r, l)` of column l%16.
template <typename T>
struct Small;

template <>
struct Small<float> {
  using Acc = f32x4;
  static __device__ __forceinline__ void run(float a, float b, Acc& c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int lane) { return 4 * (lane >> 4) + r; }
  static __device__ __forceinline__ float load(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
    return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rsrc, off, 0, 0));
  }
  static __device__ __forceinline__ void load4(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, float (&v)[4]) {
    const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 0, 0));
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = __builtin_bit_cast(float, (uint32_t)x[e]);
  }
};

template <>
struct Small<double> {
  using Acc = f64x4;
  static __device__ __forceinline__ void run(double a, double b, Acc& c) {
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int lane) { return 4 * r + (lane >> 4); }
  static __device__ __forceinline__ double load(__amdgpu_buffer_rsrc_t rsrc, uint32_t off) {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rsrc, off, 0, 0));
  }
  static __device__ __forceinline__ void load4(__amdgpu_buffer_rsrc_t rsrc, uint32_t off, double (&v)[4]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const u32x4 x = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, off + 16u * h, 0, 0));
#pragma unroll
      for (int e = 0; e < 2; ++e) v[2 * h + e] = __builtin_bit_cast(double, u32x2{x[2 * e], x[2 * e + 1]});
    }
  }
};

constexpr uint32_t kNoTap = 0x7fff0000u;    // a row displacement that fails every bounds test
constexpr uint32_t kOutside = 0x80000000u;  // byte offset beyond any blob of at most 2^30 bytes: reads as zero

// ---------------------------------------------------------------------------------------------------------------------
// D[m][col] = sum_kk A[m][kk] * gather(in)[kk][col] (see CorrArgs), kk = (gathered channel, tap row, tap column).
// WMODE: how the weights are read.  0: rows along kk (forward), 16-byte loads; 1: one load per value through a table of
// offsets (backward data: kk runs over the output channels); 2: the same, and a row phase lacks some taps (stride > 1); 3:
// backward data at unit stride, a channel's taps as 16-byte loads.  With single loads the sixteen rows of the weights, a
// channel's taps apart, are sixteen cache lines in each of four loads: 20 -> 50 channels, 5x5 at 12x12, batch 64, 27.2 against 18.3 us.
// PAD: some place of the gather may lie outside the image.  Its row and column compares are most of the eight vector
// instructions a value takes; without them 1x1 layers take 0.87 of the time (3160 -> 64 at 330 places 24.5 -> 16.2 us).
// One bit per tap and column instead (the tiled kernels' way) was 3 % faster on the mean, 15 % slower where reductions are short.
template <typename T, int MB, int NB, int WAVES, int WMODE, bool PAD>
__global__ __launch_bounds__(64 * WAVES) void corr_small_kernel(const CorrSmallArgs a) {
  using S = Small<T>;
  constexpr int BM = 16 * MB, BN = 16 * NB, kThreads = 64 * WAVES, kRing = 3;
  constexpr int kPitch = BN + 4;  // rows four apart start 16 banks apart
  extern __shared__ __align__(16) uint32_t lds[];
  int4* const rowtab = reinterpret_cast<int4*>(lds);  // as in corr_epilogue: {offset, row shift, column shift, -}
  int4* const coltab = rowtab + BM;
  T* const rowbias = reinterpret_cast<T*>(coltab + BN);
  uint32_t* const tab = reinterpret_cast<uint32_t*>(rowbias + BM);  // per kk; the waves' sums take their place at the end
  T* const red = reinterpret_cast<T*>(tab);
  const int KT = a.KT;
  uint32_t* const tab_off = tab;               // byte offset in the gathered blob
  uint32_t* const tab_rc = tab + KT;           // row displacement << 16 | column displacement
  uint32_t* const tab_w = tab + 2 * KT;        // WMODE > 0: byte offset in the weights
  uint32_t* const tab_tap = tab + 3 * KT;      // WMODE 2: tap of row phase 0, row << 16 | column

  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  uint32_t lin = xcd_contiguous_block_id();
  const uint32_t m_tile = lin % (uint32_t)a.m_tiles;
  lin /= (uint32_t)a.m_tiles;
  const uint32_t col_tile = lin % (uint32_t)a.col_tiles, g = lin / (uint32_t)a.col_tiles;

  for (int kk = t; kk < KT; kk += kThreads) {
    // WMODE 3: taps in the order of the weights, each channel's padded to a multiple of four
    const uint32_t c = mdiv((uint32_t)kk, a.mPitch), r = (uint32_t)kk - c * (uint32_t)a.tap_pitch;
    uint32_t i = mdiv(r, a.mTW), j = r - i * (uint32_t)a.TW;
    bool in = kk < a.Kred;
    if (WMODE == 3) {
      in = r < (uint32_t)a.THW && c < (uint32_t)a.Cg_in;
      i = in ? (uint32_t)a.Qh - 1 - i : 0;
      j = in ? (uint32_t)a.TW - 1 - j : 0;
    }
    tab_off[kk] = (uint32_t)sizeof(T) * (c * (uint32_t)a.IHW + i * (uint32_t)(a.dh * a.IW) + j * (uint32_t)a.dw);
    // past the reduction: an offset beyond any blob with every column's, or a row that fails every bounds test (rows are below
    // 2^14, padding at most 2^12)
    if (!PAD && !in) tab_off[kk] = 0x40000000u;
    if (PAD) tab_rc[kk] = in ? (i * (uint32_t)a.dh) << 16 | j * (uint32_t)a.dw : kNoTap;
    if (WMODE == 3) {
      if ((kk & 3) == 0) tab_w[kk >> 2] = in ? (uint32_t)sizeof(T) * (c * (uint32_t)a.w_chan_stride + r) : kOutside;
    } else if (WMODE > 0) {
      const uint32_t ki = (uint32_t)a.step_h * ((uint32_t)a.Qh - 1 - i), kj = (uint32_t)a.step_w * ((uint32_t)a.TW - 1 - j);
      tab_w[kk] = in ? (uint32_t)sizeof(T) * (c * (uint32_t)a.w_chan_stride + ki * (uint32_t)a.kw + kj) : kOutside;
      if (WMODE == 2) tab_tap[kk] = ki << 16 | kj;
    }
  }
  if (t < BM) {
    const uint32_t gm = m_tile * BM + t;
    int off = 0, hh = -(1 << 28), ww = 0;
    T bb = 0;
    if (gm < (uint32_t)a.Mrows) {
      const uint32_t c = mdiv(gm, a.mRShw), rem = gm - c * a.RShw;
      uint32_t rh = mdiv(rem, a.mRSw), rw = rem - rh * a.RSw;
      if (a.tab_h) rh = (uint32_t)a.phase_h[rh];
      if (a.tab_w) rw = (uint32_t)a.phase_w[rw];
      const uint32_t chan = g * a.chan_per_grp + c;
      hh = (int)rh - a.opad_h;
      ww = (int)rw - a.opad_w;
      off = (int)(chan * (uint32_t)(a.OHd * a.OWd)) + hh * a.OWd + ww;
      if (a.bias) bb = reinterpret_cast<const T*>(a.bias)[chan];
    }
    rowtab[t] = make_int4(off, hh, ww, 0);
    rowbias[t] = bb;
  } else if (t >= 64 && t < 64 + BN) {
    const int cl = t - 64;
    const uint32_t col = col_tile * BN + cl;
    int off = 0, hh = -(1 << 28), ww = 0;
    if (col < (uint32_t)a.ncols) {
      const uint32_t n = mdiv(col, a.mP), pix = col - n * a.P, pa = mdiv(pix, a.mPW), pb = pix - pa * a.PW;
      hh = (int)pa * a.OSh;
      ww = (int)pb * a.OSw;
      off = (int)(n * (uint32_t)a.out_img_stride) + hh * a.OWd + ww;
    }
    coltab[cl] = make_int4(off, hh, ww, 0);
  }

  // this lane's columns of the gather and rows of the weights
  uint32_t cbase[NB], rbase[MB];
  int ih0[NB], iw0[NB], lim_h[MB], lim_w[MB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const uint32_t col = col_tile * BN + j * 16 + (lane & 15);
    cbase[j] = PAD ? 0u : kOutside;
    ih0[j] = -(1 << 29);
    iw0[j] = 0;
    if (col < (uint32_t)a.ncols) {
      const uint32_t n = mdiv(col, a.mP), pix = col - n * a.P, pa = mdiv(pix, a.mPW), pb = pix - pa * a.PW;
      ih0[j] = (int)pa * a.sh - a.ph;
      iw0[j] = (int)pb * a.sw - a.pw;
      cbase[j] = (uint32_t)sizeof(T) * (n * (uint32_t)a.in_img_stride + g * (uint32_t)a.in_grp_stride +
                                        (uint32_t)(ih0[j] * a.IW + iw0[j]));
    }
  }
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const uint32_t gm = m_tile * BM + i * 16 + (lane & 15);
    rbase[i] = kOutside;
    lim_h[i] = lim_w[i] = 0;
    if (gm < (uint32_t)a.Mrows) {
      uint32_t c = gm, rh = 0, rw = 0;
      if (WMODE == 2) {
        c = mdiv(gm, a.mRShw);
        const uint32_t rem = gm - c * a.RShw;
        rh = mdiv(rem, a.mRSw);
        rw = rem - rh * a.RSw;
        if (a.tab_h) rh = (uint32_t)a.phase_h[rh];
        if (a.tab_w) rw = (uint32_t)a.phase_w[rw];
        lim_h[i] = a.kh - (int)rh;
        lim_w[i] = a.kw - (int)rw;
      }
      rbase[i] = (uint32_t)sizeof(T) * (g * (uint32_t)a.w_grp_stride + c * (uint32_t)a.w_row_stride + rh * (uint32_t)a.kw + rw);
    }
  }
  const __amdgpu_buffer_rsrc_t in_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.in), 0, (int)a.in_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t w_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.A), 0, (int)a.w_bytes, 0x00020000);

  // Running sums of floats in kSums parts, added up at the end: the tiled kernels' slices kept their sums as short, and
  // the instructions of a one-block tile do not wait for each other.
  constexpr int kSums = sizeof(T) == 8 ? 1 : MB * NB > 4 ? 2 : 4;
  typename S::Acc acc[kSums][MB][NB];
#pragma unroll
  for (int q = 0; q < kSums; ++q)
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NB; ++j) acc[q][i][j] = typename S::Acc{0, 0, 0, 0};
  __syncthreads();

  const int groups = KT / 16, mine = (groups - wv + WAVES - 1) / WAVES;
  T av[kRing][MB][4], bv[kRing][NB][4];
  int next = wv;  // the group loaded next; past the last one that one again, never multiplied
  auto load = [&](T(&A)[MB][4], T(&B)[NB][4]) {
    const int kk = next * 16 + 4 * (lane >> 4);
    const u32x4 off = *reinterpret_cast<const u32x4*>(tab_off + kk);
    u32x4 rc;
    if (PAD) rc = *reinterpret_cast<const u32x4*>(tab_rc + kk);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!PAD) {
          B[j][e] = S::load(in_rsrc, cbase[j] + off[e]);
          continue;
        }
        const int ih = ih0[j] + (int)(rc[e] >> 16), iw = iw0[j] + (int)(rc[e] & 0xffffu);
        const bool ok = ((uint32_t)ih < (uint32_t)a.IH) & ((uint32_t)iw < (uint32_t)a.IW);
        B[j][e] = S::load(in_rsrc, ok ? cbase[j] + off[e] : kOutside);
      }
    if (WMODE == 0) {
      if (next * 16 + 16 <= a.Kred) {
#pragma unroll
        for (int i = 0; i < MB; ++i) S::load4(w_rsrc, rbase[i] + (uint32_t)sizeof(T) * (uint32_t)kk, A[i]);
      } else {  // the last group: what lies behind a row is the next one
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            A[i][e] = S::load(w_rsrc, kk + e < a.Kred ? rbase[i] + (uint32_t)sizeof(T) * (uint32_t)(kk + e) : kOutside);
      }
    } else if (WMODE == 3) {
      const uint32_t wo = tab_w[kk >> 2];
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        S::load4(w_rsrc, rbase[i] + wo, A[i]);
#pragma unroll
        for (int e = 1; e < 4; ++e) A[i][e] = rc[e] == kNoTap ? (T)0 : A[i][e];  // behind a channel's taps lies the next row
      }
    } else {
      const u32x4 wo = *reinterpret_cast<const u32x4*>(tab_w + kk);
      u32x4 tp;
      if (WMODE == 2) tp = *reinterpret_cast<const u32x4*>(tab_tap + kk);
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bool ok = true;
          if (WMODE == 2) ok = ((int)(tp[e] >> 16) < lim_h[i]) & ((int)(tp[e] & 0xffffu) < lim_w[i]);
          A[i][e] = S::load(w_rsrc, ok ? rbase[i] + wo[e] : kOutside);
        }
    }
    if (next + WAVES < groups) next += WAVES;
  };
  auto multiply = [&](const T(&A)[MB][4], const T(&B)[NB][4]) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) S::run(A[i][e], B[j][e], acc[e % kSums][i][j]);
  };
  if (mine > 0) {
#pragma unroll
    for (int b = 0; b < kRing; ++b) load(av[b], bv[b]);
    int i = 0;
    for (; i + kRing <= mine; i += kRing)
#pragma unroll
      for (int b = 0; b < kRing; ++b) {
        multiply(av[b], bv[b]);
        load(av[b], bv[b]);
      }
#pragma unroll
    for (int b = 0; b < kRing - 1; ++b)
      if (i + b < mine) multiply(av[b], bv[b]);
  }

  __syncthreads();  // every wave has read the tables
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        T s = acc[0][i][j][r];
        if (kSums == 2) s += acc[1 % kSums][i][j][r];
        if (kSums == 4) s = (s + acc[1 % kSums][i][j][r]) + (acc[2 % kSums][i][j][r] + acc[3 % kSums][i][j][r]);
        red[(wv * BM + i * 16 + S::row(r, lane)) * kPitch + j * 16 + (lane & 15)] = s;
      }
  __syncthreads();
  T* const out = reinterpret_cast<T*>(a.out);
#pragma unroll
  for (int idx = t; idx < BM * BN; idx += kThreads) {
    const int row = idx / BN, cl = idx % BN;
    T s = red[row * kPitch + cl];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += red[(w * BM + row) * kPitch + cl];
    const int4 rt = rowtab[row], ct = coltab[cl];
    if ((uint32_t)(rt.y + ct.y) < (uint32_t)a.OHd && (uint32_t)(rt.z + ct.z) < (uint32_t)a.OWd) {
      T* const dst = out + (rt.x + ct.x);
      s += rowbias[row];
      *dst = a.accumulate ? *dst + s : s;
    }
  }
}

template <typename T, int MB, int NB, int WAVES, int WMODE, bool PAD>
int launch_corr_small_b(const CorrSmallArgs& a, hipStream_t s) {
  constexpr size_t fixed = 16 * (16 * MB + 16 * NB) + 16 * MB * sizeof(T);
  constexpr size_t red = (size_t)WAVES * 16 * MB * (16 * NB + 4) * sizeof(T);
  static_assert(fixed + red <= 64 * 1024, "LDS without an opt-in");
  const size_t tab = (size_t)a.KT * (WMODE == 3 ? 9 : 4 * (2 + WMODE));
  hipLaunchKernelGGL((corr_small_kernel<T, MB, NB, WAVES, WMODE, PAD>), dim3((uint32_t)(a.G * a.m_tiles * a.col_tiles)),
                     dim3(64 * WAVES), fixed + (tab > red ? tab : red), s, a);
  return (int)hipGetLastError();
}

template <typename T, int MB, int NB, int WAVES, int WMODE>
int launch_corr_small_m(const CorrSmallArgs& a, hipStream_t s) {
  if constexpr (WMODE <= 1)  // backward data of more than one tap always reaches outside
    if (!a.pad) return launch_corr_small_b<T, MB, NB, WAVES, WMODE, false>(a, s);
  return launch_corr_small_b<T, MB, NB, WAVES, WMODE, true>(a, s);
}

template <typename T, int MB, int NB, int WAVES>
int launch_corr_small_t(const CorrSmallArgs& a, hipStream_t s) {
  switch (a.wmode) {
    case 0: return launch_corr_small_m<T, MB, NB, WAVES, 0>(a, s);
    case 1: return launch_corr_small_m<T, MB, NB, WAVES, 1>(a, s);
    case 2: return launch_corr_small_m<T, MB, NB, WAVES, 2>(a, s);
    default: return launch_corr_small_m<T, MB, NB, WAVES, 3>(a, s);
  }
}

// ---------------------------------------------------------------------------------------------------------------------
// part[s][g][k][nn] = sum over (image, pixel) of dy[n, g*Kg + k, p] * x[n, g*Cg + c, window of p at tap (i, j)], nn =
// (c, i, j) (see WgradArgs).  The reduction runs in blocks of 64 places: sixteen runs of four pixels of one image, the last
// run of an image padded.  A wave writes the places' offsets to LDS for itself (lane = place), so they are worked out once
// and not once per row or column.  With one slice the workgroup finishes dw (and db) itself.
// XV 1: 1x1 kernels at unit stride without padding -- four places are one 16-byte load of x as well.  2 (floats): unit column
// stride -- the runs are cut at the ends of the output's rows, so that they are: 374 -> 35, 3x3 at 74x74, two images, 103 -> 51
// us; 1.18 times as fast as 0 in the geometric mean of the gradients over 8 us, slower where rows end in short runs.
// PAD: some tap may lie outside the image; else the places' and columns' offsets alone tell what reads as zero (5 to 15 %).
template <typename T, int MB, int NB, int WAVES, int XV, bool PAD>
__global__ __launch_bounds__(64 * WAVES) void wgrad_small_kernel(const WgradSmallArgs a) {
  using S = Small<T>;
  constexpr int BM = 16 * MB, BN = 16 * NB, kThreads = 64 * WAVES;
  constexpr int kPitch = BN + 4;
  constexpr bool XVEC = XV == 1;
  extern __shared__ __align__(16) uint32_t lds[];
  const int t = threadIdx.x, lane = t & 63;
  const int wv = __builtin_amdgcn_readfirstlane(t >> 6);
  // the wave's places, two blocks: offset in x, row << 16 | column (signed) of the window, offset in dy
  uint32_t* const places = lds + wv * (2 * 3 * 64);
  T* const red = reinterpret_cast<T*>(lds);  // at the end

  uint32_t lin = xcd_contiguous_block_id();
  const uint32_t n_tile = lin % (uint32_t)a.n_tiles;
  lin /= (uint32_t)a.n_tiles;
  const uint32_t m_tile = lin % (uint32_t)a.m_tiles;
  lin /= (uint32_t)a.m_tiles;
  const uint32_t g = lin % (uint32_t)a.G, split = lin / (uint32_t)a.G;
  const int b0 = (int)split * a.blocks_per_split;
  int b1 = b0 + a.blocks_per_split;
  if (b1 > a.blocks) b1 = a.blocks;

  uint32_t rbase[MB], cbase[NB];
  int idh[NB], jdw[NB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    const uint32_t m = m_tile * BM + i * 16 + (lane & 15);
    rbase[i] = m < (uint32_t)a.Kg ? (uint32_t)sizeof(T) * m * (uint32_t)a.P : 0x40000000u;
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const uint32_t col = n_tile * BN + j * 16 + (lane & 15);
    cbase[j] = 0;
    idh[j] = 1 << 20;  // past the last column: fails every bounds test
    jdw[j] = 0;
    if (col < (uint32_t)a.Kred) {
      const uint32_t c = mdiv(col, a.mKHW), r = col - c * (uint32_t)a.khw, i = mdiv(r, a.mKW), jj = r - i * (uint32_t)a.kw;
      idh[j] = (int)i * a.dh;
      jdw[j] = (int)jj * a.dw;
      cbase[j] = (uint32_t)sizeof(T) * (c * (uint32_t)a.HW + (uint32_t)(idh[j] * a.W + jdw[j]));
    } else if (XVEC || !PAD) {
      cbase[j] = 0x40000000u;
    }
  }
  const __amdgpu_buffer_rsrc_t dy_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.dy), 0, (int)a.dy_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t x_rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.x), 0, (int)a.x_bytes, 0x00020000);

  constexpr int kSums = sizeof(T) == 8 ? 1 : 4 / (MB * NB);  // running sums of floats in parts, as in corr_small_kernel
  typename S::Acc acc[kSums][MB][NB];
  T rowsum[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    rowsum[i] = 0;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int q = 0; q < kSums; ++q) acc[q][i][j] = typename S::Acc{0, 0, 0, 0};
  }
  const bool ragged = ((XV == 2 ? a.PW : a.P) & 3) != 0;
  constexpr uint32_t kNoPlace = 0x80000000u;  // row -32768: no tap reaches the image
  auto fill = [&](int block, int buf) {
    const uint32_t run = (uint32_t)block * 16 + (uint32_t)(lane >> 2);
    const uint32_t n = mdiv(run, a.mRuns), in_image = run - n * (uint32_t)a.runs;
    uint32_t p = in_image * 4 + (uint32_t)(lane & 3), pa = mdiv(p, a.mPW), pb = p - pa * (uint32_t)a.PW;
    bool in = block < b1 && n < (uint32_t)a.N && p < (uint32_t)a.P;
    if (XV == 2) {
      pa = mdiv(in_image, a.mRowRuns);
      pb = (in_image - pa * (uint32_t)a.row_runs) * 4 + (uint32_t)(lane & 3);
      p = pa * (uint32_t)a.PW + pb;
      in = block < b1 && n < (uint32_t)a.N && pb < (uint32_t)a.PW;
    }
    const int ih = (int)pa * a.sh - a.ph, iw = (int)pb * a.sw - a.pw;
    uint32_t* const dst = places + buf * (3 * 64) + lane;
    dst[0] = in ? (uint32_t)sizeof(T) * ((n * (uint32_t)a.C + g * (uint32_t)a.Cg) * (uint32_t)a.HW + (uint32_t)(ih * a.W + iw)) : kOutside;
    dst[64] = in ? (uint32_t)ih << 16 | ((uint32_t)iw & 0xffffu) : kNoPlace;
    dst[128] = in ? (uint32_t)sizeof(T) * ((n * (uint32_t)a.Ktot + g * (uint32_t)a.Kg) * (uint32_t)a.P + p) : kOutside;
  };
  T av[4][MB][4], bv[4][NB][4];
  auto load = [&](int buf, int gi, T(&A)[MB][4], T(&B)[NB][4]) {
    const uint32_t* const src = places + buf * (3 * 64) + gi * 16 + 4 * (lane >> 4);
    const u32x4 xo = *reinterpret_cast<const u32x4*>(src), rc = *reinterpret_cast<const u32x4*>(src + 64);
    const uint32_t dyo = src[128];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      S::load4(dy_rsrc, dyo + rbase[i], A[i]);
      if (ragged)  // the places behind an image's last pixel hold the next row's
#pragma unroll
        for (int e = 1; e < 4; ++e) A[i][e] = rc[e] == kNoPlace ? (T)0 : A[i][e];
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      if (XVEC) {
        S::load4(x_rsrc, xo[0] + cbase[j], B[j]);
        if (ragged)
#pragma unroll
          for (int e = 1; e < 4; ++e) B[j][e] = rc[e] == kNoPlace ? (T)0 : B[j][e];
      } else if (XV == 2) {
        const int ih = ((int)rc[0] >> 16) + idh[j], iw = (int)(int16_t)(rc[0] & 0xffffu) + jdw[j];
        const bool row = !PAD || (uint32_t)ih < (uint32_t)a.H;
        const uint32_t at = xo[0] + cbase[j];
        if (PAD && __any(row && (int)at < 0)) {  // left of the blob's first pixel: the address must not wrap
#pragma unroll
          for (int e = 0; e < 4; ++e) B[j][e] = S::load(x_rsrc, row && iw + e >= 0 ? at + (uint32_t)sizeof(T) * e : kOutside);
        } else {
          S::load4(x_rsrc, row ? at : kOutside, B[j]);
        }
        if (PAD || ragged)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            B[j][e] = (!PAD || (uint32_t)(iw + e) < (uint32_t)a.W) && rc[e] != kNoPlace ? B[j][e] : (T)0;
      } else if (!PAD) {
#pragma unroll
        for (int e = 0; e < 4; ++e) B[j][e] = S::load(x_rsrc, xo[e] + cbase[j]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int ih = ((int)rc[e] >> 16) + idh[j], iw = (int)(int16_t)(rc[e] & 0xffffu) + jdw[j];
          const bool ok = ((uint32_t)ih < (uint32_t)a.H) & ((uint32_t)iw < (uint32_t)a.W);
          B[j][e] = S::load(x_rsrc, ok ? xo[e] + cbase[j] : kOutside);
        }
      }
    }
  };
  const bool sum_rows = a.bias_part != nullptr && n_tile == 0;
  int b = b0 + wv;
  if (b < b1) {
    fill(b, 0);
    wave_sync();  // a lane reads what others wrote
#pragma unroll
    for (int gi = 0; gi < 4; ++gi) load(0, gi, av[gi], bv[gi]);
    int buf = 1;
    for (; b < b1; b += WAVES, buf ^= 1) {
      fill(b + WAVES, buf);  // past the last block: nothing is read from the blobs
      wave_sync();  // a lane reads what others wrote
#pragma unroll
      for (int gi = 0; gi < 4; ++gi) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j) S::run(av[gi][i][e], bv[gi][j][e], acc[e % kSums][i][j]);
        if (sum_rows)
#pragma unroll
          for (int i = 0; i < MB; ++i) rowsum[i] += (av[gi][i][0] + av[gi][i][1]) + (av[gi][i][2] + av[gi][i][3]);
        load(buf, gi, av[gi], bv[gi]);
      }
    }
  }

  __syncthreads();
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        T s = acc[0][i][j][r];
        if (kSums == 2) s += acc[1 % kSums][i][j][r];
        if (kSums == 4) s = (s + acc[1 % kSums][i][j][r]) + (acc[2 % kSums][i][j][r] + acc[3 % kSums][i][j][r]);
        red[(wv * BM + i * 16 + S::row(r, lane)) * kPitch + j * 16 + (lane & 15)] = s;
      }
  T* const sums = red + WAVES * BM * kPitch;  // [wave][quarter][row]
  if (sum_rows)
#pragma unroll
    for (int i = 0; i < MB; ++i) sums[(wv * 4 + (lane >> 4)) * BM + i * 16 + (lane & 15)] = rowsum[i];
  __syncthreads();
  const bool whole = a.S == 1;
  T* const dst = whole ? reinterpret_cast<T*>(a.dw_out) : reinterpret_cast<T*>(a.part) + (size_t)split * a.part_stride;
#pragma unroll
  for (int idx = t; idx < BM * BN; idx += kThreads) {
    const int row = idx / BN, cl = idx % BN;
    T s = red[row * kPitch + cl];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) s += red[(w * BM + row) * kPitch + cl];
    const uint32_t m = m_tile * BM + row, col = n_tile * BN + cl;
    if (m < (uint32_t)a.Kg && col < (uint32_t)a.Kred) {
      T* const to = dst + (size_t)(g * (uint32_t)a.Kg + m) * (uint32_t)a.Kred + col;
      if (whole) {
        if (a.col_bias) s += reinterpret_cast<const T*>(a.col_bias)[col];
        if (a.beta != 0.f) s += *to;
        if (a.relu) s = s > 0 ? s : 0;
      }
      *to = s;
    }
  }
  if (sum_rows && t < BM) {
    T s = 0;
#pragma unroll
    for (int w = 0; w < 4 * WAVES; ++w) s += sums[w * BM + t];
    const uint32_t m = m_tile * BM + t;
    if (m < (uint32_t)a.Kg) {
      T* const to = reinterpret_cast<T*>(a.bias_part) + (whole ? 0 : (size_t)split * a.Ktot) + g * (uint32_t)a.Kg + m;
      if (whole && a.beta != 0.f) s += *to;
      *to = s;
    }
  }
}

template <typename T, int MB, int NB, int WAVES>
int launch_wgrad_small_t(const WgradSmallArgs& a, hipStream_t s) {
  constexpr size_t places = (size_t)WAVES * 2 * 3 * 64 * 4;
  constexpr size_t red = ((size_t)WAVES * 16 * MB * (16 * NB + 4) + (size_t)WAVES * 4 * 16 * MB) * sizeof(T);
  constexpr size_t lds = places > red ? places : red;
  static_assert(lds <= 64 * 1024, "LDS without an opt-in");
  const dim3 grid((uint32_t)a.S * a.G * a.m_tiles * a.n_tiles);
  if constexpr (sizeof(T) == 4)
    if (a.xvec == 2) {
      if (a.pad)
        hipLaunchKernelGGL((wgrad_small_kernel<T, MB, NB, WAVES, 2, true>), grid, dim3(64 * WAVES), lds, s, a);
      else
        hipLaunchKernelGGL((wgrad_small_kernel<T, MB, NB, WAVES, 2, false>), grid, dim3(64 * WAVES), lds, s, a);
      return (int)hipGetLastError();
    }
  if (a.xvec == 1)
    hipLaunchKernelGGL((wgrad_small_kernel<T, MB, NB, WAVES, 1, false>), grid, dim3(64 * WAVES), lds, s, a);
  else if (a.pad)
    hipLaunchKernelGGL((wgrad_small_kernel<T, MB, NB, WAVES, 0, true>), grid, dim3(64 * WAVES), lds, s, a);
  else
    hipLaunchKernelGGL((wgrad_small_kernel<T, MB, NB, WAVES, 0, false>), grid, dim3(64 * WAVES), lds, s, a);
  return (int)hipGetLastError();
}

}  // namespace

const SmallTile kCorrSmallTiles[CORR_SMALL_COUNT] = {{1, 1, 4}, {1, 1, 8}, {2, 1, 4}, {1, 2, 4}, {2, 2, 4}, {3, 1, 4}, {3, 2, 4}};
const SmallTile kWgradSmallTiles[WGRAD_SMALL_COUNT] = {{1, 1, 8}, {1, 2, 8}, {2, 1, 8}, {2, 2, 8}, {2, 2, 4}};

int launch_corr_small(int32_t tile, const CorrSmallArgs& a, bool f64, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (tile + (f64 ? CORR_SMALL_COUNT : 0)) {
    case 0: return launch_corr_small_t<float, 1, 1, 4>(a, s);
    case 1: return launch_corr_small_t<float, 1, 1, 8>(a, s);
    case 2: return launch_corr_small_t<float, 2, 1, 4>(a, s);
    case 3: return launch_corr_small_t<float, 1, 2, 4>(a, s);
    case 4: return launch_corr_small_t<float, 2, 2, 4>(a, s);
    case 5: return launch_corr_small_t<float, 3, 1, 4>(a, s);
    case 6: return launch_corr_small_t<float, 3, 2, 4>(a, s);
    case CORR_SMALL_COUNT + 0: return launch_corr_small_t<double, 1, 1, 4>(a, s);
    case CORR_SMALL_COUNT + 1: return launch_corr_small_t<double, 1, 1, 8>(a, s);
    case CORR_SMALL_COUNT + 2: return launch_corr_small_t<double, 2, 1, 4>(a, s);
    case CORR_SMALL_COUNT + 3: return launch_corr_small_t<double, 1, 2, 4>(a, s);
    case CORR_SMALL_COUNT + 4: return launch_corr_small_t<double, 2, 2, 4>(a, s);
    case CORR_SMALL_COUNT + 5: return launch_corr_small_t<double, 3, 1, 4>(a, s);
    default: return (int)hipErrorInvalidValue;
  }
}

int launch_wgrad_small(int32_t tile, const WgradSmallArgs& a, bool f64, void* stream) {
  hipStream_t s = (hipStream_t)stream;
  switch (tile + (f64 ? WGRAD_SMALL_COUNT : 0)) {
    case 0: return launch_wgrad_small_t<float, 1, 1, 8>(a, s);
    case 1: return launch_wgrad_small_t<float, 1, 2, 8>(a, s);
    case 2: return launch_wgrad_small_t<float, 2, 1, 8>(a, s);
    case 3: return launch_wgrad_small_t<float, 2, 2, 8>(a, s);
    case 4: return launch_wgrad_small_t<float, 2, 2, 4>(a, s);
    case WGRAD_SMALL_COUNT + 0: return launch_wgrad_small_t<double, 1, 1, 8>(a, s);
    case WGRAD_SMALL_COUNT + 1: return launch_wgrad_small_t<double, 1, 2, 8>(a, s);
    case WGRAD_SMALL_COUNT + 2: return launch_wgrad_small_t<double, 2, 1, 8>(a, s);
    case WGRAD_SMALL_COUNT + 4: return launch_wgrad_small_t<double, 2, 2, 4>(a, s);
    default: return (int)hipErrorInvalidValue;
  }
}

}  // namespace mi355conv
