// Policy-gradient loss arithmetic of the paper's reinforcement-learning trainer (Appendix A:
// Sigmoid model, Appendix B: Softmax model): action sampling, discounted rewards (a reverse
// recurrence per episode), Dlogps and the modulated Bottom.diff.  All of it is element-wise or a
// short scan: one read and one write per value, HBM-bound.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "device_utils.h"
#include "internal.h"
#include "mi355pg.h"

namespace mi355conv {

namespace {

// Where a model's passes touch more than the last-level cache holds, what a pass reads or writes and no other of them reads again goes
// around it, so that the sampled actions and discounted rewards are still there for the passes that read them.  A step is seven words of
// the Sigmoid model's, three rows and three words of the Softmax model's.  Measured (us, all through the cache -> around it): Sigmoid
// passes, 6 M steps (168 MB) 40.8 -> 41.2, 8 M 52.5 -> 53.5, 10 M 67.6 -> 65.4, 16 M 114.8 -> 101.7; Softmax pass with the discounted
// rewards, 6 actions, 2 M steps (168 MB) 32.8 -> 37.1, 4 M (336 MB) 69.0 -> 64.4, 8 M 131 -> 116, and with a following kernel that
// reads bottom_diff 47.4 -> 53.0, 93.7 -> 93.3, 199 -> 188; 12 actions, 8 M 239 -> 210.  From about 14 actions on what stays in the cache
// is too little beside the rows (14 actions, 8 M steps 275 -> 273; 18, 351 -> 359; 24, 488 -> 506).
constexpr size_t kCacheBytes = (size_t)256 << 20;
constexpr int kStreamActions = 14;

// A template argument: of a branch between both forms the compiler makes one plain access.
template <bool STREAM>
__device__ __forceinline__ void store4(float* to, float4 v) {
  typedef float V __attribute__((ext_vector_type(4)));
  const V u = {v.x, v.y, v.z, v.w};
  if constexpr (STREAM)
    __builtin_nontemporal_store(u, reinterpret_cast<V*>(to));
  else
    *reinterpret_cast<V*>(to) = u;
}

template <bool STREAM>
__device__ __forceinline__ float4 load4(const float* from) {
  typedef float V __attribute__((ext_vector_type(4)));
  const V* const at = reinterpret_cast<const V*>(from);
  V u;
  if constexpr (STREAM)
    u = __builtin_nontemporal_load(at);
  else
    u = *at;
  return make_float4(u[0], u[1], u[2], u[3]);
}

// ---- step 3: action = (random < Aprob) ? 0 : 1 ----
// Four consecutive steps per thread (16-byte loads and stores); the last, partial group of a
// launch goes element by element.
template <bool STREAM>
__global__ __launch_bounds__(256) void pg_sample_kernel(const float* __restrict__ aprob,
                                                        const float* __restrict__ random, int32_t* __restrict__ action,
                                                        int steps) {
  const int t = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (t + 3 < steps) {
    const float4 ap = *reinterpret_cast<const float4*>(aprob + t);
    const float4 rn = load4<STREAM>(random + t);
    *reinterpret_cast<int4*>(action + t) =
        make_int4(rn.x < ap.x ? 0 : 1, rn.y < ap.y ? 0 : 1, rn.z < ap.z ? 0 : 1, rn.w < ap.w ? 0 : 1);
  } else {
    for (int i = t; i < steps; ++i) action[i] = random[i] < aprob[i] ? 0 : 1;
  }
}

// ---- step 9: R[t] = reward[t] + gamma * R[t+1] inside each episode ----
// One wave per episode at a time, walking it from its end in chunks of 256 steps: lane l holds the
// four consecutive steps 4l .. 4l+3 of the chunk (one 16-byte access on a 4-byte boundary; lanes at
// the edges of the episode go element by element).  A lane first runs the recurrence over its own
// four steps; the lane totals then form the same recurrence with gamma^4 per lane, a weighted
// suffix sum: four DPP row shifts with the weights (gamma^4)^1, ^2, ^4, ^8 finish each row of 16
// lanes, three lane reads chain the rows, and the value carried in from the later chunk is added
// with the weight (gamma^4)^(64 - lane).  Each step's result is its in-lane partial plus
// gamma^(4-j) times the total of the next lane.  The scans of the chunks that are loaded together
// are independent; only the carry links them.  A wave walks several episodes with the next one's
// loads already in flight.
constexpr int kChunksInFlight = 2;
constexpr int kChunkSteps = 256;

struct Quad {
  float v[4];
};
struct __attribute__((packed, aligned(4))) QuadMem {
  float v[4];
};

// Lane l receives the value of lane l + N of its row of 16 lanes, 0 past the row's end.
template <int N>
__device__ __forceinline__ float row_shift_down(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x100 + N, 0xF, 0xF, true));
}

struct ScanWeights {
  float g1, g2, g4, g8, g16;  // powers of the per-lane factor
  float to_row_end;           // factor^(16 - lane % 16): from this lane to the first lane of the next row
  float to_chunk_end;         // factor^(64 - lane): from this lane to the first lane of the later chunk
};

__device__ __forceinline__ ScanWeights scan_weights(float factor, int lane) {
  ScanWeights w;
  w.g1 = factor;
  w.g2 = w.g1 * w.g1;
  w.g4 = w.g2 * w.g2;
  w.g8 = w.g4 * w.g4;
  w.g16 = w.g8 * w.g8;
  const int li = lane & 15;
  float p = 1.f;
  p *= (16 - li) & 1 ? w.g1 : 1.f;
  p *= (16 - li) & 2 ? w.g2 : 1.f;
  p *= (16 - li) & 4 ? w.g4 : 1.f;
  p *= (16 - li) & 8 ? w.g8 : 1.f;
  p *= (16 - li) & 16 ? w.g16 : 1.f;
  w.to_row_end = p;
  const int rows_after = 3 - (lane >> 4);
  float q = p;
  q *= rows_after & 1 ? w.g16 : 1.f;
  q *= rows_after & 2 ? w.g16 * w.g16 : 1.f;
  w.to_chunk_end = q;
  return w;
}

// v[l] <- sum over the lanes m >= l of the wave of factor^(m - l) * v[m]; t16/t32/t48 return the
// finished values of lanes 16, 32, 48 (the row heads) without the carry of a later chunk.
__device__ __forceinline__ float suffix_scan(float v, int lane, const ScanWeights& w, float& t1, float& t2, float& t3) {
  v += w.g1 * row_shift_down<1>(v);
  v += w.g2 * row_shift_down<2>(v);
  v += w.g4 * row_shift_down<4>(v);
  v += w.g8 * row_shift_down<8>(v);
  const int iv = __builtin_bit_cast(int, v);
  t3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 48));
  t2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 32)) + w.g16 * t3;
  t1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16)) + w.g16 * t2;
  const int row = lane >> 4;
  const float later_rows = row == 0 ? t1 : row == 1 ? t2 : row == 2 ? t3 : 0.f;
  return v + w.to_row_end * later_rows;
}

__global__ __launch_bounds__(256) void pg_discount_kernel(const float* __restrict__ reward,
                                                          const int32_t* __restrict__ offsets, int episodes,
                                                          int steps, float gamma, float* __restrict__ discounted) {
  const int lane = threadIdx.x & 63;
  const int stride = (int)gridDim.x * 4;  // waves in the grid: a wave takes episodes e, e + stride, ...
  int e = (int)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (e >= episodes) return;
  const float g2 = gamma * gamma, g3 = g2 * gamma, g4 = g2 * g2;
  const ScanWeights w = scan_weights(g4, lane);
  const int row = lane >> 4;

  auto bounds = [&](int ep, int& b, int& end) {  // clamped to [0, steps]; empty for ep >= episodes
    b = end = 0;
    if (ep < episodes) {
      b = offsets[ep];
      end = offsets[ep + 1];
      b = b < 0 ? 0 : (b > steps ? steps : b);
      end = end < b ? b : (end > steps ? steps : end);
    }
  };
  auto fetch = [&](Quad(&r)[kChunksInFlight], int b, int hi, int end) {  // the chunks below hi
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) {
      const int t = hi - kChunkSteps * (c + 1) + 4 * lane;
      if (t >= b && t + 3 < end) {
        const QuadMem m = *reinterpret_cast<const QuadMem*>(reward + t);
#pragma unroll
        for (int j = 0; j < 4; ++j) r[c].v[j] = m.v[j];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[c].v[j] = (t + j >= b && t + j < end) ? reward[t + j] : 0.f;
      }
    }
  };

  // The rewards of the wave's next episode (its last chunks) and the bounds of the one after that
  // are requested before the current episode is scanned, so that their memory latency overlaps
  // the scan.
  int b, end, nb, nend;
  bounds(e, b, end);
  bounds(e + stride, nb, nend);
  Quad r[kChunksInFlight], rn[kChunksInFlight];
  fetch(r, b, end, end);
  for (;;) {
    int nnb, nnend;
    bounds(e + 2 * stride, nnb, nnend);
    fetch(rn, nb, nend, nend);
    float carry = 0.f;  // R of the first step of the later chunk
    for (int hi = end; hi > b; hi -= kChunkSteps * kChunksInFlight) {
      if (hi != end) fetch(r, b, hi, end);  // long episodes: further rounds
      float s[kChunksInFlight][4], total[kChunksInFlight], t1[kChunksInFlight], t2[kChunksInFlight], t3[kChunksInFlight];
#pragma unroll
      for (int c = 0; c < kChunksInFlight; ++c) {
        s[c][3] = r[c].v[3];
        s[c][2] = r[c].v[2] + gamma * s[c][3];
        s[c][1] = r[c].v[1] + gamma * s[c][2];
        s[c][0] = r[c].v[0] + gamma * s[c][1];
        total[c] = suffix_scan(s[c][0], lane, w, t1[c], t2[c], t3[c]);
      }
#pragma unroll
      for (int c = 0; c < kChunksInFlight; ++c) {
        const int t = hi - kChunkSteps * (c + 1) + 4 * lane;
        const float with_carry = total[c] + w.to_chunk_end * carry;
        // total of the next lane (with the carry): inside a row by a shift, at a row's last lane the
        // head of the next row, at lane 63 the carry itself
        const float h1 = t1[c] + w.g16 * w.g16 * w.g16 * carry;  // lane 16: 48 lanes before the chunk's end
        const float h2 = t2[c] + w.g16 * w.g16 * carry;
        const float h3 = t3[c] + w.g16 * carry;
        float next = row_shift_down<1>(with_carry);
        if ((lane & 15) == 15) next = row == 0 ? h1 : row == 1 ? h2 : row == 2 ? h3 : carry;
        Quad out;
        out.v[0] = with_carry;
        out.v[1] = s[c][1] + g3 * next;
        out.v[2] = s[c][2] + g2 * next;
        out.v[3] = s[c][3] + gamma * next;
        if (t >= b && t + 3 < end) {
          QuadMem m;
#pragma unroll
          for (int j = 0; j < 4; ++j) m.v[j] = out.v[j];
          *reinterpret_cast<QuadMem*>(discounted + t) = m;
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (t + j >= b && t + j < end) discounted[t + j] = out.v[j];
        }
        carry = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, with_carry)));
      }
    }
    e += stride;
    if (e >= episodes) break;
    b = nb;
    end = nend;
    nb = nnb;
    nend = nnend;
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) r[c] = rn[c];
  }
}

// ---- the same for many short episodes ----
// A wave per episode leaves most of its lanes idle: one wave takes a group of up to 64 consecutive episodes, about kGroupSteps
// steps, as one run of steps with the same scan.  Every addition is left out where an episode ends in between: lanes mark the last
// steps of the group's episodes in LDS, and a lane knows from the ballot of marked lanes how many lanes on the first end lies.
// Left out and not weighted by zero: the next episode's values may be infinite.  Bound by the latency of a load, the scan and a
// store; groups of 200 steps were up to 1.9 times as slow beyond 50 steps an episode.
constexpr int kGroupSteps = 384;  // a group of average length fits the chunks in flight
// A group's episodes follow from the mean length alone, so long ones that stand together would all fall to one wave, 1.1 us a round of
// 512 steps.  Groups of more than kGroupMost steps beside their longest episode are therefore left to further waves: each looks
// through a share of the groups and takes one part of every such group that it finds, parts of equal steps, as many as a group has
// episodes where that makes kPartWaves waves or fewer.  64 neighbours of 10000 steps among 60000 episodes of one step 706 -> 23 us
// (30 in the form above), 64 of 1000 among 65536 of four 112 -> 8.3 (21); evenly drawn lengths 1 to 4 % slower, 300000 episodes 13 %.
// Cut by steps and not by count, which needs a search in the offsets before the loads, those took 1.1 to 2 times as long.
constexpr int kGroupMost = 2048, kPartWaves = 1024, kLeastParts = 4;
constexpr int kShareGroups = 256;  // groups in a share: four loads a lane, all in flight
// Their place: behind all groups of a grid that is resident as a whole (2048 blocks), where nothing waits for their blocks; near the start of a
// larger one, at whose end they are waited for (300000 episodes of 3 to 33 steps: 10.3 us without them, 14.2 there, 11.6 early).
constexpr int kResidentBlocks = 2048, kEarly = 256;
// Taken from the number of episodes on at which a wave of the other form walks several, and up to an average length: 44013
// episodes of 3 to 33 steps 4.9 us, there 16.8; 60000 of 8 to 120 10.2 and 22.9; 16000 of 8 to 200 6.9 and 8.8; 8000 of 5 to 60
// 4.8 and 5.8; but 65536 of 8 to 500 32.0 and 25.6, 4000 of 5 to 60 4.8 and 4.5.
constexpr int kShortEpisodes = 8192, kShortSteps = 128;

// v[l] <- sum over the lanes m >= l of factor^(m - l) * v[m], up to the first lane in which an episode ends: `ends` has a bit for
// each such lane, `reach` is the distance to the first one (64: none).  t1/t2/t3 return the finished values of lanes 16, 32, 48
// (the row heads) without the carry of a later chunk.
__device__ __forceinline__ float segment_scan(float v, int lane, uint64_t ends, int reach, const ScanWeights& w, float& t1, float& t2,
                                             float& t3) {
  float o = w.g1 * row_shift_down<1>(v);
  v += reach >= 1 ? o : 0.f;
  o = w.g2 * row_shift_down<2>(v);
  v += reach >= 2 ? o : 0.f;
  o = w.g4 * row_shift_down<4>(v);
  v += reach >= 4 ? o : 0.f;
  o = w.g8 * row_shift_down<8>(v);
  v += reach >= 8 ? o : 0.f;
  const int iv = __builtin_bit_cast(int, v);
  t3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 48));
  t2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 32)) + ((ends >> 32 & 0xffff) == 0 ? w.g16 * t3 : 0.f);
  t1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(iv, 16)) + ((ends >> 16 & 0xffff) == 0 ? w.g16 * t2 : 0.f);
  const int row = lane >> 4;
  const float later_rows = row == 0 ? t1 : row == 1 ? t2 : row == 2 ? t3 : 0.f;
  return v + (reach >= 16 - (lane & 15) ? w.to_row_end * later_rows : 0.f);
}

// Episodes of the steps [b, end), n of them, lane l holding one past the last step of episode l.
__device__ __forceinline__ void discount_run(const float* __restrict__ reward, float* __restrict__ discounted, int b, int end, int my_end,
                                             int n, int lane, float gamma, const ScanWeights& w, uint32_t (&marks)[kChunksInFlight][64]) {
  const float g2 = gamma * gamma, g3 = g2 * gamma;
  const int row = lane >> 4;

  float carry = 0.f;  // R of the first step of the later chunk
  for (int hi = (end + 3) & ~3; hi > b; hi -= kChunkSteps * kChunksInFlight) {
    Quad r[kChunksInFlight];
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) {
      const int t = hi - kChunkSteps * (c + 1) + 4 * lane;
      if (t >= b && t + 3 < end) {
        const QuadMem m = *reinterpret_cast<const QuadMem*>(reward + t);
#pragma unroll
        for (int j = 0; j < 4; ++j) r[c].v[j] = m.v[j];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) r[c].v[j] = (t + j >= b && t + j < end) ? reward[t + j] : 0.f;
      }
    }
    uint32_t mark[kChunksInFlight];
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) marks[c][lane] = 0;
    wave_sync();
    const int back = hi - my_end;  // steps between the end of my episode and the end of the chunks
    if (lane < n && my_end > b && back >= 0 && back < kChunkSteps * kChunksInFlight) {
      const int place = kChunkSteps - 1 - (back & (kChunkSteps - 1));
      atomicOr(&marks[back / kChunkSteps][place >> 2], 1u << (place & 3));
    }
    wave_sync();
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) mark[c] = marks[c][lane];
    wave_sync();
    float s[kChunksInFlight][4], total[kChunksInFlight], t1[kChunksInFlight], t2[kChunksInFlight], t3[kChunksInFlight];
    uint64_t ends[kChunksInFlight];
    int reach[kChunksInFlight];
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) {
      ends[c] = __ballot(mark[c] != 0);
      const uint64_t from_here = ends[c] >> lane;
      reach[c] = from_here ? __builtin_ctzll(from_here) : 64;
      s[c][3] = r[c].v[3];
#pragma unroll
      for (int j = 2; j >= 0; --j) s[c][j] = r[c].v[j] + (mark[c] >> j & 1 ? 0.f : gamma * s[c][j + 1]);
      total[c] = segment_scan(s[c][0], lane, ends[c], reach[c], w, t1[c], t2[c], t3[c]);
    }
#pragma unroll
    for (int c = 0; c < kChunksInFlight; ++c) {
      const int t = hi - kChunkSteps * (c + 1) + 4 * lane;
      const float with_carry = total[c] + (reach[c] >= 64 - lane ? w.to_chunk_end * carry : 0.f);
      // value of the first step of the next lane
      float next = row_shift_down<1>(with_carry);
      if ((lane & 15) == 15) {
        const float from3 = ends[c] >> 48 ? t3[c] : t3[c] + w.g16 * carry;
        const float from2 = ends[c] >> 32 ? t2[c] : t2[c] + w.g16 * w.g16 * carry;
        const float from1 = ends[c] >> 16 ? t1[c] : t1[c] + w.g16 * w.g16 * w.g16 * carry;
        next = row == 3 ? carry : row == 2 ? from3 : row == 1 ? from2 : from1;
      }
      Quad out;
      out.v[3] = s[c][3] + (mark[c] >> 3 ? 0.f : gamma * next);
      out.v[2] = s[c][2] + (mark[c] >> 2 ? 0.f : g2 * next);
      out.v[1] = s[c][1] + (mark[c] >> 1 ? 0.f : g3 * next);
      out.v[0] = with_carry;
      if (t >= b && t + 3 < end) {
        QuadMem m;
#pragma unroll
        for (int j = 0; j < 4; ++j) m.v[j] = out.v[j];
        *reinterpret_cast<QuadMem*>(discounted + t) = m;
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (t + j >= b && t + j < end) discounted[t + j] = out.v[j];
      }
      carry = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, with_carry)));
    }
  }
}

__global__ __launch_bounds__(256) void pg_discount_short_kernel(const float* __restrict__ reward,
                                                                const int32_t* __restrict__ offsets, int episodes, int steps, int per_wave,
                                                                int groups, int shares, int parts, int lead, int part_blocks, float gamma,
                                                                float* __restrict__ discounted) {
  __shared__ uint32_t marks[4][kChunksInFlight][64];  // per wave, chunk and lane: which of its four steps end an episode
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  auto clamped = [&](int v) { return v < 0 ? 0 : v > steps ? steps : v; };
  auto size = [&](int group) { return episodes - group * per_wave < per_wave ? episodes - group * per_wave : per_wave; };
  const float g2 = gamma * gamma;
  const ScanWeights w = scan_weights(g2 * g2, lane);
  const int place = (int)blockIdx.x - lead;  // the parts' blocks stand behind the first `lead` of the groups'
  if (place < 0 || place >= part_blocks) {
    const int group = (place < 0 ? (int)blockIdx.x : (int)blockIdx.x - part_blocks) * 4 + wv;
    if (group >= groups) return;
    const int e0 = group * per_wave, n = size(group);
    const int my_end = lane < n ? clamped(offsets[e0 + lane + 1]) : 0;  // lane l: one past the last step of episode l
    const int b = __builtin_amdgcn_readfirstlane(clamped(offsets[e0])), end = __builtin_amdgcn_readlane(my_end, n - 1);
    if (end - b > kGroupMost) {
      const int before = __shfl_up(my_end, 1, 64);
      int longest = lane < n ? my_end - (lane ? before : b) : 0;
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) longest = max(longest, __shfl_xor(longest, d, 64));
      if (end - b - longest > kGroupMost) return;
    }
    discount_run(reward, discounted, b, end, my_end, n, lane, gamma, w, marks[wv]);
    return;
  }
  // part `part` of the groups share, share + shares, ...
  const int wave = place * 4 + wv, part = wave % parts, share = wave / parts;
  if (share >= shares) return;
  int from[4], to[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t group = share + (int64_t)(lane + 64 * j) * shares;
    from[j] = to[j] = 0;
    if (group < groups) {
      from[j] = clamped(offsets[(int)group * per_wave]);
      to[j] = clamped(offsets[(int)group * per_wave + size((int)group)]);
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    bool is_long = to[j] - from[j] > kGroupMost;
    if (is_long) {
      const int group = share + (lane + 64 * j) * shares, n = size(group);
      int longest = 0, start = from[j];
#pragma unroll 4
      for (int i = 1; i <= n; ++i) {
        const int stop = clamped(offsets[group * per_wave + i]);
        longest = max(longest, stop - start);
        start = stop;
      }
      is_long = to[j] - from[j] - longest > kGroupMost;
    }
    for (uint64_t left = __ballot(is_long); left; left &= left - 1) {
      const int l = (int)__builtin_ctzll(left), group = share + (l + 64 * j) * shares, n = size(group), e0 = group * per_wave;
      const int start = __builtin_amdgcn_readlane(from[j], l), total = __builtin_amdgcn_readlane(to[j], l) - start;
      const int begin = lane < n ? clamped(offsets[e0 + lane]) : 0, stop = lane < n ? clamped(offsets[e0 + lane + 1]) : 0;
      // the part's episodes: neighbours, as their starts ascend
      const uint64_t lanes = __ballot(lane < n && (int64_t)(begin - start) * parts / total == part);
      if (lanes == 0) continue;
      const int first = (int)__builtin_ctzll(lanes), count = (int)__builtin_popcountll(lanes);
      const int my_end = __shfl(stop, first + lane, 64);
      discount_run(reward, discounted, __builtin_amdgcn_readlane(begin, first), __builtin_amdgcn_readlane(my_end, count - 1), my_end, count, lane,
                   gamma, w, marks[wv]);
    }
  }
}

// ---- Sigmoid model, steps 8, 10, 11 ----
template <bool STREAM>
__global__ __launch_bounds__(256) void pg_sigmoid_kernel(const float* __restrict__ aprob,
                                                         const int32_t* __restrict__ action,
                                                         const float* __restrict__ discounted,
                                                         float* __restrict__ dlogps, float* __restrict__ bottom_diff,
                                                         int steps) {
  const int t = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (t + 3 < steps) {
    const float4 ap = *reinterpret_cast<const float4*>(aprob + t);
    const int4 ac = *reinterpret_cast<const int4*>(action + t);
    float4 w = make_float4(1.f, 1.f, 1.f, 1.f);
    if (discounted) w = *reinterpret_cast<const float4*>(discounted + t);
    const float4 d = make_float4(ac.x == 0 ? 1.f - ap.x : 0.f - ap.x, ac.y == 0 ? 1.f - ap.y : 0.f - ap.y,
                                 ac.z == 0 ? 1.f - ap.z : 0.f - ap.z, ac.w == 0 ? 1.f - ap.w : 0.f - ap.w);
    if (dlogps) store4<STREAM>(dlogps + t, d);
    store4<STREAM>(bottom_diff + t, make_float4(-d.x * w.x, -d.y * w.y, -d.z * w.z, -d.w * w.w));
  } else {
    for (int i = t; i < steps; ++i) {
      const float ap = aprob[i];
      const float d = action[i] == 0 ? 1.f - ap : 0.f - ap;
      if (dlogps) dlogps[i] = d;
      bottom_diff[i] = -d * (discounted ? discounted[i] : 1.f);
    }
  }
}

// ---- Softmax model, steps 8, 10, 11 ----
// Up to 32 actions: a block takes 256 consecutive rows, stages them through LDS with coalesced
// loads (row stride padded to an odd number of words so that one row per lane is conflict-free),
// lets each thread do its own row, and streams the results back out the same way.
template <bool STREAM>
__global__ __launch_bounds__(256) void pg_softmax_rows_kernel(const float* __restrict__ logits,
                                                              const int32_t* __restrict__ action,
                                                              const float* __restrict__ discounted,
                                                              float* __restrict__ probs,
                                                              float* __restrict__ bottom_diff, int steps, int A,
                                                              Magic mA, bool vec_ok) {
  extern __shared__ float tile[];  // [256][A | 1], then a second copy for the gradient
  const int AP = A | 1;
  float* const ptile = tile;
  float* const dtile = tile + 256 * AP;
  const int row0 = blockIdx.x * 256;
  const int nrows = steps - row0 < 256 ? steps - row0 : 256;
  const int count = nrows * A;
  const size_t base = (size_t)row0 * A;
  // Four-element global accesses when the block's slice is a multiple of four elements and the
  // blobs are 16-byte aligned (a block's slice then starts on such a boundary too: 256*A elements
  // per block); the (row, column) of the first element comes from one division, the next three
  // follow by stepping the column.
  const bool vec = vec_ok && (count & 3) == 0;
  if (vec) {
    for (int i = threadIdx.x * 4; i < count; i += 1024) {
      const float4 v = load4<STREAM>(logits + base + i);
      int r = (int)mdiv((uint32_t)i, mA), c = i - r * A;
      const float e[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        ptile[r * AP + c] = e[q];
        if (++c == A) {
          c = 0;
          ++r;
        }
      }
    }
  } else {
    for (int i = threadIdx.x; i < count; i += 256) {
      const int r = (int)mdiv((uint32_t)i, mA);
      ptile[r * AP + (i - r * A)] = logits[base + i];
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < nrows) {
    float* const l = ptile + threadIdx.x * AP;
    float* const g = dtile + threadIdx.x * AP;
    const int act = action[row0 + threadIdx.x];
    const float w = discounted ? discounted[row0 + threadIdx.x] : 1.f;
    float top = l[0];
    for (int a = 1; a < A; ++a) top = fmaxf(top, l[a]);
    float sum = 0.f;
    for (int a = 0; a < A; ++a) {
      const float ex = expf(l[a] - top);
      l[a] = ex;
      sum += ex;
    }
    const float inv = 1.f / sum;
    for (int a = 0; a < A; ++a) {
      const float p = l[a] * inv;
      l[a] = p;
      g[a] = (p - (a == act ? 1.f : 0.f)) * w;
    }
  }
  __syncthreads();
  if (vec) {
    for (int i = threadIdx.x * 4; i < count; i += 1024) {
      int r = (int)mdiv((uint32_t)i, mA), c = i - r * A;
      float pv[4], dv[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        pv[q] = ptile[r * AP + c];
        dv[q] = dtile[r * AP + c];
        if (++c == A) {
          c = 0;
          ++r;
        }
      }
      if (probs) store4<STREAM>(probs + base + i, make_float4(pv[0], pv[1], pv[2], pv[3]));
      store4<STREAM>(bottom_diff + base + i, make_float4(dv[0], dv[1], dv[2], dv[3]));
    }
  } else {
    for (int i = threadIdx.x; i < count; i += 256) {
      const int r = (int)mdiv((uint32_t)i, mA);
      const int o = r * AP + (i - r * A);
      if (probs) probs[base + i] = ptile[o];
      bottom_diff[base + i] = dtile[o];
    }
  }
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
  return v;
}

__device__ __forceinline__ float wave_add(float v) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// More than 32 actions: one wave per row, lanes along the row.
__global__ __launch_bounds__(256) void pg_softmax_wide_kernel(const float* __restrict__ logits,
                                                              const int32_t* __restrict__ action,
                                                              const float* __restrict__ discounted,
                                                              float* __restrict__ probs,
                                                              float* __restrict__ bottom_diff, int steps, int A) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= steps) return;
  const float* const l = logits + (size_t)t * A;
  float top = -INFINITY;
  for (int a = lane; a < A; a += 64) top = fmaxf(top, l[a]);
  top = wave_max(top);
  float sum = 0.f;
  for (int a = lane; a < A; a += 64) sum += expf(l[a] - top);
  sum = wave_add(sum);
  const float inv = 1.f / sum;
  const int act = action[t];
  const float w = discounted ? discounted[t] : 1.f;
  for (int a = lane; a < A; a += 64) {
    const float p = expf(l[a] - top) * inv;
    if (probs) probs[(size_t)t * A + a] = p;
    bottom_diff[(size_t)t * A + a] = (p - (a == act ? 1.f : 0.f)) * w;
  }
}

constexpr int32_t kMaxSteps = 0x7FFF0000;  // index arithmetic of the kernels stays below 2^31

int done(void) {
  const int e = (int)hipGetLastError();
  return e ? record_hip_error(e) : CONV_OK;
}

}  // namespace

}  // namespace mi355conv

using namespace mi355conv;

extern "C" {

int pg_sigmoid_sample_action(const float* aprob, const float* random, int32_t* action, int32_t steps,
                             void* hip_stream) {
  if (steps < 0) return CONV_EINVAL;
  if (steps > kMaxSteps) return CONV_ESHAPE;
  if (steps == 0) return CONV_OK;
  if (!aprob || !random || !action) return CONV_EINVAL;
  hipLaunchKernelGGL((size_t)steps * 28 > kCacheBytes ? pg_sample_kernel<true> : pg_sample_kernel<false>, dim3((steps + 1023) / 1024), dim3(256), 0, (hipStream_t)hip_stream, aprob,
                     random, action, steps);
  return done();
}

int pg_discount_rewards(const float* reward, const int32_t* episode_offsets, int32_t episodes, int32_t steps,
                        float gamma, float* discounted, void* hip_stream) {
  if (episodes < 0 || steps < 0) return CONV_EINVAL;
  if (steps > kMaxSteps || episodes > kMaxSteps) return CONV_ESHAPE;
  if (episodes == 0 || steps == 0) return CONV_OK;
  if (!reward || !episode_offsets || !discounted) return CONV_EINVAL;
  if (episodes >= kShortEpisodes && steps / episodes < kShortSteps) {
    const int per_wave = (int)std::min<int64_t>(64, std::max<int64_t>(1, (int64_t)kGroupSteps * episodes / steps));
    const int groups = (int)(((int64_t)episodes + per_wave - 1) / per_wave);
    const int shares = std::max(std::min(groups, kPartWaves / per_wave), (groups + kShareGroups - 1) / kShareGroups);
    const int parts = std::min(per_wave, std::max(kLeastParts, kPartWaves / shares));
    const int group_blocks = (groups + 3) / 4, part_blocks = per_wave == 1 ? 0 : (shares * parts + 3) / 4;
    hipLaunchKernelGGL(pg_discount_short_kernel, dim3(group_blocks + part_blocks), dim3(256), 0, (hipStream_t)hip_stream, reward,
                       episode_offsets, episodes, steps, per_wave, groups, shares, parts, group_blocks <= kResidentBlocks ? group_blocks : kEarly, part_blocks, gamma, discounted);
    return done();
  }
  int blocks = (episodes + 3) / 4;
  if (blocks > 256 * 8) blocks = 256 * 8;  // eight resident workgroups on each of the 256 compute units
  hipLaunchKernelGGL(pg_discount_kernel, dim3(blocks), dim3(256), 0, (hipStream_t)hip_stream, reward,
                     episode_offsets, episodes, steps, gamma, discounted);
  return done();
}

int pg_sigmoid_bottom_diff(const float* aprob, const int32_t* action, const float* discounted, float* dlogps,
                           float* bottom_diff, int32_t steps, void* hip_stream) {
  if (steps < 0) return CONV_EINVAL;
  if (steps > kMaxSteps) return CONV_ESHAPE;
  if (steps == 0) return CONV_OK;
  if (!aprob || !action || !bottom_diff) return CONV_EINVAL;
  hipLaunchKernelGGL((size_t)steps * 28 > kCacheBytes ? pg_sigmoid_kernel<true> : pg_sigmoid_kernel<false>, dim3((steps + 1023) / 1024), dim3(256), 0, (hipStream_t)hip_stream, aprob,
                     action, discounted, dlogps, bottom_diff, steps);
  return done();
}

int pg_softmax_bottom_diff(const float* logits, const int32_t* action, const float* discounted, float* probs,
                           float* bottom_diff, int32_t steps, int32_t actions, void* hip_stream) {
  if (steps < 0 || actions < 1) return CONV_EINVAL;
  if ((int64_t)steps * actions >= ((int64_t)1 << 31)) return CONV_ESHAPE;
  if (steps == 0) return CONV_OK;
  if (!logits || !action || !bottom_diff) return CONV_EINVAL;
  if (actions <= 32) {
    const size_t lds = (size_t)2 * 256 * (actions | 1) * sizeof(float);  // at most 66 KB
    const bool stream = actions <= kStreamActions && (size_t)steps * (12 * actions + 12) > kCacheBytes;
    auto* const kernel = stream ? pg_softmax_rows_kernel<true> : pg_softmax_rows_kernel<false>;
    static LdsOptIn opt_in[2];  // 32 actions need 66 KB: opt in to the largest size, once per process and kernel
    if (lds > 64 * 1024) {
      const int e = lds_opt_in(opt_in[stream], kernel, 2 * 256 * 33 * (int)sizeof(float));
      if (e) return record_hip_error(e);
    }
    const bool vec_ok = (((uintptr_t)logits | (uintptr_t)probs | (uintptr_t)bottom_diff) & 15u) == 0;
    hipLaunchKernelGGL(kernel, dim3((steps + 255) / 256), dim3(256), lds, (hipStream_t)hip_stream,
                       logits, action, discounted, probs, bottom_diff, steps, actions, make_magic((uint32_t)actions),
                       vec_ok);
  } else {
    hipLaunchKernelGGL(pg_softmax_wide_kernel, dim3((steps + 3) / 4), dim3(256), 0, (hipStream_t)hip_stream, logits,
                       action, discounted, probs, bottom_diff, steps, actions);
  }
  return done();
}

}  // extern "C"
