// Teams: T waves of one workgroup serve one group of up to 64 targets
// together, for launches with too few groups to fill the chip one wave each.
//
// A wave that walks and sums a group alone is a serial chain (about 100
// dependent node loads and 50 candidate tiles, 150-250 us a neighbour pass):
// with few active particles the chip idles while a few hundred such chains
// run. A team splits both halves. The walk becomes a search of the flat list
// of the octree's terminal nodes (the nodes that a walk takes whole) in tree
// order: 64 terminals form a window with a box of its own, a lane tests a
// window or a terminal against the group's box, and only what passes takes
// the exact test of every target. The waves take the windows in turn, the
// accepted members are laid out in tree order, and the waves take the
// 64-candidate tiles in turn.
//
// The accepted terminals are exactly those of the one-wave walk: a terminal
// is reached there when it and every ancestor pass the box test of some
// lane, and an ancestor's box (and largest h) contains the terminal's, so
// with box_dist2 monotone in the box the terminal's own test decides. The
// order and the cut into tiles of 64 are the walk's too.
#pragma once
#include "g3_device.h"

namespace g3 {

constexpr int kTermWindow = 64;
// Up to this many accepted terminals of a window are written one after another
// by the whole wave (about 30 instructions each), more by a lane each (about 5
// instructions a member of the largest). Only the first form: 2670 us for a
// forest of 40 snapshots, 6000 for density and force with gradients at 1.25e5
// particles; 2550 and 5740 with both (lines of 10 to 32 within 1 %).
constexpr int kFewTerms = 16;

// Squared distance of two boxes with the rounding steps of box_dist2: never
// larger than box_dist2 of a point inside [a_lo, a_hi].
__device__ __forceinline__ float box_box_dist2(float4 a_lo, float4 a_hi, float4 lo, float4 hi) {
#pragma clang fp contract(off)
  const float dx = fmaxf(fmaxf(lo.x - a_hi.x, a_lo.x - hi.x), 0.0f);
  const float dy = fmaxf(fmaxf(lo.y - a_hi.y, a_lo.y - hi.y), 0.0f);
  const float dz = fmaxf(fmaxf(lo.z - a_hi.z, a_lo.z - hi.z), 0.0f);
  return dist2_exact(dx, dy, dz);
}

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// A round holds one or more tiles of every wave of the team, as many of each.
template <int T>
struct TeamLds {
  static constexpr int kTiles = T == 12 ? 24 : 16;
  static_assert(kTiles % T == 0, "as many tiles for every wave");
  static constexpr int kRound = kTiles * kWave;
  int32_t cand[kRound];
  uint64_t wmask[kTermWindow];
  int32_t wid[kTermWindow], wcnt[kTermWindow];
  int32_t group;
  uint32_t next;  // tiles of the round taken so far
};

// The team's waves take the round's tiles one at a time (their costs differ).
template <int T>
__device__ __forceinline__ int team_next_tile(TeamLds<T> &S) {
  uint32_t j = 0;
  if ((threadIdx.x & 63u) == 0u) j = atomicAdd(&S.next, 1u);
  return __builtin_amdgcn_readfirstlane((int)j);
}

// The team's next group, or -1 (every thread of the block calls it).
template <int T>
__device__ __forceinline__ int team_next_group(const Groups &gs, int &range, TeamLds<T> &S) {
  __syncthreads();  // the previous group's LDS use is over
  if (threadIdx.x < (unsigned)kWave) {
    const int g = next_group(gs, range);
    if (threadIdx.x == 0) S.group = g;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(S.group);
}

__device__ __forceinline__ int wave_incl_sum(int v, int lane) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    const int o = __shfl_up(v, (unsigned)d, kWave);
    if (lane >= d) v += o;
  }
  return v;
}

// Finds the candidates of the group in tree order and hands them to
// `round(ntiles, count)`: S.cand[0..count) are candidates (sorted indices)
// that make up ntiles tiles of 64 (the last one of a group may be short).
// Every wave calls it with the same group: lane i holds target i.
//   xi, want2  the target and its walk limit: reach2(want2, terminal's hmax)
//              is the squared radius that a box must come within (negative
//              for a lane without a target)
//   tlo, thi   the box of the lanes that want anything, gmax2 their largest
//              want2 (wave-uniform)
// `round` runs on every wave and may use __syncthreads (uniformly).
// kDeep: for long lists, and for few targets among many members. A row of windows
// is looked at only where its block passes; and where a group is wide against its
// radius, so that almost every terminal lies in its box though few lie near a
// target, its windows take the exact test too, shared out to the waves, before
// their terminals do. Candidates and order are the same. 64 random targets of 4e6:
// force 4580 us without, 1610 so; density of 10^6 with terminals of 16 members 7.3
// and 4.2 ms. A kernel that has both ways costs all others 2 to 4 % (registers),
// so the launch chooses.
template <int T, bool kDeep, typename Reach, typename Round>
__device__ __forceinline__ void team_search(const Terms &tm, int snap, TeamLds<T> &S, float3 xi,
                                            float want2, float4 tlo, float4 thi, float gmax2,
                                            const Reach &reach2, const Round &round) {
  constexpr int kRound = TeamLds<T>::kRound;
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  const int2 tr = tm.range[snap];
  const int tb = __builtin_amdgcn_readfirstlane(tr.x), te = __builtin_amdgcn_readfirstlane(tr.y);
  if (tb >= te) return;
  const int w0 = tb / kTermWindow, w1 = (te - 1) / kTermWindow;
  int tc = 0;  // candidates waiting in S.cand
  // the windows c0 + b for the bits b of M (at least one), by every wave
  auto windows = [&](int c0, uint64_t M) {
    const int nw = __popcll(M);
    // the wave's first window stays in registers: its accepted terminals, a
    // lane's first member, count and the members up to and with it
    uint64_t acc0 = 0ull;
    int st0 = 0, cnt0 = 0, inc0 = 0;
    {
      uint64_t mm = M;
      for (int k = 0; k < w; ++k) mm &= mm - 1ull;  // (0 stays 0)
      for (int k = w; k < nw; k += T) {
        const int win = c0 + (int)__builtin_ctzll(mm);
        const int t = win * kTermWindow + lane;
        const bool in = t >= tb && t < te;
        float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
        int cnt = 0;
        if (in) {
          lo = tm.lo[t];
          hi = tm.hi[t];
          cnt = __float_as_int(tm.hi[t + 1].w) - __float_as_int(hi.w);
        }
        uint64_t B = __ballot(in && box_box_dist2(tlo, thi, lo, hi) < reach2(gmax2, lo.w));
        uint64_t acc = 0ull;
        while (B) {
          const int b = (int)__builtin_ctzll(B);
          B &= B - 1ull;
          const float4 bl = make_float4(lane_value(lo.x, b), lane_value(lo.y, b),
                                        lane_value(lo.z, b), lane_value(lo.w, b));
          const float4 bh = make_float4(lane_value(hi.x, b), lane_value(hi.y, b),
                                        lane_value(hi.z, b), 0.0f);
          if (__ballot(box_dist2(xi, bl, bh) < reach2(want2, bl.w)) != 0ull) acc |= 1ull << b;
        }
        const int mine = ((acc >> lane) & 1ull) ? cnt : 0;
        const int inc = wave_incl_sum(mine, lane);
        const int tot = __builtin_amdgcn_readlane(inc, kWave - 1);
        if (k == w) {
          acc0 = acc;
          st0 = __float_as_int(hi.w);
          cnt0 = mine;
          inc0 = inc;
        }
        if (lane == 0) {
          S.wmask[k] = acc;
          S.wid[k] = win;
          S.wcnt[k] = tot;
        }
        for (int q = 0; q < T; ++q) mm &= mm - 1ull;
      }
    }
    __syncthreads();
    // window k's candidates are the positions [tc + off_k, tc + off_k + cnt_k)
    const int wc = lane < nw ? S.wcnt[lane] : 0;
    const int winc = wave_incl_sum(wc, lane);
    const int total = tc + __shfl(winc, kWave - 1, kWave);
    for (int r0 = 0; r0 < total; r0 += kRound) {
      for (int k = w; k < nw; k += T) {
        const int kc = __shfl(wc, k, kWave), p1 = tc + __shfl(winc, k, kWave), p0 = p1 - kc;
        if (kc == 0 || p0 >= r0 + kRound || p1 <= r0) continue;
        uint64_t acc = acc0;
        int st = st0, cnt = cnt0, inc = inc0;
        if (k != w) {
          acc = S.wmask[k];
          const int t = S.wid[k] * kTermWindow + lane;
          st = cnt = 0;
          if ((acc >> lane) & 1ull) {
            st = __float_as_int(tm.hi[t].w);
            cnt = __float_as_int(tm.hi[t + 1].w) - st;
          }
          inc = wave_incl_sum(cnt, lane);
        }
        const int at = p0 + inc - cnt - r0;  // position in the round
        if (__popcll(acc) > kFewTerms) {
          // a lane writes the members of its terminal
          const int i0 = max(0, -at), i1 = min(cnt, kRound - at);
          for (int i = i0; __ballot(i < i1) != 0ull; ++i)
            if (i < i1) S.cand[at + i] = st + i;
          continue;
        }
        uint64_t left = acc;
        while (left) {
          const int b = (int)__builtin_ctzll(left);
          left &= left - 1ull;
          const int bs = __builtin_amdgcn_readlane(st, b), bc = __builtin_amdgcn_readlane(cnt, b);
          const int ba = __builtin_amdgcn_readlane(at, b);
          const int i1 = min(bc, kRound - ba);
          for (int i = max(0, -ba) + lane; i < i1; i += kWave) S.cand[ba + i] = bs + i;
        }
      }
      if (total - r0 < kRound) break;  // not a full round: wait for more
      if (threadIdx.x == 0) S.next = 0;
      __syncthreads();
      round(TeamLds<T>::kTiles, kRound);
      __syncthreads();
    }
    tc = total % kRound;
    __syncthreads();  // wmask, wid and wcnt are free again
  };
  if constexpr (!kDeep) {
    for (int c0 = w0; c0 <= w1; c0 += kWave) {
      bool maybe = false;
      if (c0 + lane <= w1) {
        const float4 lo = tm.wlo[c0 + lane], hi = tm.whi[c0 + lane];
        maybe = box_box_dist2(tlo, thi, lo, hi) < reach2(gmax2, lo.w);
      }
      const uint64_t M = __ballot(maybe);
      if (M != 0ull) windows(c0, M);
    }
  } else {
    const float ex = fmaxf(thi.x - tlo.x, fmaxf(thi.y - tlo.y, thi.z - tlo.z));
    const bool wide = ex * ex > 16.0f * reach2(gmax2, 0.0f);
    for (int b0 = w0 / kWave; b0 <= w1 / kWave; b0 += kWave) {
      bool look = false;
      if (b0 + lane <= w1 / kWave) {
        const float4 lo = tm.blo[b0 + lane], hi = tm.bhi[b0 + lane];
        look = box_box_dist2(tlo, thi, lo, hi) < reach2(gmax2, lo.w);
      }
      for (uint64_t blocks = __ballot(look); blocks; blocks &= blocks - 1ull) {
        const int c0 = (b0 + (int)__builtin_ctzll(blocks)) * kWave;
        bool maybe = false;
        float4 wl = make_float4(0.f, 0.f, 0.f, 0.f), wh = wl;
        if (c0 + lane >= w0 && c0 + lane <= w1) {
          wl = tm.wlo[c0 + lane];
          wh = tm.whi[c0 + lane];
          maybe = box_box_dist2(tlo, thi, wl, wh) < reach2(gmax2, wl.w);
        }
        uint64_t M = __ballot(maybe);
        if (M == 0ull) continue;
        if (wide) {
          uint64_t mine = 0ull, mm = M;
          for (int k = 0; mm; ++k, mm &= mm - 1ull) {
            if (k % T != w) continue;
            const int b = (int)__builtin_ctzll(mm);
            const float4 bl = make_float4(lane_value(wl.x, b), lane_value(wl.y, b),
                                          lane_value(wl.z, b), lane_value(wl.w, b));
            const float4 bh = make_float4(lane_value(wh.x, b), lane_value(wh.y, b),
                                          lane_value(wh.z, b), 0.0f);
            if (__ballot(box_dist2(xi, bl, bh) < reach2(want2, bl.w)) != 0ull) mine |= 1ull << b;
          }
          if (lane == 0) S.wmask[w] = mine;
          __syncthreads();
          M = 0ull;
          for (int v = 0; v < T; ++v) M |= S.wmask[v];
          M = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(M >> 32)) << 32) |
              (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)M);
          __syncthreads();  // wmask is free again
          if (M == 0ull) continue;
        }
        windows(c0, M);
      }
    }
  }
  if (tc > 0) {
    if (threadIdx.x == 0) S.next = 0;
    __syncthreads();
    round((tc + kWave - 1) / kWave, tc);
    __syncthreads();
  }
}

// The tiles' partial sums, merged in tile order by waves 0..C-1, one
// component each: the compensated totals are those of one wave that adds
// every tile itself, whatever the team's size.
template <int T, int C>
struct TeamSums {
  static_assert(T >= C, "one wave a component");
  float part[TeamLds<T>::kTiles][C][kWave];
  int32_t count[T][kWave];

  __device__ __forceinline__ void put(int tile, int lane, const float (&v)[C]) {
#pragma unroll
    for (int k = 0; k < C; ++k) part[tile][k][lane] = v[k];
  }
  // Adds this wave's component of the round's tiles to (s, c); barriers on
  // both sides keep the tiles' writers away.
  __device__ __forceinline__ void merge(int ntiles, int w, int lane, float &s, float &c) {
    __syncthreads();
    if (w < C)
      for (int j = 0; j < ntiles; ++j) neumaier_add(s, c, part[j][w][lane]);
  }
};

// The waves' own totals (sum, compensation) added into wave 0's, in the order
// of the waves; buf: [T] areas of kWords floats, at least C x 64, whose earlier
// use by their wave is over.
template <int T, int C, int kWords>
__device__ __forceinline__ void team_totals(float *buf, int w, int lane, float (&sum)[C],
                                            float (&cmp)[C]) {
  static_assert(kWords >= C * kWave, "the areas hold one float a lane and component");
  float *mine = buf + (size_t)w * kWords + lane;
#pragma unroll
  for (int k = 0; k < C; ++k) mine[k * kWave] = sum[k];
  __syncthreads();
  if (w == 0)
#pragma unroll 1
    for (int v = 1; v < T; ++v)
#pragma unroll
      for (int k = 0; k < C; ++k)
        neumaier_add(sum[k], cmp[k], buf[(size_t)v * kWords + k * kWave + lane]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < C; ++k) mine[k * kWave] = cmp[k];
  __syncthreads();
  if (w == 0)
#pragma unroll 1
    for (int v = 1; v < T; ++v)
#pragma unroll
      for (int k = 0; k < C; ++k) cmp[k] += buf[(size_t)v * kWords + k * kWave + lane];
}

// The waves' counts added up (a wave's area holds one word a lane or more).
template <int T, int kWords>
__device__ __forceinline__ void team_count(int *buf, int w, int lane, int &n) {
  __syncthreads();
  buf[(size_t)w * kWords + lane] = n;
  __syncthreads();
  n = 0;
#pragma unroll
  for (int v = 0; v < T; ++v) n += buf[(size_t)v * kWords + lane];
}

}  // namespace g3
