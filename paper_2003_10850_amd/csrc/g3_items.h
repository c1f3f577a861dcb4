// The Barnes-Hut walk of a team: the work items of a group, taken in rounds
// by the waves of a workgroup. An item is the children of an opened node (they
// lie side by side, see CNode) or the members of an opened leaf, with the
// 64-bit mask of the lanes (targets) that opened it.
#pragma once
#include "g3_device.h"
#include "g3_internal.h"

namespace g3 {

// Items that wait in a depth-first walk: at most 7 siblings on each of the 22
// levels.
constexpr int kDepth = 7 * (kMaxLevel + 1) + 1;
// A team of kT waves takes up to kItems items a round from the end of the
// list; while more than one is taken the list stays below kStack - kDepth, so
// a depth-first descent always fits.
template <int kT>
struct Team {
  static constexpr int kItems = 4 * kT;
  static constexpr int kStack = kDepth + 16 * kItems;
  int4 stack[kStack];
  int4 out[8 * kItems];  // the items that an item opens
  int32_t nout[kItems];
  int32_t group;
};

// The team's next group, or -1 (every thread of the block calls it).
template <int kT>
__device__ __forceinline__ int team_take_group(const Groups &gs, int &range, Team<kT> &S) {
  __syncthreads();  // the previous group's LDS use is over
  if (threadIdx.x < (unsigned)kWave) {
    const int g = next_group(gs, range);
    if (threadIdx.x == 0) S.group = g;
  }
  __syncthreads();
  return __builtin_amdgcn_readfirstlane(S.group);
}

// Takes every item from the root's (its one child, mask `all`) on:
// item(first, count, mask, opened) handles one - `count` children at
// cnodes[first], or -count members from `first` (all wave-uniform) - and calls
// opened(first, count, mask) for at most 8 items that it opens. Item j of a
// round goes to wave j % kT, and the items that a round opens follow in the
// order of their parents, so the walk does not depend on timing.
template <int kT, typename Item>
__device__ __forceinline__ void team_items(Team<kT> &S, int root, uint64_t all, int w, int lane,
                                           const Item &item) {
  constexpr int kItems = Team<kT>::kItems;
  auto pack = [](int first, int count, uint64_t m) {
    return make_int4(first, count, (int)(uint32_t)m, (int)(uint32_t)(m >> 32));
  };
  auto unpack = [&](const int4 &e, int &first, int &count, uint64_t &m) {
    first = __builtin_amdgcn_readfirstlane(e.x);
    count = __builtin_amdgcn_readfirstlane(e.y);
    m = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(e.w) << 32) |
        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane(e.z);
  };
  if (threadIdx.x == 0) S.stack[0] = pack(root, 1, all);
  int sp = 1;
  while (sp > 0) {
    __syncthreads();
    // (7 more entries an item at most)
    const int room = (Team<kT>::kStack - kDepth - sp) / 7;
    const int n = min(min(kItems, sp), max(room, 1));
    for (int j = w; j < n; j += kT) {
      int first, count, r = 0;
      uint64_t mask;
      unpack(S.stack[sp - n + j], first, count, mask);
      item(first, count, mask, [&](int f, int c, uint64_t m) {
        if (lane == 0) S.out[8 * j + r] = pack(f, c, m);
        ++r;
      });
      if (lane == 0) S.nout[j] = r;
    }
    __syncthreads();
    sp -= n;
    int tot_new = 0;
    for (int j0 = 0; j0 < n; j0 += kWave) {  // every wave counts, all copy
      const int mine = j0 + lane < n ? S.nout[j0 + lane] : 0;
      int inc = mine;
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        const int o = __shfl_up(inc, (unsigned)d, kWave);
        if (lane >= d) inc += o;
      }
      for (int q = w; q * 8 < min(n - j0, kWave); q += kT) {
        const int j = q * 8 + (lane >> 3), r = lane & 7;  // 8 items' slots
        const int cnt = __shfl(mine, j, kWave), at = __shfl(inc, j, kWave) - cnt;
        if (r < cnt) S.stack[sp + tot_new + at + r] = S.out[8 * (j0 + j) + r];
      }
      tot_new += __shfl(inc, kWave - 1, kWave);
    }
    sp += __builtin_amdgcn_readfirstlane(tot_new);
  }
}

}  // namespace g3
