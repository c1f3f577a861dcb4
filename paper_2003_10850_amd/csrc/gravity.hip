// Barnes-Hut gravity with per-particle opening decisions, walked by a whole
// wavefront at a time.
//
// A wave serves 64 Morton-consecutive targets, one per lane, and every lane
// takes the per-particle Barnes-Hut decision for each node the wave visits
// (Barnes & Hut 1986): accept the monopole or open it; a lane whose ancestor
// was accepted is out of the node's mask. A work item is the children of an
// opened node (they lie side by side, see CNode) or the members of an opened
// leaf, with the 64-bit mask of the lanes that opened it. The wave reads an
// item with a few scalar loads, decides and sums each child or member from
// scalar registers, all lanes at once with the mask on the inverse distance,
// and stacks the children that some lane opens.
//
// Bound by vector issue on a full chip: a child costs about 25 instructions
// with its term (the distance of the decision serves the term). The walk
// before this one read one node a step in preorder, a dependent scalar load
// each (0.5 us, 2600 steps a group), and wrote what it accepted to LDS tiles
// that it summed later, about 40 instructions a node.
#include <type_traits>

#include "g3_device.h"
#include "g3_internal.h"
#include "g3_items.h"

namespace g3 {

namespace {

// Terms of plain FP32 partial sums between two compensated additions, at most.
constexpr int kFlush = 64;

// The opening test, exact in FP32: fl(l * l) < fl(theta2 * r2).
__device__ __forceinline__ bool open_accept(float l, float theta2, float r2) {
#pragma clang fp contract(off)
  const float lhs = l * l;
  const float rhs = theta2 * r2;
  return lhs < rhs;
}

// Mixed precision (kF64): positions are stored in FP64 and the node centres
// of mass come from FP64 moments. Decision and term work on the FP32 rounding
// of the FP64 offset of the source from the target; near the threshold, where
// the FP32 test could disagree with the FP64 one, the FP64 test decides.
// The waves of a workgroup share a group: they take its items in rounds, item
// j of a round by wave j % kT, and the items that these open follow in the
// order of their parents, so the sums do not depend on timing. Held to 64
// registers, 8 waves a SIMD: two teams of 16 share a CU (352 us for 2^17
// particles of a clustered box, 451 at 4 waves a SIMD). All particles of a
// clustered 2^21 box: 6.5 ms with the preorder walk of one wave a group, 4.9
// with the items of one wave, 4.3 with teams of 4 or 8, 5.0 with teams of 16;
// of 2^12 particles: 0.50, 0.38, 0.16, 0.10 and 0.08 ms.
template <bool kF64, bool kInside, int kT>
__global__ __launch_bounds__(kT * kWave, 8) void k_gravity(
    const CNode *__restrict__ cnodes, const uint64_t *__restrict__ ckeys,
    const double4 *__restrict__ cc64, const float4 *__restrict__ xm,
    const double4 *__restrict__ x64, const uint64_t *__restrict__ keys,
    const int32_t *__restrict__ perm, const Groups gs, float theta2, float eps2, float G,
    int inside_test, double theta64, float *__restrict__ acc, float *__restrict__ pot,
    int32_t *__restrict__ nterms) {
  __shared__ Team<kT> S;
  // running totals (acc, pot) and their Neumaier compensations, one slot per
  // lane: touched only every kFlush terms, so the walk carries no totals in
  // registers
  __shared__ float4 tots[kT][kWave], comps[kT][kWave];
  __shared__ int32_t nts[kT][kWave];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  float4 *tot = tots[w], *comp = comps[w];
  int range = 0;
  for (int g; (g = team_take_group(gs, range, S)) >= 0;) {
  const Group grp = group_at(gs, g);
  const int64_t t = grp.t0 + lane;
  const bool valid = lane < grp.count;
  const int s = valid ? (gs.targets ? gs.targets[t] : (int)t) : 0;
  const double side = gs.sbox[grp.snap].w;  // root cube side
  // a node's level from its cube side: l = (float)side * 2^-level exactly
  const int root_exp = ilogbf((float)side);
  const float4 me = xm[s];
  const double4 p64 = kF64 ? x64[s] : make_double4(0, 0, 0, 0);
  const uint64_t ki = keys[s];

  tot[lane] = make_float4(0.f, 0.f, 0.f, 0.f);
  comp[lane] = make_float4(0.f, 0.f, 0.f, 0.f);
  float px = 0.f, py = 0.f, pz = 0.f, pp = 0.f;
  int pn = 0, since = 0;
  auto flush = [&]() {
    float4 a = tot[lane], c = comp[lane];
    neumaier_add(a.x, c.x, px);
    neumaier_add(a.y, c.y, py);
    neumaier_add(a.z, c.z, pz);
    neumaier_add(a.w, c.w, pp);
    tot[lane] = a;
    comp[lane] = c;
    px = py = pz = pp = 0.f;
    since = 0;
  };
  // one source at offset (dx, dy, dz), inverse softened distance rinv
  auto add = [&](bool use, float dx, float dy, float dz, float rinv, float m) {
    const float mr = m * rinv;
    const float mr3 = mr * rinv * rinv;
    px += mr3 * dx;
    py += mr3 * dy;
    pz += mr3 * dz;
    pp -= mr;
    pn += use ? 1 : 0;
  };
  // a member, for the lanes that use it: the inverse distance is masked, so that
  // an unused one adds exact zeros also at r2s = 0 (the own particle with zero
  // softening)
  auto term = [&](bool use, float dx, float dy, float dz, float r2s, float m) {
    add(use, dx, dy, dz, use ? __builtin_amdgcn_rsqf(r2s) : 0.0f, m);
  };
  // A node, for the lanes that accept it. Its mass may be above FP32's largest
  // number near the root, where every lane opens it, and infinity times a masked
  // distance of zero is no zero: the lanes branch (all of a clustered 2^21 box:
  // 4143 us with the distance masked, 4030 so). Below a lighter root, teams of 16
  // and launches with a workgroup for every group mask: few waves hide the branch
  // there (3 % of teams of 16; 2 to 4e4 targets of such a box in teams of 4:
  // 1.16 ms masked, 1.26 with the branch).
  constexpr bool kMayMask = !kF64;
  auto node_term = [&](auto mask_c, bool use, float dx, float dy, float dz, float r2s, float m) {
    if constexpr (decltype(mask_c)::value) {
      term(use, dx, dy, dz, r2s, m);
    } else if (use) {
      add(true, dx, dy, dz, __builtin_amdgcn_rsqf(r2s), m);
    }
  };

  // One item: `count` children at cnodes[first], or -count members from
  // `first`, for the lanes of `mask` (all wave-uniform); open(first, count,
  // mask) receives the items that it opens.
  auto items = [&](auto mask_c) {
  return [&](int first, int count, uint64_t mask, const auto &opened) {
    const bool act = __builtin_amdgcn_inverse_ballot_w64(mask);
    if (count > 0) {
      auto visit = [&](const CNode &nd, const double4 &cn, uint64_t nk) {
        const float l = __int_as_float(nd.meta.w);
        float dx, dy, dz;
        if constexpr (kF64) {
          dx = (float)(cn.x - p64.x);
          dy = (float)(cn.y - p64.y);
          dz = (float)(cn.z - p64.z);
        } else {
          dx = sub_exact(nd.com_m.x, me.x);
          dy = sub_exact(nd.com_m.y, me.y);
          dz = sub_exact(nd.com_m.z, me.z);
        }
        const float r2 = dist2_exact(dx, dy, dz);
        bool accept, open;
        if constexpr (!kF64 && !kInside) {
          // the exact test fl(l l) < fl(theta2 r2); neither holds for a
          // distance that is not a number
          float rhs;
          {
#pragma clang fp contract(off)
            rhs = theta2 * r2;
          }
          const float lhs = sq_exact(l);
          accept = act && lhs < rhs;
          open = act && lhs >= rhs;
        } else {
          accept = act && open_accept(l, theta2, r2);
          if constexpr (kF64) {
            // the FP32 r2 of exact-to-2^-24 offsets is within about 2^-22 of
            // the FP64 value (relative); inside 2^-19 of the threshold FP64
            // decides
            const float lhs = l * l, rhs = theta2 * r2;
            if (act && fabsf(lhs - rhs) <= rhs * 1.9073486e-6f)
              accept = open_accept64(ldexp(side, -(root_exp - ilogbf(l))), theta64, cn, p64);
          }
          if (kInside || (kF64 && inside_test)) {
            const int level = root_exp - ilogbf(l);
            const bool inside = ((ki ^ nk) >> (3 * (kMaxLevel - level))) == 0ull;
            accept = accept && !inside;
          }
          open = act && !accept;
        }
        node_term(mask_c, accept, dx, dy, dz, r2 + eps2, nd.com_m.w);
        const uint64_t om = __ballot(open);
        if (om) opened(nd.meta.x, nd.meta.y, om);
      };
      constexpr int kBatch = kF64 ? 2 : 4;  // children in scalar registers at a time
      for (int c0 = 0; c0 < count; c0 += kBatch) {
        CNode nd[kBatch];
        double4 cn[kBatch];
        uint64_t nk[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {  // (the arrays are padded)
          nd[q] = cnodes[first + c0 + q];
          cn[q] = kF64 ? cc64[first + c0 + q] : make_double4(0, 0, 0, 0);
          nk[q] = kInside || kF64 ? ckeys[first + c0 + q] : 0ull;
        }
#pragma unroll
        for (int q = 0; q < kBatch; ++q)
          if (c0 + q < count) visit(nd[q], cn[q], nk[q]);
      }
      since += count;
    } else {
      const int end = first - count;
      int m = first;
      auto member = [&](int j) {
        const bool use = act && s != j;
        if constexpr (kF64) {
          const double4 q = x64[j];
          const float dx = (float)(q.x - p64.x), dy = (float)(q.y - p64.y),
                      dz = (float)(q.z - p64.z);
          term(use, dx, dy, dz, dist2_exact(dx, dy, dz) + eps2, (float)q.w);
        } else {
          const float4 q = xm[j];
          const float dx = q.x - me.x, dy = q.y - me.y, dz = q.z - me.z;
          term(use, dx, dy, dz, dist2_exact(dx, dy, dz) + eps2, q.w);
        }
      };
      for (; m + 4 <= end; m += 4) {
#pragma unroll
        for (int q = 0; q < 4; ++q) member(m + q);
        since += 4;
        if (since > kFlush - 4) flush();
      }
      for (; m < end; ++m, ++since) member(m);
    }
    if (since > kFlush - 8) flush();  // (the next item may be 8 children)
  };
  };

  const int root = __builtin_amdgcn_readfirstlane(grp.snap);
  const uint64_t all = grp.count < kWave ? (1ull << grp.count) - 1ull : ~0ull;
  if constexpr (kMayMask) {
    if (cnodes[root].com_m.w < INFINITY &&
        (kT == 16 || gs.gstart[*gs.nseg] <= (int)gridDim.x))
      team_items(S, root, all, w, lane, items(std::true_type{}));
    else
      team_items(S, root, all, w, lane, items(std::false_type{}));
  } else {
    team_items(S, root, all, w, lane, items(std::false_type{}));
  }
  flush();
  float4 tt = tot[lane], tc4 = comp[lane];
  nts[w][lane] = pn;
  __syncthreads();
  if (w > 0) continue;
#pragma unroll 1
  for (int v = 1; v < kT; ++v) {  // the waves' totals in their order
    const float4 a = tots[v][lane], c = comps[v][lane];
    neumaier_add(tt.x, tc4.x, a.x);
    neumaier_add(tt.y, tc4.y, a.y);
    neumaier_add(tt.z, tc4.z, a.z);
    neumaier_add(tt.w, tc4.w, a.w);
    tc4.x += c.x;
    tc4.y += c.y;
    tc4.z += c.z;
    tc4.w += c.w;
    pn += nts[v][lane];
  }

  if (valid) {
    const int cid = perm[s];
    if (acc) {
      acc[3 * cid] = G * (tt.x + tc4.x);
      acc[3 * cid + 1] = G * (tt.y + tc4.y);
      acc[3 * cid + 2] = G * (tt.z + tc4.z);
    }
    if (pot) pot[cid] = G * (tt.w + tc4.w);
    if (nterms) nterms[cid] = pn;
  }
  }  // groups
}

}  // namespace

hipError_t launch_gravity(const Octree &all, const Groups &gs, int64_t max_groups,
                          const GravParams &gp, float *acc, float *pot, int32_t *nterms,
                          hipStream_t s) {
  if (max_groups <= 0 || all.nnodes == 0) return hipSuccess;
  if (!all.cnodes) return hipErrorInvalidValue;
  // FP32: the containment test is compiled in or out; FP64: a runtime flag
  auto pick = [&](auto team_c) {
    constexpr int kT = decltype(team_c)::value;
    return gp.f64 ? k_gravity<true, false, kT>
                  : (gp.inside_test ? k_gravity<false, true, kT> : k_gravity<false, false, kT>);
  };
  auto kern = gp.team == 16  ? pick(std::integral_constant<int, 16>{})
              : gp.team == 8 ? pick(std::integral_constant<int, 8>{})
              : gp.team == 4 ? pick(std::integral_constant<int, 4>{})
                             : nullptr;
  if (!kern) return hipErrorInvalidValue;  // (no such team)
  const int block = gp.team * kWave;
  kern<<<persistent_grid((const void *)kern, block, max_groups, gp.team), block, 0, s>>>(
      all.cnodes, all.ckeys, all.cc64, all.xm, all.x64, all.keys, all.perm, gs, gp.theta2,
      gp.eps2, gp.G, gp.inside_test, gp.theta, acc, pot, nterms);
  return hipGetLastError();
}

}  // namespace g3
