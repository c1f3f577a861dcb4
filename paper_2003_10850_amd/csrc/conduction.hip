// Thermal conduction: the paper's third ported SPH module (section 1, the
// list of modules moved to the GPU). The paper prints no formula; Gadget's
// conduction (Jubelgas, Springel & Dolag 2004) uses the SPH form of
// rho du/dt = div(kappa grad u) of Brookshaw (1985):
//   du_i/dt = sum_j m_j (kappa_i + kappa_j) (u_i - u_j) Fbar_ij / (rho_i rho_j),
//   Fbar_ij = (F(r, h_i) + F(r, h_j)) / 2,  F = (1/r) dW/dr,
// over gas j with r < max(h_i, h_j): the hydro force's symmetric pairs, so
// the kernel has the hydro force's search and tiles with a lighter pair.
//
// A team of waves serves a group of up to 64 Morton-consecutive targets
// (g3_team.h) with each lane's radius max(h_i, hmax(terminal)); 64-entry tiles
// in LDS after the group-box cull are scanned by every lane with the exact
// symmetric test.
#include <cmath>

#include "g3_device.h"
#include "g3_internal.h"
#include "g3_team.h"

namespace g3 {
namespace {

constexpr int kTile = kWave;

// Sorted-order inputs of the pair: ch[s] = (h, u, kappa, 1/rho) with
// kappa = kappa0 u^kappa_exp.
template <typename HT>
__global__ void k_cond_prep(const int32_t *__restrict__ perm, int64_t m,
                            const float *__restrict__ u, const HT *__restrict__ h,
                            const float *__restrict__ rho, float kappa0, float kappa_exp,
                            float4 *__restrict__ ch) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const int j = perm[s];
  const float uj = fmaxf(u[j], 0.0f);
  const float kj = kappa_exp == 0.0f ? kappa0 : kappa0 * powf(uj, kappa_exp);
  ch[s] = make_float4((float)h[j], u[j], kj, 1.0f / rho[j]);
}

struct CondTile {
  float4 xm[kTile], ch[kTile];
};

// kT > 1: a team serves a group, each wave keeping the totals of its own
// tiles. kT = 1: a wave walks the octree (hmax refit from h) by itself, four
// to a workgroup: the pair is light, so with groups to fill the chip the
// team's search is what it gains back. What depends on j alone is formed once
// a candidate. 2.5e5 targets: 1945 us with one wave a group, 985 with teams;
// 4.2e6: 8181 before, 7779 with one wave now, 9138 with teams.
template <int kT>
constexpr int kWavesOf = kT > 1 ? kT : 4;
struct NoLds {};

template <int kT, bool kDeep = false>
__global__ __launch_bounds__(kWavesOf<kT> * kWave, 8) void k_conduction(
    const Node *__restrict__ nodes, const float4 *__restrict__ xm,
    const float4 *__restrict__ ch, const int32_t *__restrict__ perm, const Groups gs,
    int walk_leaf, const Terms tm, float *__restrict__ dudt, int32_t *__restrict__ npairs) {
  constexpr int kWaves = kWavesOf<kT>;
  __shared__ typename std::conditional<(kT > 1), TeamLds<kWaves>, NoLds>::type search;
  __shared__ CondTile tiles[kWaves];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  CondTile &T = tiles[w];
  int range = 0;
  auto take_group = [&]() {
    if constexpr (kT > 1) return team_next_group(gs, range, search);
    else return next_group(gs, range);
  };
  for (int g; (g = take_group()) >= 0;) {
    const Group grp = group_at(gs, g);
    const int64_t t = grp.t0 + lane;
    const bool valid = lane < grp.count;
    const int s = valid ? (gs.targets ? gs.targets[t] : (int)t) : 0;
    const float4 me = xm[s], mc = ch[s];
    const float3 xi = make_float3(me.x, me.y, me.z);
    const float hi = valid ? mc.x : -1.0f;  // invalid lanes never want anything
    const float hi2 = valid ? sq_exact(hi) : -1.0f;
    const float ui = mc.y, kappai = mc.z, rinvi = mc.w;
    const float hinvi = 1.0f / mc.x;
    const float hi5 = (hinvi * hinvi) * (hinvi * hinvi) * hinvi;
    float du = 0.f, cdu = 0.f;  // this wave's tiles
    int np = 0, cand = 0;
    // the group's target box and largest squared radius (group-box cull)
    float4 tlo = make_float4(valid ? xi.x : INFINITY, valid ? xi.y : INFINITY,
                             valid ? xi.z : INFINITY, 0.f);
    float4 thi = make_float4(valid ? xi.x : -INFINITY, valid ? xi.y : -INFINITY,
                             valid ? xi.z : -INFINITY, 0.f);
    float hmax2 = hi2, gh = hi;  // gh: the group's largest h
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
      gh = fmaxf(gh, __shfl_xor(gh, m));
      tlo.x = fminf(tlo.x, __shfl_xor(tlo.x, m));
      tlo.y = fminf(tlo.y, __shfl_xor(tlo.y, m));
      tlo.z = fminf(tlo.z, __shfl_xor(tlo.z, m));
      thi.x = fmaxf(thi.x, __shfl_xor(thi.x, m));
      thi.y = fmaxf(thi.y, __shfl_xor(thi.y, m));
      thi.z = fmaxf(thi.z, __shfl_xor(thi.z, m));
      hmax2 = fmaxf(hmax2, __shfl_xor(hmax2, m));
    }
    auto su = [](float v) {
      return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
    };
    tlo = make_float4(su(tlo.x), su(tlo.y), su(tlo.z), 0.f);
    thi = make_float4(su(thi.x), su(thi.y), su(thi.z), 0.f);
    hmax2 = su(hmax2);
    gh = su(gh);

    auto flush = [&](int nc) {
      {
        float4 vx = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
        float4 vc = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lane < nc) {
          vx = xm[cand];
          vc = ch[cand];
        }
        // a candidate beyond both the group's largest radius and its own h
        // fails every lane's symmetric test
        const float d2 = box_dist2(make_float3(vx.x, vx.y, vx.z), tlo, thi);
        const bool keep = lane < nc && (d2 < hmax2 || d2 < sq_exact(vc.x));
        const uint64_t km = __ballot(keep);
        const int slot = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
        if (keep) {
          // what depends on j alone, once a candidate: (x, fl(h^2)) and
          // (1/h, u, kappa, m/rho)
          T.xm[slot] = make_float4(vx.x, vx.y, vx.z, sq_exact(vc.x));
          T.ch[slot] = make_float4(1.0f / vc.x, vc.y, vc.z, vx.w * vc.w);
        }
        nc = __popcll(km);
      }
      wave_sync();
      float pu = 0.f;
      for (int k = 0; k < nc; ++k) {
        const float4 q = T.xm[k];
        const float4 qc = T.ch[k];
        const float dx = sub_exact(q.x, xi.x), dy = sub_exact(q.y, xi.y),
                    dz = sub_exact(q.z, xi.z);
        const float r2 = dist2_exact(dx, dy, dz);
        // r2 < fl(max(h_i, h_j)^2) as two compares (rounding is monotone)
        if (r2 < hi2 || r2 < q.w) {
          ++np;
          if (r2 > 0.0f) {
            const float r = r2 * __builtin_amdgcn_rsqf(r2);
            const float hj5 = (qc.x * qc.x) * (qc.x * qc.x) * qc.x;
            const float f = hi5 * wendland_f(r * hinvi) + hj5 * wendland_f(r * qc.x);
            pu += qc.w * (kappai + qc.z) * (ui - qc.y) * f;
          }
        }
      }
      neumaier_add(du, cdu, pu);
      wave_sync();
    };
    float sum[1] = {}, cmp[1] = {};
    if constexpr (kT > 1) {
      team_search<kT, kDeep>(
          tm, grp.snap, search, xi, hi, tlo, thi, gh,
          [](float h, float hmax) { return h > 0.0f ? sq_exact(fmaxf(h, hmax)) : -1.0f; },
          [&](int ntiles, int count) {
            for (int j = w; j < ntiles; j += kT) {
              const int nc = min(kTile, count - j * kTile);
              cand = lane < nc ? search.cand[j * kTile + lane] : 0;
              flush(nc);
            }
          });
      sum[0] = du;
      cmp[0] = cdu;
      team_totals<kT, 1, sizeof(CondTile) / 4>((float *)tiles, w, lane, sum, cmp);
      team_count<kT, sizeof(CondTile) / 4>((int *)tiles, w, lane, np);
    } else {
      int cur = grp.root, tc = 0;
      while (cur < grp.end) {
        const Node nd = nodes[cur];
        const bool want = hi > 0.0f && box_dist2(xi, nd.lo_h, nd.hi_l) <
                                           sq_exact(fmaxf(hi, nd.lo_h.w));
        if (__ballot(want) == 0ull) {
          cur = nd.meta.x;
          continue;
        }
        // a small subtree is taken whole: its members are one contiguous run
        if (!(nd.meta.w & kLeafBit) && nd.meta.z > walk_leaf) {
          ++cur;
          continue;
        }
        int st = nd.meta.y, c = nd.meta.z;
        while (c > 0) {
          const int take = min(c, kTile - tc);
          if (lane >= tc && lane < tc + take) cand = st + lane - tc;
          tc += take;
          st += take;
          c -= take;
          if (tc == kTile) {
            flush(kTile);
            tc = 0;
          }
        }
        cur = nd.meta.x;
      }
      if (tc > 0) flush(tc);
      sum[0] = du;
      cmp[0] = cdu;
    }
    // (a target without a pair at r > 0 has none also where its rho is 0)
    const float v = sum[0] + cmp[0], total = v == 0.0f ? v : v * (0.5f * kWendlandF * rinvi);
    if (valid && (kT == 1 || w == 0)) {
      const int cid = perm[s];
      if (dudt) dudt[cid] = total;
      if (npairs) npairs[cid] = np - 1;  // the self pair passes the test
    }
  }  // groups
}

inline unsigned nblk(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

hipError_t launch_conduction_prep(Octree &gas, const float *u, const void *h, int f64,
                                  const float *rho, float kappa0, float kappa_exp,
                                  float4 *ch, hipStream_t s) {
  if (gas.n == 0) return hipSuccess;
  if (f64)
    k_cond_prep<double><<<nblk(gas.n, 256), 256, 0, s>>>(
        gas.perm, gas.n, u, (const double *)h, rho, kappa0, kappa_exp, ch);
  else
    k_cond_prep<float><<<nblk(gas.n, 256), 256, 0, s>>>(
        gas.perm, gas.n, u, (const float *)h, rho, kappa0, kappa_exp, ch);
  return hipGetLastError();
}

hipError_t launch_conduction(const Octree &gas, const Groups &gs, int64_t max_groups,
                             int walk_leaf, const Terms &tm, int team, const float4 *ch,
                             float *dudt, int32_t *npairs, hipStream_t s) {
  if (max_groups <= 0 || gas.nnodes == 0) return hipSuccess;
  auto pick = [&](auto deep_c) {
    constexpr bool d = decltype(deep_c)::value;
    return team == 16  ? k_conduction<16, d>
           : team == 8 ? k_conduction<8, d>
           : team == 4 ? k_conduction<4, d>
           : team == 1 ? k_conduction<1>
                       : nullptr;
  };
  auto kern = tm.deep ? pick(std::true_type{}) : pick(std::false_type{});
  if (!kern) return hipErrorInvalidValue;  // (no such team)
  const int block = (team > 1 ? team : 4) * kWave;
  kern<<<persistent_grid((const void *)kern, block, max_groups, team), block, 0, s>>>(
      gas.nodes, gas.xm, ch, gas.perm, gs, walk_leaf, tm, dudt, npairs);
  return hipGetLastError();
}

}  // namespace g3
