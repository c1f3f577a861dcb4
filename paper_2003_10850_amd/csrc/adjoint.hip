// Adjoint (backward) kernels of the density, hydro force and gravity: the
// gradients of a scalar loss with respect to positions, masses, smoothing
// lengths (and the hydro inputs), given its gradients with respect to the
// module outputs at the active particles. Neighbour sets and Barnes-Hut
// decisions are those of the forward call (the forward map is piecewise
// smooth in them) and h is an input; the derivative through the h solve is
// the density adjoint with a seed derived from the solve's constraint.
//
// SPH adjoints are gathered: every gas particle walks its symmetric
// neighbourhood r < max(h_p, h_q) once and adds both what its own sums owe
// to its inputs and what its neighbours' sums owe to them, so each
// gradient is written by one lane in a fixed order (deterministic). The
// gravity adjoint is scattered: a wave sums the source-side terms of a tile
// entry over its lanes with DPP row operations and adds them with one
// atomic per entry, in 64-bit fixed point (integer additions commute, so
// the result does not depend on the order of the waves: deterministic); node
// adjoints are then pushed down to the members.
#include "g3_device.h"
#include "g3_internal.h"
#include "g3_items.h"
#include "g3_team.h"

namespace g3 {

namespace {

constexpr int kBlock = 256;
constexpr int kTile = kWave;
constexpr float kC = 6.7889530412636603f;  // 1365 / (64 pi)

inline unsigned nblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// Wendland C6 (support h, q = r/h) and the derivatives the adjoints need,
// each zero at and beyond the support:
//   W    = C/h^3 (1-q)^8 (1 + 8q + 25q^2 + 32q^3)
//   W_h  = dW/dh        = C/h^4 (1-q)^7 (-3 - 21q - 29q^2 + 133q^3 + 448q^4)
//   F    = (1/r) dW/dr  = -22 C/h^5 (1-q)^7 (1 + 7q + 16q^2)
//   G    = (1/r) dW_h/dr = dF/dh = 22 C/h^6 (1-q)^6 (5 + 30q + 21q^2 - 224q^3)
//   W_hh = d^2W/dh^2    = 6 C/h^5 (1-q)^6 (2 + 12q - 13q^2 - 218q^3 - 287q^4 + 1120q^5)
// An SPH sum's gradients weigh F and G together, W_h and W_hh, and W and W_h,
// each with the same two upstream factors (y, z); with the particle's powers
// of 1/h folded into four coefficients a pair needs only the polynomials:
//   y F  + z G    = t6 (f1 t p1 + f2 p2)
//   y W_h + z W_hh = t6 (e1 t p3 + e2 p4)
//   y W  + z W_h  = t7 (w1 t p5 + w2 p3)
struct WcCoef {
  float f1, f2, e1, e2, w1, w2;
};
__device__ __forceinline__ WcCoef wc6_coef(float y, float z, float hinv) {
  const float h2 = hinv * hinv, h3 = h2 * hinv, h4 = h2 * h2, h5 = h4 * hinv, h6 = h3 * h3;
  return {-22.0f * kC * h5 * y, 22.0f * kC * h6 * z, kC * h4 * y,
          6.0f * kC * h5 * z,   kC * h3 * y,         kC * h4 * z};
}
__device__ __forceinline__ float wc6_yf_zg(float q, float t, float t6, float f1, float f2) {
  return t6 * (f1 * t * (1.0f + q * (7.0f + q * 16.0f)) +
               f2 * (5.0f + q * (30.0f + q * (21.0f - q * 224.0f))));
}
__device__ __forceinline__ float wc6_wh_poly(float q) {
  return -3.0f + q * (-21.0f + q * (-29.0f + q * (133.0f + q * 448.0f)));
}
__device__ __forceinline__ float wc6_whh_poly(float q) {
  return 2.0f + q * (12.0f + q * (-13.0f + q * (-218.0f + q * (-287.0f + q * 1120.0f))));
}

// ---------------------------------------------------------------- density

// Upstream gradients of the density outputs folded into the two sums:
// Omega = 1 + h rho' / (3 rho) gives
//   gbar_rho  = g_rho  - g_omega h rho' / (3 rho^2)
//   gbar_rho' = g_rho' + g_omega h / (3 rho)
//   dL/dh    += g_omega rho' / (3 rho)        (the explicit h of Omega)
// written into bw[s] = (h, gbar_rho, gbar_rho', 1/h) at the active gas rows.
__global__ void k_density_bwd_prep(const int32_t *__restrict__ active, int64_t n_act,
                                   const int32_t *__restrict__ iperm, int64_t n_caller,
                                   const float *__restrict__ h, const float *__restrict__ rho,
                                   const float *__restrict__ drho, const float *__restrict__ g_rho,
                                   const float *__restrict__ g_drho,
                                   const float *__restrict__ g_omega, float4 *__restrict__ bw,
                                   float *__restrict__ g_h) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n_act) return;
  const int32_t id = active ? active[a] : (int32_t)a;
  if (id < 0 || (int64_t)id >= n_caller) return;
  const int32_t s = iperm[id];
  if (s < 0) return;
  const float hi = h[id], r = rho[id], rp = drho[id];
  const float go = g_omega ? g_omega[id] : 0.0f;
  const float gr = (g_rho ? g_rho[id] : 0.0f) - go * hi * rp / (3.0f * r * r);
  const float gd = (g_drho ? g_drho[id] : 0.0f) + go * hi / (3.0f * r);
  bw[s] = make_float4(hi, gr, gd, 1.0f / hi);
  if (g_h && go != 0.0f) g_h[id] += go * rp / (3.0f * r);
}

__global__ void k_density_bwd_init(const int32_t *__restrict__ perm, int64_t m,
                                   const float *__restrict__ h, float4 *__restrict__ bw) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const float hs = h[perm[s]];
  bw[s] = make_float4(hs, 0.0f, 0.0f, 1.0f / hs);
}

// Adjoint of the smoothing-length solve. Each active gas h_i is the root of
// F_i = N_eff(h_i) - N_ngb with N_eff = (4 pi/3) h^3 rho / m_i. By the
// implicit function theorem an upstream g_h_i reaches the positions and
// masses as the density adjoint seeded with
//   gbar_rho_i = -g_h_i h_i / (3 rho_i + h_i drho_i/dh)
// plus the explicit 1/m_i of N_eff:
//   dL/dm_i += g_h_i h_i rho_i / (m_i (3 rho_i + h_i drho_i/dh)).
// A row whose N_eff misses N_ngb by more than 1e-3 (relative: an h that did
// not converge, or one held at the cap) has no constraint and passes nothing.
__global__ void k_hsolve_bwd_prep(const int32_t *__restrict__ active, int64_t n_act,
                                  const int32_t *__restrict__ iperm, int64_t n_caller,
                                  const float *__restrict__ h, const float *__restrict__ rho,
                                  const float *__restrict__ drho, const float *__restrict__ g_h,
                                  const float4 *__restrict__ xm, float n_ngb,
                                  float4 *__restrict__ bw, float *__restrict__ g_mass) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n_act) return;
  const int32_t id = active ? active[a] : (int32_t)a;
  if (id < 0 || (int64_t)id >= n_caller) return;
  const int32_t s = iperm[id];
  if (s < 0) return;
  const float hi = h[id], r = rho[id], rp = drho[id], mi = xm[s].w, gh = g_h[id];
  const float N = 4.18879020f * hi * hi * hi * r / mi;  // (4 pi/3) h^3 rho / m
  const float den = 3.0f * r + hi * rp;                 // 3 rho Omega
  if (!(fabsf(N / n_ngb - 1.0f) <= 1e-3f) || !(den > 0.0f) || gh == 0.0f) return;
  bw[s] = make_float4(hi, -gh * hi / den, 0.0f, 1.0f / hi);
  if (g_mass) g_mass[id] += gh * hi * r / (mi * den);
}

// One lane per gas particle p, over every q with r < max(h_p, h_q):
//   own sums (r < h_p):  a = gbar_rho_p m_q F(r,h_p) + gbar_rho'_p m_q G(r,h_p)
//       dL/dx_p += a (x_p - x_q)
//       dL/dh_p += m_q (gbar_rho_p W_h(r,h_p) + gbar_rho'_p W_hh(r,h_p))
//   q's sums (r < h_q):  b = gbar_rho_q m_p F(r,h_q) + gbar_rho'_q m_p G(r,h_q)
//       dL/dx_p += b (x_p - x_q)
//       dL/dm_p += gbar_rho_q W(r,h_q) + gbar_rho'_q W_h(r,h_q)
// The pair q = p (r = 0) adds the self terms of h and m.
// A team of waves serves a group (g3_team.h); the tiles go to the waves in
// turn and the waves' totals are added in their order, so the gradients are
// the same on every run. 1.25e5 members of ~295 neighbours: 2886 us with one
// wave a group, 1179 with teams of 4, 1108 at 80 registers (6 waves a SIMD),
// 930 with the coefficients formed once a particle, 828 with teams of 8.
struct DTile {
  float4 x[kTile];  // position, mass
  float4 b[kTile];  // fl(h^2) or -1, 1/h, f1, f2
  float2 w[kTile];  // w1, w2
};
template <int kT, bool kDeep = false>
__global__ __launch_bounds__(kT * kWave, kT < 16 ? 6 : 1) void k_density_bwd(
    const float4 *__restrict__ xm, const float4 *__restrict__ bw,
    const int32_t *__restrict__ perm, const Groups gs, const Terms tm,
    float *__restrict__ g_pos, float *__restrict__ g_mass, float *__restrict__ g_h) {
  __shared__ TeamLds<kT> search;
  __shared__ DTile tiles[kT];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  float4 *tx = tiles[w].x, *tb = tiles[w].b;
  float2 *tw = tiles[w].w;
  int range = 0;
  for (int g; (g = team_next_group(gs, range, search)) >= 0;) {
    const Group grp = group_at(gs, g);
    const bool valid = lane < grp.count;
    const int s = valid ? grp.t0 + lane : grp.t0;
    const float4 me = xm[s], mb = bw[s];
    const float hp = valid ? mb.x : -1.0f;
    const float hp2 = sq_exact(hp), hinv = mb.w;
    const WcCoef kp = wc6_coef(mb.y, mb.z, hinv);
    const bool own_on = valid && (mb.y != 0.0f || mb.z != 0.0f);
    float sum[5] = {}, cmp[5] = {};  // position, mass, h
    int cand = 0;
    // the box of the group's particles and the largest radius of their own
    // sums: a candidate q whose box_dist2 to the box reaches that radius and
    // (when q's sums carry gradients) fl(h_q^2) meets no lane's test, since
    // box_dist2 never exceeds the r2 of a point inside the box
    float4 tlo = make_float4(valid ? me.x : INFINITY, valid ? me.y : INFINITY,
                             valid ? me.z : INFINITY, 0.f);
    float4 thi = make_float4(valid ? me.x : -INFINITY, valid ? me.y : -INFINITY,
                             valid ? me.z : -INFINITY, 0.f);
    // a member without h (or with a NaN) is still its neighbours' neighbour
    const float want = valid ? fmaxf(hp, 0.0f) : -1.0f;
    float hmax2 = own_on ? hp2 : -1.0f, hg = want;  // hg: the group's largest
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
      hg = fmaxf(hg, __shfl_xor(hg, m));
      tlo.x = fminf(tlo.x, __shfl_xor(tlo.x, m));
      tlo.y = fminf(tlo.y, __shfl_xor(tlo.y, m));
      tlo.z = fminf(tlo.z, __shfl_xor(tlo.z, m));
      thi.x = fmaxf(thi.x, __shfl_xor(thi.x, m));
      thi.y = fmaxf(thi.y, __shfl_xor(thi.y, m));
      thi.z = fmaxf(thi.z, __shfl_xor(thi.z, m));
      hmax2 = fmaxf(hmax2, __shfl_xor(hmax2, m));
    }
    {
      auto su = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
      tlo = make_float4(su(tlo.x), su(tlo.y), su(tlo.z), 0.f);
      thi = make_float4(su(thi.x), su(thi.y), su(thi.z), 0.f);
      hmax2 = su(hmax2);
      hg = su(hg);
    }
    auto flush = [&](int nc) {
      {
        float4 vx = make_float4(INFINITY, INFINITY, INFINITY, 0.f), vb = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lane < nc) {
          vx = xm[cand];
          vb = bw[cand];
        }
        const float d2 = box_dist2(make_float3(vx.x, vx.y, vx.z), tlo, thi);
        const bool on = vb.y != 0.0f || vb.z != 0.0f;
        const bool keep = lane < nc && (d2 < hmax2 || (on && d2 < sq_exact(vb.x)));
        const uint64_t km = __ballot(keep);
        const int slot = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
        // kept candidates in their order at the front; the scan stops at nc
        if (keep) {
          const WcCoef kq = wc6_coef(vb.y, vb.z, vb.w);
          tx[slot] = vx;
          tb[slot] = make_float4(on ? sq_exact(vb.x) : -1.0f, vb.w, kq.f1, kq.f2);
          tw[slot] = make_float2(kq.w1, kq.w2);
        }
        nc = __popcll(km);
      }
      wave_sync();
      float px = 0.f, py = 0.f, pz = 0.f, pm = 0.f, ph = 0.f;
      for (int k = 0; k < nc; ++k) {
        const float4 q = tx[k], qb = tb[k];
        const float dx = sub_exact(q.x, me.x), dy = sub_exact(q.y, me.y),
                    dz = sub_exact(q.z, me.z);
        const float r2 = dist2_exact(dx, dy, dz);
        const bool own = own_on && r2 < hp2;
        const bool nbr = valid && r2 < qb.x;
        if (own || nbr) {
          const float r = __builtin_amdgcn_sqrtf(r2);
          float a = 0.0f;
          if (own) {
            const float u = r * hinv, v = fmaxf(1.0f - u, 0.0f), v3 = v * v * v, v6 = v3 * v3;
            a = q.w * wc6_yf_zg(u, v, v6, kp.f1, kp.f2);
            ph += q.w * v6 * (kp.e1 * v * wc6_wh_poly(u) + kp.e2 * wc6_whh_poly(u));
          }
          if (nbr) {
            const float2 qw = tw[k];
            const float u = r * qb.y, v = fmaxf(1.0f - u, 0.0f), v3 = v * v * v, v6 = v3 * v3;
            a += me.w * wc6_yf_zg(u, v, v6, qb.z, qb.w);
            pm += v6 * v * (qw.x * v * (1.0f + u * (8.0f + u * (25.0f + u * 32.0f))) +
                            qw.y * wc6_wh_poly(u));
          }
          // x_p - x_q = -(dx, dy, dz)
          px -= a * dx;
          py -= a * dy;
          pz -= a * dz;
        }
      }
      neumaier_add(sum[0], cmp[0], px);
      neumaier_add(sum[1], cmp[1], py);
      neumaier_add(sum[2], cmp[2], pz);
      neumaier_add(sum[3], cmp[3], pm);
      neumaier_add(sum[4], cmp[4], ph);
      wave_sync();
    };
    team_search<kT, kDeep>(
        tm, grp.snap, search, make_float3(me.x, me.y, me.z), want, tlo, thi, hg,
        [](float h, float hmax) { return h < 0.0f ? -1.0f : sq_exact(fmaxf(h, hmax)); },
        [&](int ntiles, int count) {
          for (int j = w; j < ntiles; j += kT) {
            const int nc = min(kTile, count - j * kTile);
            cand = lane < nc ? search.cand[j * kTile + lane] : 0;
            flush(nc);
          }
        });
    team_totals<kT, 5, sizeof(DTile) / 4>((float *)tiles, w, lane, sum, cmp);
    if (valid && w == 0) {
      const int cid = perm[s];
      if (g_pos) {
        g_pos[3 * cid] += sum[0] + cmp[0];
        g_pos[3 * cid + 1] += sum[1] + cmp[1];
        g_pos[3 * cid + 2] += sum[2] + cmp[2];
      }
      if (g_mass) g_mass[cid] += sum[3] + cmp[3];
      if (g_h) g_h[cid] += sum[4] + cmp[4];
    }
  }
}

// ---------------------------------------------------------------- gravity

// v from the lane paired with this one by a DPP permutation (every lane
// active, every lane a source)
template <int kCtrl>
__device__ __forceinline__ float dpp_from(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf,
                                                    false));
}

// Sums over the 64 lanes of v[0..15], spread so that lane l ends with the
// total of value (l >> 2) & 15, by recursive halving: at each of four steps
// the lanes pair off across one lane bit (5, 4, 3, 2), and each keeps the
// half of its values that its bit selects plus its partner's copy of that
// half; two pairwise exchanges (bits 1, 0) then complete the quads' sums.
// Bits 5 and 4 by the half-wave and row swaps (one swap serves both
// partners), then the DPP row mirror (xor 15), half-row mirror (xor 7) and
// the quad permutations xor 3, xor 1; each pairs lanes that differ in the
// step's bit and agree in the bits above it. Every lane must be active.
__device__ __forceinline__ float wave_reduce_scatter16(float (&v)[16], int lane) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    // (a.lo, b.lo) and (a.hi, b.hi) of a = v[i], b = v[i + 8]
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]),
                                                    __float_as_uint(v[i + 8]), false, false);
    v[i] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]),
                                                    __float_as_uint(v[i + 4]), false, false);
    v[i] = __uint_as_float(p[0]) + __uint_as_float(p[1]);
  }
  {
    const bool up = (lane & 8) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float send = up ? v[i] : v[i + 2];
      const float keep = up ? v[i + 2] : v[i];
      v[i] = keep + dpp_from<0x140>(send);  // row mirror: lane ^ 15 in its row
    }
  }
  {
    const bool up = (lane & 4) != 0;
    const float send = up ? v[0] : v[1];
    const float keep = up ? v[1] : v[0];
    v[0] = keep + dpp_from<0x141>(send);  // half-row mirror: lane ^ 7
  }
  v[0] += dpp_from<0x1b>(v[0]);  // quad permutation (3, 2, 1, 0): lane ^ 3
  v[0] += dpp_from<0xb1>(v[0]);  // quad permutation (1, 0, 3, 2): lane ^ 1
  return v[0];
}

// Deterministic accumulation of the gravity adjoint's scattered sums. Every
// value v is added as two 64-bit integers, hi = trunc(v 2^F) and
// lo = rint((v 2^F - hi) 2^kFxLoBits), to a pair of counters: integer
// addition is exact and commutes, so the totals do not depend on the order
// in which waves add them. F is one per call, taken from a bound B on every
// counter's partial sums (|sum hi| <= B 2^F <= 2^62): with S = r^2 + eps^2 >=
// eps^2, a term's position part is at most G m (4 |g_a| S^-3/2 + |g_phi|
// S^-1) and its mass part G (|g_a| S^-1 + |g_phi| S^-1/2), |g_a| <= sqrt(3)
// times the largest upstream component, m at most n times the largest mass
// (a node), and a counter takes at most n_act such terms from the source
// side and at most n from its own target side. The overestimate (many
// orders of magnitude) costs nothing: the low counter resolves 2^-(62 + 36)
// of B, about 2^-30 of the largest true total even at 2e7 particles, far
// below the FP32 rounding of the terms; lo stays below 2^63 for up to 2^26
// additions per counter. Needs eps > 0 (else no such bound: FP32 atomics).
constexpr int kFxLoBits = 36;

// The scale 2^F from the device maxima (float bits) of the upstream
// gradient components, the upstream potential gradients and the masses.
__device__ __forceinline__ double fx_scale(const unsigned *__restrict__ mx, float eps2, float G,
                                           int64_t n, int64_t n_act) {
  const double ga = 1.7320508075688772 * (double)__uint_as_float(mx[0]);
  const double gp = (double)__uint_as_float(mx[1]);
  const double mm = (double)__uint_as_float(mx[2]);
  const double e2 = (double)eps2, e1 = sqrt(e2);
  const double T = 4.0 * ga / (e2 * e1) + gp / e2 + ga / e2 + gp / e1;
  const double B = 2.0 * fabs((double)G) * T * ((double)n * mm + 1.0) *
                   ((double)n + (double)n_act + 1.0);
  // (no finite bound, from non-finite inputs: any scale; the sums are then
  // as meaningless as the inputs)
  const int F = (B > 0.0 && B < 1e300) ? 62 - (ilogb(B) + 1) : 0;
  return ldexp(1.0, F);
}

__device__ __forceinline__ void fx_add(unsigned long long *dst, float v, double scale) {
  const double d = (double)v * scale;
  const double hi = trunc(d);  // d - hi is exact
  const long long lo = (long long)rint((d - hi) * (double)(1ll << kFxLoBits));
  atomicAdd(dst, (unsigned long long)(long long)hi);
  atomicAdd(dst + 1, (unsigned long long)lo);
}

// The largest |upstream gradient component|, |upstream potential gradient|
// (over the active rows; ids outside [0, m) are skipped, as by the walk) and
// mass (over every member), as float bits into mx[0..2] (zero on entry).
constexpr int kFxBoundBlocks = 1024;
__global__ __launch_bounds__(kBlock) void k_fx_bound(
    const int32_t *__restrict__ active, int64_t n_act, const float *__restrict__ g_acc,
    const float *__restrict__ g_pot, const float4 *__restrict__ xm, int64_t m,
    unsigned *__restrict__ mx) {
  // a grid-stride pass, then one atomic per block and value (one per wave
  // on three words had serialised)
  __shared__ float part[3][kBlock / kWave];
  float a = 0.0f, p = 0.0f, w = 0.0f;
  const int64_t n = n_act > m ? n_act : m;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t id = i < n_act ? (active ? active[i] : i) : -1;
    if (id >= 0 && id < m) {
      if (g_acc)
        a = fmaxf(a, fmaxf(fabsf(g_acc[3 * id]),
                           fmaxf(fabsf(g_acc[3 * id + 1]), fabsf(g_acc[3 * id + 2]))));
      if (g_pot) p = fmaxf(p, fabsf(g_pot[id]));
    }
    if (i < m) w = fmaxf(w, fabsf(xm[i].w));
  }
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) {
    a = fmaxf(a, __shfl_xor(a, k));
    p = fmaxf(p, __shfl_xor(p, k));
    w = fmaxf(w, __shfl_xor(w, k));
  }
  const int wv = (int)(threadIdx.x >> 6);
  if ((threadIdx.x & 63u) == 0u) {
    part[0][wv] = a;
    part[1][wv] = p;
    part[2][wv] = w;
  }
  __syncthreads();
  if (threadIdx.x < 3u) {
    float v = part[threadIdx.x][0];
    for (int k = 1; k < kBlock / kWave; ++k) v = fmaxf(v, part[threadIdx.x][k]);
    atomicMax(&mx[threadIdx.x], __float_as_uint(v));
  }
}

// Fixed-point counter pairs (hi, lo) x 4 components back to float4.
__global__ void k_fx_to_f4(const unsigned long long *__restrict__ fx, int64_t m,
                           const unsigned *__restrict__ mx, float eps2, float G, int64_t n,
                           int64_t n_act, float4 *__restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const double inv = 1.0 / fx_scale(mx, eps2, G, n, n_act);
  double v[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const long long hi = (long long)fx[8 * i + 2 * c], lo = (long long)fx[8 * i + 2 * c + 1];
    v[c] = ((double)hi + ldexp((double)lo, -kFxLoBits)) * inv;
  }
  out[i] = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
}

struct __align__(16) GEntry {
  float4 p;   // source position, mass
  int4 meta;  // sorted source index, or -(node + 1); mask low, mask high; unused
};
// a lane's mask word: meta.y (lanes 0..31) or meta.z (lanes 32..63), the
// 32-bit words 5 and 6 of an entry
constexpr int kGMaskWord = 5;

__device__ __forceinline__ bool open_accept(float l, float theta2, float r2) {
#pragma clang fp contract(off)
  const float lhs = l * l;
  const float rhs = theta2 * r2;
  return lhs < rhs;
}

// The Barnes-Hut walk of the forward kernel by teams (g3_items.h); what a wave
// accepts waits in its own tile of 64 entries. Each term of target i with
// source s (x = x_i - x_s, S = r^2 + eps^2) and upstream gradients
// (ga, gp) of a_i and phi_i contributes
//   dL/dx  = G m ( -ga / S^(3/2) + 3 (ga . x) x / S^(5/2) + gp x / S^(3/2) )
//   dL/dx_i += dL/dx,  dL/dx_s -= dL/dx,  dL/dm_s = -G ((ga . x) / S^(3/2) + gp / S^(1/2)).
// The source side of a tile entry is summed over the wave's lanes and added
// once: to the particle's sorted slot, or to the node's (dL/dc, dL/dM).
// kFixed: the sums go to fixed-point counter pairs (gsrc_fx [n][4][2],
// gnode_fx [nnodes][4][2], scale from mx), else to FP32 atomics (gsrc,
// gnode).
// Bound by vector issue: about 65 instructions an entry, 10 of them the
// reduction (16 and three LDS permutes before the half-wave swaps; sums by
// the matrix cores, one-hot rows times the values, came to 4.8 ms, the FP32
// products do not overlap), 3 the fixed-point conversion of 16 entries at
// once; the atomics cost 0.3 ms. 5e5 targets of a clustered box: 3.6 ms with one
// wave a group, 3.4 with teams of 4; 2^22: 24.5 and 27.6 (24.6 with the preorder
// walk before the items); 2^14 targets: 1.5 and 0.23 with teams of 16.
template <bool kFixed, bool kInside, int kT>
__global__ __launch_bounds__(kT * kWave, kT < 16 ? 6 : 1) void k_gravity_bwd(
    const CNode *__restrict__ cnodes, const uint64_t *__restrict__ ckeys,
    const float4 *__restrict__ xm, const uint64_t *__restrict__ keys, const int32_t *__restrict__ perm, const Groups gs,
    float theta2, float eps2, float G, const float *__restrict__ g_acc,
    const float *__restrict__ g_pot, float4 *__restrict__ gsrc, float4 *__restrict__ gnode,
    unsigned long long *__restrict__ gsrc_fx, unsigned long long *__restrict__ gnode_fx,
    const unsigned *__restrict__ mx, int64_t n_all, int64_t n_act) {
  __shared__ Team<kT> S;
  __shared__ GEntry tiles[kT][kTile];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  GEntry *tile = tiles[w];
  const double scale = kFixed ? fx_scale(mx, eps2, G, n_all, n_act) : 1.0;
  int range = 0;
  for (int g; (g = team_take_group(gs, range, S)) >= 0;) {
    const Group grp = group_at(gs, g);
    const int64_t t = grp.t0 + lane;
    const bool valid = lane < grp.count;
    const int s = valid ? (gs.targets ? gs.targets[t] : (int)t) : 0;
    const float4 me = xm[s];
    const uint64_t ki = keys[s];
    const int cid = perm[s];
    const float gax = valid && g_acc ? g_acc[3 * cid] : 0.f;
    const float gay = valid && g_acc ? g_acc[3 * cid + 1] : 0.f;
    const float gaz = valid && g_acc ? g_acc[3 * cid + 2] : 0.f;
    const float gpp = valid && g_pot ? g_pot[cid] : 0.f;
    float ox = 0.f, oy = 0.f, oz = 0.f, cox = 0.f, coy = 0.f, coz = 0.f;
    int tc = 0;
    const bool hiword = lane >= 32;
    const uint32_t bitpos = (uint32_t)lane & 31u;
    const uint32_t *maskw = (const uint32_t *)tile + kGMaskWord + (hiword ? 1 : 0);
    auto flush = [&](int nc) {
      // padded to a multiple of four with entries no lane uses
      const int n4 = (nc + 3) & ~3;
      if (lane >= nc && lane < n4) {
        tile[lane].p = make_float4(0.f, 0.f, 0.f, 0.f);
        tile[lane].meta = make_int4(0, 0, 0, 0);
      }
      wave_sync();
      float px = 0.f, py = 0.f, pz = 0.f;
      // sixteen entries a round: after their four sums every lane holds one
      // total, of entry k0 + 4 (lane & 3) + (lane >> 4)
      for (int k0 = 0; k0 < n4; k0 += 16) {
        float tot = 0.0f;
#pragma unroll 1
        for (int q = 0; q < 4 && k0 + 4 * q < n4; ++q) {
          // the source sides of four entries without the factor G:
          // (-dL/dx_i, dL/dm_s) per entry
          float v[16];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int k = k0 + 4 * q + e;
            const float4 ep = tile[k].p;
            // 0 or all ones: the lane's bit (its own target's bit is clear)
            const int32_t use = __builtin_amdgcn_sbfe(
                (int32_t)maskw[k * (int)(sizeof(GEntry) / 4)], bitpos, 1u);
            const float dx = ep.x - me.x, dy = ep.y - me.y, dz = ep.z - me.z;  // x_s - x_i
            const float S =
                __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, __builtin_fmaf(dx, dx, eps2)));
            // masked here, so that an unused entry adds exact zeros even at S = 0
            const float inv = __int_as_float(__float_as_int(__builtin_amdgcn_rsqf(S)) & use);
            const float inv2 = inv * inv, inv3 = inv2 * inv;
            const float gd = gax * dx + gay * dy + gaz * dz;  // -ga . x, x = x_i - x_s
            const float m3 = ep.w * inv3;
            // dL/dx = -m3 ga - c (dx, dy, dz), x = -(dx, dy, dz)
            const float c = m3 * (gpp - 3.0f * gd * inv2);
            const float Dx = m3 * gax + c * dx, Dy = m3 * gay + c * dy, Dz = m3 * gaz + c * dz;
            px -= Dx;
            py -= Dy;
            pz -= Dz;
            v[4 * e] = Dx;
            v[4 * e + 1] = Dy;
            v[4 * e + 2] = Dz;
            v[4 * e + 3] = gd * inv3 - gpp * inv;
          }
          // lane l holds the wave's total of entry l >> 4, component (l >> 2) & 3
          const float sum = wave_reduce_scatter16(v, lane);
          tot = (lane & 3) == q ? sum : tot;
        }
        const int k = k0 + 4 * (lane & 3) + (lane >> 4), comp = (lane >> 2) & 3;
        if (k < nc) {
          const int src = tile[k].meta.x;
          if constexpr (kFixed) {
            unsigned long long *dst = src >= 0 ? gsrc_fx + 8 * (int64_t)src
                                               : gnode_fx + 8 * (int64_t)(-src - 1);
            fx_add(dst + 2 * comp, G * tot, scale);
          } else {
            float *dst = src >= 0 ? (float *)&gsrc[src] : (float *)&gnode[-src - 1];
            atomicAdd(dst + comp, G * tot);
          }
        }
      }
      neumaier_add(ox, cox, px);
      neumaier_add(oy, coy, py);
      neumaier_add(oz, coz, pz);
      wave_sync();
    };
    // the walk of the forward kernel: the same items, decisions and masks
    const int root_exp = ilogbf((float)gs.sbox[grp.snap].w);
    const int root = __builtin_amdgcn_readfirstlane(grp.snap);
    const uint64_t all = grp.count < kWave ? (1ull << grp.count) - 1ull : ~0ull;
    team_items(S, root, all, w, lane, [&](int first, int count, uint64_t mask, const auto &opened) {
      const bool act = __builtin_amdgcn_inverse_ballot_w64(mask);
      if (count > 0) {
        auto visit = [&](const CNode &nd, uint64_t nk) {
          const float l = __int_as_float(nd.meta.w);
          const float r2 = dist2_exact(sub_exact(nd.com_m.x, me.x), sub_exact(nd.com_m.y, me.y),
                                       sub_exact(nd.com_m.z, me.z));
          bool accept, open;
          if constexpr (!kInside) {
            float rhs;
            {
#pragma clang fp contract(off)
              rhs = theta2 * r2;
            }
            const float lhs = sq_exact(l);
            accept = act && lhs < rhs;
            open = act && lhs >= rhs;
          } else {
            const int level = root_exp - ilogbf(l);
            accept = act && open_accept(l, theta2, r2) &&
                     ((ki ^ nk) >> (3 * (kMaxLevel - level))) != 0ull;
            open = act && !accept;
          }
          const uint64_t amask = __ballot(accept), om = __ballot(open);
          if (amask) {
            tc = __builtin_amdgcn_readfirstlane(tc);
            if (tc == kTile) {
              flush(kTile);
              tc = 0;
            }
            if (lane == 0) {
              GEntry e;
              e.p = nd.com_m;
              e.meta = make_int4(-(nd.meta.z + 1), (int)(uint32_t)amask,
                                 (int)(uint32_t)(amask >> 32), 0);
              tile[tc] = e;
            }
            ++tc;
          }
          if (om) opened(nd.meta.x, nd.meta.y, om);
        };
        for (int c = 0; c < count; ++c)
          visit(cnodes[first + c], kInside ? ckeys[first + c] : 0ull);
      } else {
        int st = first, c = -count;
        while (c > 0) {
          tc = __builtin_amdgcn_readfirstlane(tc);
          if (tc == kTile) {
            flush(kTile);
            tc = 0;
          }
          const int take = min(c, kTile - tc);
          if (lane < take) {
            GEntry e;
            e.p = xm[st + lane];
            e.meta = make_int4(st + lane, (int)(uint32_t)mask, (int)(uint32_t)(mask >> 32), 0);
            tile[tc + lane] = e;
          }
          wave_sync();
          // an opening lane whose own target is among these members clears
          // its bit in that member's entry (one lane per entry)
          const int rel = s - st;
          if (act && rel >= 0 && rel < take) {
            uint32_t *wd = (uint32_t *)&tile[tc + rel] + kGMaskWord + (hiword ? 1 : 0);
            *wd &= ~(1u << bitpos);
          }
          tc += take;
          st += take;
          c -= take;
        }
      }
    });
    if (tc > 0) flush(tc);
    if (valid) {
      if constexpr (kFixed) {
        fx_add(gsrc_fx + 8 * (int64_t)s, G * (ox + cox), scale);
        fx_add(gsrc_fx + 8 * (int64_t)s + 2, G * (oy + coy), scale);
        fx_add(gsrc_fx + 8 * (int64_t)s + 4, G * (oz + coz), scale);
      } else {
        atomicAdd(&gsrc[s].x, G * (ox + cox));
        atomicAdd(&gsrc[s].y, G * (oy + coy));
        atomicAdd(&gsrc[s].z, G * (oz + coz));
      }
    }
  }
}

__global__ void k_zero_f4(float4 *__restrict__ p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Node adjoints (dL/dc, dL/dM) to the members. With c = sum m x / M and
// M = sum m, a member k of node a receives (m_k / M_a) dL/dc_a on x_k and
// dL/dM_a + dL/dc_a . (x_k - c_a) / M_a on m_k. Summed over the ancestors of
// k's leaf l, top-down in FP64:
//   P_n = sum_a dL/dc_a / M_a,  Q_n = sum_a dL/dM_a,
//   R_n = sum_a dL/dc_a . (c_n - c_a) / M_a = R_parent + P_parent . (c_n - c_parent)
// and then x_k gets m_k P_l, m_k gets Q_l + R_l + P_l . (x_k - c_l).
__global__ void k_push_init(const float4 *__restrict__ gnode, const double4 *__restrict__ mom,
                            int64_t nn, double4 *__restrict__ pq, double *__restrict__ rr) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nn) return;
  const float4 g = gnode[k];
  const double M = mom[k].x;
  const double inv = M > 0.0 ? 1.0 / M : 0.0;
  pq[k] = make_double4(g.x * inv, g.y * inv, g.z * inv, (double)g.w);
  rr[k] = 0.0;
}

__global__ void k_push_level(const Node *__restrict__ nodes, const double4 *__restrict__ mom,
                             int64_t nn, int level, double4 *__restrict__ pq,
                             double *__restrict__ rr) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nn) return;
  const int4 meta = nodes[k].meta;
  if ((meta.w & 255) != level || (meta.w & kLeafBit)) return;
  const double4 P = pq[k];
  const double R = rr[k];
  const double4 mk = mom[k];
  const double ik = mk.x > 0.0 ? 1.0 / mk.x : 0.0;
  const double cx = mk.y * ik, cy = mk.z * ik, cz = mk.w * ik;
  int64_t c = k + 1;
  while (c < meta.x) {
    const double4 mc = mom[c];
    const double ic = mc.x > 0.0 ? 1.0 / mc.x : 0.0;
    double4 q = pq[c];
    q.x += P.x;
    q.y += P.y;
    q.z += P.z;
    q.w += P.w;
    pq[c] = q;
    rr[c] = R + P.x * (mc.y * ic - cx) + P.y * (mc.z * ic - cy) + P.z * (mc.w * ic - cz);
    c = nodes[c].meta.x;
  }
}

__global__ void k_push_leaves(const Node *__restrict__ nodes, const double4 *__restrict__ mom,
                              int64_t nn, const float4 *__restrict__ xm,
                              const double4 *__restrict__ pq, const double *__restrict__ rr,
                              float4 *__restrict__ gsrc) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nn) return;
  const int4 meta = nodes[k].meta;
  if (!(meta.w & kLeafBit)) return;
  const double4 P = pq[k];
  const double R = rr[k];
  const double4 mk = mom[k];
  const double ik = mk.x > 0.0 ? 1.0 / mk.x : 0.0;
  const double cx = mk.y * ik, cy = mk.z * ik, cz = mk.w * ik;
  for (int s = meta.y; s < meta.y + meta.z; ++s) {
    const float4 p = xm[s];
    float4 g = gsrc[s];
    g.x += (float)(p.w * P.x);
    g.y += (float)(p.w * P.y);
    g.z += (float)(p.w * P.z);
    g.w += (float)(P.w + R + P.x * (p.x - cx) + P.y * (p.y - cy) + P.z * (p.z - cz));
    gsrc[s] = g;
  }
}

__global__ void k_scatter_grad(const int32_t *__restrict__ perm, int64_t m,
                               const float4 *__restrict__ gsrc, float *__restrict__ g_pos,
                               float *__restrict__ g_mass) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const int cid = perm[s];
  const float4 g = gsrc[s];
  if (g_pos) {
    g_pos[3 * cid] += g.x;
    g_pos[3 * cid + 1] += g.y;
    g_pos[3 * cid + 2] += g.z;
  }
  if (g_mass) g_mass[cid] += g.w;
}

// ------------------------------------------------------------------ hydro

// F = (1/r) dW/dr and its derivatives dF/dr, dF/dh (= G above):
//   F_r = 528 C/h^6 q (1-q)^6 (1 + 6q)
__device__ __forceinline__ void wc6_f_derivs(float r, float hinv, float &F, float &Fr,
                                             float &Fh) {
  const float q = r * hinv;
  const float t = fmaxf(1.0f - q, 0.0f);
  const float t2 = t * t, t3 = t2 * t, t6 = t3 * t3;
  const float h2 = hinv * hinv, h5 = h2 * h2 * hinv, h6 = h5 * hinv;
  F = -22.0f * kC * h5 * t6 * t * (1.0f + q * (7.0f + q * 16.0f));
  Fr = 528.0f * kC * h6 * t6 * q * (1.0f + 6.0f * q);
  Fh = 22.0f * kC * h6 * t6 * (5.0f + q * (30.0f + q * (21.0f - q * 224.0f)));
}

// One side of a particle's hydro data: position and mass, velocity and h,
// (A, c, rho, 1/h), and the upstream gradients (g_acc, g_dudt) of its sums.
struct HSide {
  float4 xm, vh, aux, up;
};
// A tile of them, array by array: (x, y, z, fl(h^2)), which is all that the
// neighbour test reads, (v, m), aux and up.
struct HSides {
  float4 xh[kTile], vm[kTile], aux[kTile], up[kTile];
};

// What one particle p of a pair is owed: by the pair term whose target is p,
// and by the one whose target is its neighbour q. A term with target i and
// neighbour j is
//   l = g_acc_i . a_ij + g_dudt_i du_ij,
//   a_ij  = -m_j (A_i g_i + A_j g_j + Pi gbar) x,   x = x_i - x_j, v = v_i - v_j
//   du_ij = m_j (A_i g_i + Pi gbar / 2) v.x,        g_k = F(r, h_k), gbar = (g_i + g_j)/2
//   Pi = -alpha (c_i + c_j - 3w) w / (rho_i + rho_j) if w = v.x / r < 0, else 0.
// d[0..2] position, d[3..5] velocity, d[6] h, d[7] A, d[8] c, d[9] rho
// through Pi, d[10] m. The chain rules used:
//   dl/dx = coef g_acc + L_vx v + (L_r / r) x,  dl/dv = L_vx x,
//   L_vx = dl/dvx + dl/dPi dPi/dw / r,  L_r = sum_k dl/dg_k F_r(r,h_k) - dl/dPi dPi/dw w / r.
// v.x, w, Pi and the kernel factors are the same in both terms (x and v change
// sign together) and are formed once; with x = x_p - x_q throughout, the
// second term's position and velocity partials take the sign of its neighbour
// side.
__device__ __forceinline__ void hydro_pair_adjoint(const HSide &P, const HSide &Q, float alpha,
                                                   bool p_on, bool q_on, float dx, float dy,
                                                   float dz, float r2, float *d) {
  const float rinv = __builtin_amdgcn_rsqf(r2), r = r2 * rinv;
  const float vxx = P.vh.x - Q.vh.x, vyy = P.vh.y - Q.vh.y, vzz = P.vh.z - Q.vh.z;
  const float vx = vxx * dx + vyy * dy + vzz * dz;
  const float w = vx * rinv;
  float gp, gpr, gph, gq, gqr, gqh;
  wc6_f_derivs(r, P.aux.w, gp, gpr, gph);
  wc6_f_derivs(r, Q.aux.w, gq, gqr, gqh);
  const float csum = P.aux.y + Q.aux.y;
  const float rs = 1.0f / (P.aux.z + Q.aux.z), ar = alpha * rs;
  const bool neg = w < 0.0f;
  const float Pi = neg ? -ar * (csum - 3.0f * w) * w : 0.0f;
  const float Pw = neg ? -ar * (csum - 6.0f * w) : 0.0f;
  const float Pc = neg ? -ar * w : 0.0f;
  const float gbar = 0.5f * (gp + gq);
  const float Tp = P.aux.x * gp, Tq = Q.aux.x * gq, V = Pi * gbar;
  const float K = Tp + Tq + V;
  const float mp = P.xm.w, mq = Q.xm.w;
  // target p: sdot = g_acc_p . x; target q: its x is -x
  const float sp = P.up.x * dx + P.up.y * dy + P.up.z * dz;
  const float sq = -(Q.up.x * dx + Q.up.y * dy + Q.up.z * dz);
  const float vp = P.up.w * vx, vq = Q.up.w * vx;  // g_dudt v.x
  const float bp = mq * (0.5f * vp - sp), bq = mp * (0.5f * vq - sq);
  const float ep = mq * (vp - sp), eq = mp * (vq - sq);
  const float b = bp + bq, dPi = b * gbar, hb = 0.5f * b * Pi;
  // dl/dg_p and dl/dg_q over both terms
  const float dgp = P.aux.x * (ep - mp * sq) + hb;
  const float dgq = Q.aux.x * (eq - mq * sp) + hb;
  const float dPw = dPi * Pw;
  // (a side without upstream gradients adds nothing, not 0 times its factors)
  const float tp = p_on ? mq * P.up.w * (Tp + 0.5f * V) : 0.0f;
  const float tq = q_on ? mp * Q.up.w * (Tq + 0.5f * V) : 0.0f;
  const float Lvx = tp + tq + dPw * rinv;
  const float lr = (dgp * gpr + dgq * gqr - dPw * w * rinv) * rinv;
  const float cp = p_on ? -mq * K : 0.0f, cq = q_on ? mp * K : 0.0f;
  d[0] += cp * P.up.x + cq * Q.up.x + Lvx * vxx + lr * dx;
  d[1] += cp * P.up.y + cq * Q.up.y + Lvx * vyy + lr * dy;
  d[2] += cp * P.up.z + cq * Q.up.z + Lvx * vzz + lr * dz;
  d[3] += Lvx * dx;
  d[4] += Lvx * dy;
  d[5] += Lvx * dz;
  d[6] += dgp * gph;
  d[7] += gp * (ep - mp * sq);
  d[8] += dPi * Pc;
  d[9] -= neg ? dPi * Pi * rs : 0.0f;
  if (q_on) d[10] += vq * (Tq + 0.5f * V) - K * sq;
}

__global__ void k_hydro_bwd_up(const int32_t *__restrict__ active, int64_t n_act,
                               const int32_t *__restrict__ iperm, int64_t n_caller,
                               const float *__restrict__ g_acc, const float *__restrict__ g_dudt,
                               float4 *__restrict__ up) {
  const int64_t a = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (a >= n_act) return;
  const int32_t id = active ? active[a] : (int32_t)a;
  if (id < 0 || (int64_t)id >= n_caller) return;
  const int32_t s = iperm[id];
  if (s < 0) return;
  up[s] = make_float4(g_acc ? g_acc[3 * id] : 0.f, g_acc ? g_acc[3 * id + 1] : 0.f,
                      g_acc ? g_acc[3 * id + 2] : 0.f, g_dudt ? g_dudt[id] : 0.f);
}

// One lane per gas particle p over every q != p with r < max(h_p, h_q):
// the pair (target p, neighbour q) if p is active, and (target q,
// neighbour p) if q is active. Then A and c are mapped back to u, rho and
// Omega: A = (gamma-1) u / (Omega rho), c = sqrt(gamma (gamma-1) u).
// Bound by VALU issue (a pair is ~150 operations); 128 registers, four waves
// a SIMD. Teams as in the density's adjoint. 1.25e5 particles of
// ~295 neighbours: 10671 us with one wave a group and the two terms of a pair
// by themselves; 1678 with teams of 4, 1430 of 8.
// A lane is a neighbour of a quarter of the entries that any lane neighbours, so
// the pairs are not taken entry by entry: the tests give each lane a bit mask of
// the tile, and the lanes take their own entries side by side, as many steps as
// the busiest lane has. Neighbours in tree order come in runs that one lane takes
// whole; a tile therefore holds every ntiles-th candidate of a round, which needs
// 0.5 to 0.66 of the steps, against 0.9 with consecutive ones. Density and force
// with gradients, entry by entry and so: 710 and 696 us at 3000 particles, 3390 and
// 3240 at 6e4, 5790 and 5180 at 2.5e5, 8160 and 7365 at 5e5 (5400 and 7360 with
// three waves a SIMD and 146 registers, nothing spilled).
template <int kT, bool kDeep = false>
__global__ __launch_bounds__(kT * kWave, kT < 16 ? 4 : 1) void k_hydro_bwd(
    const float4 *__restrict__ xm, const float4 *__restrict__ vh,
    const float4 *__restrict__ aux, const float4 *__restrict__ up,
    const int32_t *__restrict__ perm, const Groups gs, const Terms tm, float alpha, float gamma, const float *__restrict__ u, const float *__restrict__ omega,
    float *__restrict__ g_pos, float *__restrict__ g_vel, float *__restrict__ g_mass,
    float *__restrict__ g_h, float *__restrict__ g_u, float *__restrict__ g_rho,
    float *__restrict__ g_omega) {
  __shared__ TeamLds<kT> search;
  __shared__ HSides T[kT];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  int range = 0;
  for (int g; (g = team_next_group(gs, range, search)) >= 0;) {
    const Group grp = group_at(gs, g);
    const bool valid = lane < grp.count;
    const int s = valid ? (gs.targets ? gs.targets[grp.t0 + lane] : grp.t0 + lane) : grp.t0;
    HSide P;
    P.xm = xm[s];
    P.vh = vh[s];
    P.aux = aux[s];
    P.up = up[s];
    const float hp = valid ? P.vh.w : -1.0f, hp2 = sq_exact(fmaxf(hp, 0.0f));
    const bool p_on = valid && (P.up.x != 0.f || P.up.y != 0.f || P.up.z != 0.f || P.up.w != 0.f);
    constexpr int kN = 11;
    float acc[kN], cmp[kN];
#pragma unroll
    for (int k = 0; k < kN; ++k) acc[k] = cmp[k] = 0.0f;
    int cand = 0;
    // the box of the group's particles and their largest fl(h^2): a
    // candidate q whose box_dist2 to the box reaches both that and
    // fl(h_q^2) is in no lane's symmetric neighbourhood, since box_dist2
    // never exceeds the r2 of a point inside the box
    float4 tlo = make_float4(valid ? P.xm.x : INFINITY, valid ? P.xm.y : INFINITY,
                             valid ? P.xm.z : INFINITY, 0.f);
    float4 thi = make_float4(valid ? P.xm.x : -INFINITY, valid ? P.xm.y : -INFINITY,
                             valid ? P.xm.z : -INFINITY, 0.f);
    // a member without h (or with a NaN) is still its neighbours' neighbour
    const float want = valid ? fmaxf(hp, 0.0f) : -1.0f;
    float hmax2 = valid ? sq_exact(hp) : -1.0f, hg = want;  // hg: the group's largest
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) {
      hg = fmaxf(hg, __shfl_xor(hg, m));
      tlo.x = fminf(tlo.x, __shfl_xor(tlo.x, m));
      tlo.y = fminf(tlo.y, __shfl_xor(tlo.y, m));
      tlo.z = fminf(tlo.z, __shfl_xor(tlo.z, m));
      thi.x = fmaxf(thi.x, __shfl_xor(thi.x, m));
      thi.y = fmaxf(thi.y, __shfl_xor(thi.y, m));
      thi.z = fmaxf(thi.z, __shfl_xor(thi.z, m));
      hmax2 = fmaxf(hmax2, __shfl_xor(hmax2, m));
    }
    {
      auto su = [](float v) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))); };
      tlo = make_float4(su(tlo.x), su(tlo.y), su(tlo.z), 0.f);
      thi = make_float4(su(thi.x), su(thi.y), su(thi.z), 0.f);
      hmax2 = su(hmax2);
      hg = su(hg);
    }
    auto flush = [&](int nc) {
      {
        HSide Q;
        Q.xm = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
        Q.vh = make_float4(0.f, 0.f, 0.f, 0.f);
        Q.aux = make_float4(0.f, 0.f, 1.f, 1.f);
        Q.up = make_float4(0.f, 0.f, 0.f, 0.f);
        if (lane < nc) {
          Q.xm = xm[cand];
          Q.vh = vh[cand];
          Q.aux = aux[cand];
          Q.up = up[cand];
        }
        const float d2 = box_dist2(make_float3(Q.xm.x, Q.xm.y, Q.xm.z), tlo, thi);
        const bool keep = lane < nc && (d2 < hmax2 || d2 < sq_exact(Q.vh.w));
        const uint64_t km = __ballot(keep);
        const int slot = (int)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(km >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)km, 0u));
        // kept candidates in their order at the front, infinity behind (the
        // tests take whole groups of kStep)
        T[w].xh[lane] = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
        if (keep) {
          T[w].xh[slot] = make_float4(Q.xm.x, Q.xm.y, Q.xm.z, sq_exact(fmaxf(Q.vh.w, 0.0f)));
          T[w].vm[slot] = make_float4(Q.vh.x, Q.vh.y, Q.vh.z, Q.xm.w);
          T[w].aux[slot] = Q.aux;
          T[w].up[slot] = Q.up;
        }
        nc = __popcll(km);
      }
      wave_sync();
      // the entries with upstream gradients; a lane without takes only these
      uint64_t qm;
      {
        const float4 qu = T[w].up[lane];
        qm = __ballot(lane < nc && (qu.x != 0.f || qu.y != 0.f || qu.z != 0.f || qu.w != 0.f));
      }
      const uint32_t on[2] = {__brev((uint32_t)qm), __brev((uint32_t)(qm >> 32))};
      float part[kN];
#pragma unroll
      for (int k = 0; k < kN; ++k) part[k] = 0.0f;
      // entries [32 half, 32 half + 32) that the lane takes, the first in the
      // highest bit
      auto tests = [&](int half) {
        constexpr int kStep = 4;
        uint32_t hits = 0;
        int k = 32 * half;
        for (; k < min(nc, 32 * half + 32); k += kStep) {
#pragma unroll
          for (int i = 0; i < kStep; ++i) {
            const float4 q = T[w].xh[k + i];
            const float r2 = dist2_exact(sub_exact(q.x, P.xm.x), sub_exact(q.y, P.xm.y),
                                         sub_exact(q.z, P.xm.z));
            hits = 2u * hits + (r2 < max_num(hp2, q.w) && r2 > 0.0f ? 1u : 0u);
          }
        }
        const int free = 32 * half + 32 - k;  // untested entries of a short tile
        hits = valid && free < 32 ? hits << free : 0u;
        return p_on ? hits : hits & on[half];
      };
      uint32_t now = tests(0), next = tests(1), q_now = on[0];
      for (int base = 0; (now | next) != 0u;) {
        if (now == 0u) {
          now = next;
          next = 0u;
          base = 32;
          q_now = on[1];
        }
        const int z = __builtin_clz(now), k = base + z;
        const uint32_t bit = 0x80000000u >> z;
        now &= ~bit;
        HSide Q;
        Q.xm = T[w].xh[k];
        Q.vh = T[w].vm[k];
        Q.aux = T[w].aux[k];
        Q.up = T[w].up[k];
        Q.xm.w = Q.vh.w;  // the mass
        const float dx = sub_exact(Q.xm.x, P.xm.x), dy = sub_exact(Q.xm.y, P.xm.y),
                    dz = sub_exact(Q.xm.z, P.xm.z);  // x_q - x_p
        hydro_pair_adjoint(P, Q, alpha, p_on, (q_now & bit) != 0u, -dx, -dy, -dz,
                           dist2_exact(dx, dy, dz), part);
      }
#pragma unroll
      for (int k = 0; k < kN; ++k) neumaier_add(acc[k], cmp[k], part[k]);
      wave_sync();
    };
    team_search<kT, kDeep>(
        tm, grp.snap, search, make_float3(P.xm.x, P.xm.y, P.xm.z), want, tlo, thi, hg,
        [](float h, float hmax) { return h < 0.0f ? -1.0f : sq_exact(fmaxf(h, hmax)); },
        [&](int ntiles, int count) {
          for (int j = w; j < ntiles; j += kT) {
            // (every ntiles-th candidate of the round)
            const int nc = (count - j + ntiles - 1) / ntiles;
            cand = lane < nc ? search.cand[j + lane * ntiles] : 0;
            flush(nc);
          }
        });
    team_totals<kT, kN, sizeof(HSides) / 4>((float *)T, w, lane, acc, cmp);
    if (valid && w == 0) {
      float tot[kN];
#pragma unroll
      for (int k = 0; k < kN; ++k) tot[k] = acc[k] + cmp[k];
      const int cid = perm[s];
      if (g_pos) {
        g_pos[3 * cid] += tot[0];
        g_pos[3 * cid + 1] += tot[1];
        g_pos[3 * cid + 2] += tot[2];
      }
      if (g_vel) {
        g_vel[3 * cid] += tot[3];
        g_vel[3 * cid + 1] += tot[4];
        g_vel[3 * cid + 2] += tot[5];
      }
      if (g_h) g_h[cid] += tot[6];
      if (g_mass) g_mass[cid] += tot[10];
      // A = (gamma-1) u / (Omega rho): dA/du = (gamma-1)/(Omega rho),
      // dA/dOmega = -A/Omega, dA/drho = -A/rho; dc/du = c / (2u)
      const float A = P.aux.x, cc = P.aux.y, rp = P.aux.z, up_ = u[cid], om = omega[cid];
      const float gA = tot[7], gc = tot[8];
      if (g_u) g_u[cid] += gA * (gamma - 1.0f) / (om * rp) + (up_ > 0.0f ? gc * cc / (2.0f * up_) : 0.0f);
      if (g_omega) g_omega[cid] += -gA * A / om;
      if (g_rho) g_rho[cid] += -gA * A / rp + tot[9];
    }
  }
}

}  // namespace

hipError_t launch_hydro_bwd(Octree &gas, const int32_t *iperm, int64_t n_caller,
                            const Groups &all_gas, int64_t max_groups, const Terms &tm,
                            int64_t n_act, const int32_t *active, float alpha, float gamma,
                            const float *u,
                            const float *omega, const float *g_acc, const float *g_dudt,
                            float4 *up, float *g_pos, float *g_vel, float *g_mass, float *g_h,
                            float *g_u, float *g_rho, float *g_omega, hipStream_t s) {
  const int64_t m = gas.n;
  if (m == 0) return hipSuccess;
  k_zero_f4<<<nblk(m), kBlock, 0, s>>>(up, m);
  const int64_t na = active ? n_act : n_caller;
  if (na > 0)
    k_hydro_bwd_up<<<nblk(na), kBlock, 0, s>>>(active, na, iperm, n_caller, g_acc, g_dudt, up);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int team = adjoint_team(m);
  auto kern = team == 16  ? k_hydro_bwd<16>
              : team == 8 ? k_hydro_bwd<8>
              : team == 4 ? k_hydro_bwd<4>
                          : nullptr;
  if (tm.deep) kern = team == 4 ? k_hydro_bwd<4, true> : nullptr;
  if (!kern) return hipErrorInvalidValue;  // (no such team)
  const int block = team * kWave;
  kern<<<persistent_grid((const void *)kern, block, max_groups, team), block, 0, s>>>(
      gas.xm, gas.vh, gas.aux, up, gas.perm, all_gas, tm, alpha, gamma, u, omega, g_pos, g_vel,
      g_mass, g_h, g_u, g_rho, g_omega);
  return hipGetLastError();
}

hipError_t launch_gravity_bwd(const Octree &all, const Groups &gs, int64_t max_groups,
                              const GravParams &gp, int64_t n_act, const int32_t *active,
                              const float *g_acc, const float *g_pot, float4 *gsrc,
                              float4 *gnode, unsigned long long *gsrc_fx,
                              unsigned long long *gnode_fx, unsigned *mx, double4 *pq,
                              double *rr, float *g_pos, float *g_mass, hipStream_t s) {
  const int64_t m = all.n, nn = all.nnodes;
  if (m == 0 || nn == 0) return hipSuccess;
  if (!all.cnodes || (gp.team != 16 && gp.team != 8 && gp.team != 4 && gp.team != 1))
    return hipErrorInvalidValue;
  const int64_t na = active ? n_act : m;
  auto pick = [&](auto fixed_c) {
    constexpr bool f = decltype(fixed_c)::value;
    if (gp.team == 16) return gp.inside_test ? k_gravity_bwd<f, true, 16> : k_gravity_bwd<f, false, 16>;
    if (gp.team == 8) return gp.inside_test ? k_gravity_bwd<f, true, 8> : k_gravity_bwd<f, false, 8>;
    if (gp.team == 4) return gp.inside_test ? k_gravity_bwd<f, true, 4> : k_gravity_bwd<f, false, 4>;
    return gp.inside_test ? k_gravity_bwd<f, true, 1> : k_gravity_bwd<f, false, 1>;
  };
  const int block = gp.team * kWave;
  if (gp.eps2 > 0.0f) {
    // fixed-point counters (two words per component, four components)
    k_zero_f4<<<nblk(4 * m), kBlock, 0, s>>>((float4 *)gsrc_fx, 4 * m);
    k_zero_f4<<<nblk(4 * nn), kBlock, 0, s>>>((float4 *)gnode_fx, 4 * nn);
    k_zero_f4<<<1, kBlock, 0, s>>>((float4 *)mx, 1);
    const int64_t nb = na > m ? na : m;
    const unsigned gb = nblk(nb) < (unsigned)kFxBoundBlocks ? nblk(nb) : (unsigned)kFxBoundBlocks;
    k_fx_bound<<<gb, kBlock, 0, s>>>(active, na, g_acc, g_pot, all.xm, m, mx);
    if (max_groups > 0) {
      auto kern = pick(std::true_type{});
      kern<<<persistent_grid((const void *)kern, block, max_groups, gp.team), block, 0, s>>>(
          all.cnodes, all.ckeys, all.xm, all.keys, all.perm, gs, gp.theta2, gp.eps2, gp.G, g_acc, g_pot,
          gsrc, gnode, gsrc_fx, gnode_fx, mx, m, na);
    }
    k_fx_to_f4<<<nblk(m), kBlock, 0, s>>>(gsrc_fx, m, mx, gp.eps2, gp.G, m, na, gsrc);
    k_fx_to_f4<<<nblk(nn), kBlock, 0, s>>>(gnode_fx, nn, mx, gp.eps2, gp.G, m, na, gnode);
  } else {
    k_zero_f4<<<nblk(m), kBlock, 0, s>>>(gsrc, m);
    k_zero_f4<<<nblk(nn), kBlock, 0, s>>>(gnode, nn);
    if (max_groups > 0) {
      auto kern = pick(std::false_type{});
      kern<<<persistent_grid((const void *)kern, block, max_groups, gp.team), block, 0, s>>>(
          all.cnodes, all.ckeys, all.xm, all.keys, all.perm, gs, gp.theta2, gp.eps2, gp.G, g_acc, g_pot,
          gsrc, gnode, nullptr, nullptr, nullptr, m, na);
    }
  }
  k_push_init<<<nblk(nn), kBlock, 0, s>>>(gnode, all.mom, nn, pq, rr);
  for (int l = 0; l < all.max_level; ++l)
    k_push_level<<<nblk(nn), kBlock, 0, s>>>(all.nodes, all.mom, nn, l, pq, rr);
  k_push_leaves<<<nblk(nn), kBlock, 0, s>>>(all.nodes, all.mom, nn, all.xm, pq, rr, gsrc);
  k_scatter_grad<<<nblk(m), kBlock, 0, s>>>(all.perm, m, gsrc, g_pos, g_mass);
  return hipGetLastError();
}

static hipError_t density_bwd(const Octree &gas, const Groups &gs, int64_t max_groups,
                              const Terms &tm, const float4 *bw, float *g_pos, float *g_mass,
                              float *g_h, hipStream_t s) {
  const int team = adjoint_team(gas.n);
  auto kern = team == 16  ? k_density_bwd<16>
              : team == 8 ? k_density_bwd<8>
              : team == 4 ? k_density_bwd<4>
                          : nullptr;
  if (tm.deep) kern = team == 4 ? k_density_bwd<4, true> : nullptr;
  if (!kern) return hipErrorInvalidValue;  // (no such team)
  const int block = team * kWave;
  kern<<<persistent_grid((const void *)kern, block, max_groups, team), block, 0, s>>>(
      gas.xm, bw, gas.perm, gs, tm, g_pos, g_mass, g_h);
  return hipGetLastError();
}

hipError_t launch_density_bwd(Octree &gas, const int32_t *iperm, int64_t n_caller,
                              const Groups &all_gas, int64_t max_groups, const Terms &tm,
                              int64_t n_act, const int32_t *active, const float *h,
                              const float *rho,
                              const float *drho, const float *g_rho, const float *g_drho,
                              const float *g_omega, float *g_pos, float *g_mass, float *g_h,
                              hipStream_t s) {
  const int64_t m = gas.n;
  if (m == 0) return hipSuccess;
  float4 *bw = gas.aux;  // (h, gbar_rho, gbar_rho', 1/h) per sorted gas member
  k_density_bwd_init<<<nblk(m), kBlock, 0, s>>>(gas.perm, m, h, bw);
  const int64_t na = active ? n_act : n_caller;
  if (na > 0)
    k_density_bwd_prep<<<nblk(na), kBlock, 0, s>>>(active, na, iperm, n_caller, h, rho, drho,
                                                    g_rho, g_drho, g_omega, bw, g_h);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return density_bwd(gas, all_gas, max_groups, tm, bw, g_pos, g_mass, g_h, s);
}

hipError_t launch_density_solve_bwd(Octree &gas, const int32_t *iperm, int64_t n_caller,
                                    const Groups &all_gas, int64_t max_groups, const Terms &tm,
                                    int64_t n_act, const int32_t *active, float n_ngb,
                                    const float *h,
                                    const float *rho, const float *drho, const float *g_h,
                                    float *g_pos, float *g_mass, hipStream_t s) {
  const int64_t m = gas.n;
  if (m == 0) return hipSuccess;
  float4 *bw = gas.aux;  // (h, gbar_rho, 0, 1/h) per sorted gas member
  k_density_bwd_init<<<nblk(m), kBlock, 0, s>>>(gas.perm, m, h, bw);
  const int64_t na = active ? n_act : n_caller;
  if (na > 0)
    k_hsolve_bwd_prep<<<nblk(na), kBlock, 0, s>>>(active, na, iperm, n_caller, h, rho, drho, g_h,
                                                   gas.xm, n_ngb, bw, g_mass);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return density_bwd(gas, all_gas, max_groups, tm, bw, g_pos, g_mass, nullptr, s);
}

}  // namespace g3
