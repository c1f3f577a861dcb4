// Octree build on the GPU: Morton keys, radix sort, permutation into sorted
// float4 arrays, preorder topology computed per particle without recursion,
// and bottom-up FP64 monopoles with tight bounding boxes.
//
// Topology (Barnes & Hut 1986 octree over Morton-sorted members): a node is
// the run of members sharing a 3l-bit key prefix; it is split while it holds
// more than B members and l < 21. Write cpl(a, b) for the number of leading
// 3-bit digits two keys share. Member p starts a node at level l exactly
// when l >= delta_p = cpl(p, p-1) + 1 (delta_0 = 0), and the deepest node
// holding p (its leaf) is at depth d_p = 1 + the B-th largest of
// cpl(p, p +- k), k = 1..B (missing neighbours count -1), capped at 21.
// So p starts the nodes of levels delta_p..d_p, and in preorder (children in
// Morton order) the nodes sorted by (first member, level) are numbered by an
// exclusive scan of the per-member counts. The node after the subtree of a
// node ending before member e is the first node that starts at e.
#include <algorithm>
#include <utility>

#include "g3_device.h"
#include "g3_internal.h"

namespace g3 {

namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ uint64_t spread3(uint32_t v) {
  uint64_t x = v & 0x1fffffu;
  x = (x | (x << 32)) & 0x1f00000000ffffull;
  x = (x | (x << 16)) & 0x1f0000ff0000ffull;
  x = (x | (x << 8)) & 0x100f00f00f00f00full;
  x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
  x = (x | (x << 2)) & 0x1249249249249249ull;
  return x;
}

// key cell in FP64 for FP32 and FP64 positions alike
template <typename T>
__device__ __forceinline__ uint32_t cell_of(T x, double lo, double scale) {
  double f = floor(((double)x - lo) * scale);
  if (!(f >= 0.0)) f = 0.0;
  if (f > (double)((1u << kMaxLevel) - 1u)) f = (double)((1u << kMaxLevel) - 1u);
  return (uint32_t)f;
}

template <typename T>
__device__ __forceinline__ uint64_t morton_key(const T *p, double lx, double ly, double lz,
                                               double scale) {
  return (spread3(cell_of(p[0], lx, scale)) << 2) | (spread3(cell_of(p[1], ly, scale)) << 1) |
         spread3(cell_of(p[2], lz, scale));
}

// keys and identity values, each particle keyed in the box of its snapshot
// (caller ids [coff[k], coff[k+1])); pm (nullable): positions and masses side
// by side, so that the gather into sorted order reads one 16-byte word a
// particle instead of two lines (102 -> 67 us on 2^21 particles)
template <typename T>
__global__ void k_keys(const T *__restrict__ pos, int64_t m, const int64_t *__restrict__ coff,
                       const double4 *__restrict__ sbox, int n_snap,
                       const float *__restrict__ mass, uint64_t *__restrict__ keys,
                       uint32_t *__restrict__ vals, float4 *__restrict__ pm) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= m) return;
  const double4 b = sbox[n_snap > 1 ? segment_of(coff, n_snap, i) : 0];
  const double scale = 2097152.0 / b.w;  // 2^21 / side
  keys[i] = morton_key(pos + 3 * i, b.x, b.y, b.z, scale);
  vals[i] = (uint32_t)i;
  if (pm)
    pm[i] = make_float4((float)pos[3 * i], (float)pos[3 * i + 1], (float)pos[3 * i + 2], mass[i]);
}

// Forest: the snapshot of each key-sorted member, for a stable sort by
// snapshot after the sort by key.
__global__ void k_snap_keys(const uint32_t *__restrict__ vals, int64_t m,
                            const int64_t *__restrict__ coff, int n_snap,
                            uint64_t *__restrict__ skey, uint32_t *__restrict__ sidx) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  skey[k] = (uint64_t)segment_of(coff, n_snap, (int64_t)vals[k]);
  sidx[k] = (uint32_t)k;
}

__global__ void k_gather_sorted(const uint32_t *__restrict__ sidx, int64_t m,
                                const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                                uint64_t *__restrict__ kout, uint32_t *__restrict__ vout) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  const uint32_t j = sidx[k];
  kout[k] = kin[j];
  vout[k] = vin[j];
}

// Sorted start of each snapshot in the all-particle octree (its caller offset).
__global__ void k_soff(const int64_t *__restrict__ coff, int n_snap, int32_t *__restrict__ soff) {
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k <= n_snap) soff[k] = (int32_t)coff[k];
}

// and in the gas octree: the gas members sorted before it (exclusive scan
// `slot` over the sorted members).
__global__ void k_gas_soff(const int32_t *__restrict__ soff_all, int n_snap,
                           const uint32_t *__restrict__ slot, int32_t *__restrict__ soff) {
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k <= n_snap) soff[k] = (int32_t)slot[soff_all[k]];
}

// The tables of one snapshot, from the call's arguments (no host copy that
// the build would have to wait for).
__global__ void k_one_snap(int64_t n, double4 box, int64_t *__restrict__ coff,
                           double4 *__restrict__ sbox, int32_t *__restrict__ soff) {
  coff[0] = 0;
  coff[1] = n;
  sbox[0] = box;
  soff[0] = 0;
  soff[1] = (int32_t)n;
}

// First node of each snapshot: the first node its first member starts.
__global__ void k_nroot(const uint32_t *__restrict__ off, const int32_t *__restrict__ soff,
                        int n_snap, int32_t *__restrict__ nroot) {
  const int k = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  if (k > n_snap) return;
  nroot[k] = (int32_t)off[soff[k]];
}

// The gas octree's members in sorted order come from the all-particle
// octree's: filtering its (snapshot, key, caller id) order keeps that order,
// which is exactly the order a sort of the gas members would give.
__global__ void k_gas_of_sorted(const int32_t *__restrict__ perm_all, int64_t n,
                                const uint8_t *__restrict__ type, uint32_t *__restrict__ flags) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < n) flags[s] = (type == nullptr || type[perm_all[s]] == 0) ? 1u : 0u;
}

// Its sorted copies are compacted with them: streams, where a gather by caller
// id would read every position from a line of its own.
__global__ void k_compact_sorted(const uint32_t *__restrict__ flags,
                                 const uint32_t *__restrict__ slot, int64_t n,
                                 const Octree all, uint64_t *__restrict__ keys,
                                 int32_t *__restrict__ perm, float4 *__restrict__ xm,
                                 double4 *__restrict__ x64, int32_t *__restrict__ iperm) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= n) return;
  if (!flags[s]) return;
  const int32_t id = all.perm[s];
  const uint32_t at = slot[s];
  iperm[id] = (int32_t)at;
  keys[at] = all.keys[s];
  perm[at] = id;
  xm[at] = all.xm[s];
  if (x64) x64[at] = all.x64[s];
}

// Sorted copies: FP32 (x, y, z, m) always; for FP64 positions also the
// exact (x, y, z, m) in FP64.
template <typename T>
__global__ void k_permute(const uint32_t *__restrict__ perm, int64_t m,
                          const T *__restrict__ pos, const float *__restrict__ mass,
                          float4 *__restrict__ xm, double4 *__restrict__ x64,
                          int32_t *__restrict__ iperm, int32_t *__restrict__ perm_out) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const uint32_t j = perm[s];
  xm[s] = make_float4((float)pos[3 * j], (float)pos[3 * j + 1], (float)pos[3 * j + 2], mass[j]);
  if (x64)
    x64[s] = make_double4((double)pos[3 * j], (double)pos[3 * j + 1], (double)pos[3 * j + 2],
                          (double)mass[j]);
  if (iperm) iperm[j] = (int32_t)s;
  if (perm_out) perm_out[s] = (int32_t)j;
}

// The same from positions and masses side by side.
__global__ void k_permute_packed(const uint32_t *__restrict__ order, int64_t m,
                                 const float4 *__restrict__ pm, float4 *__restrict__ xm,
                                 int32_t *__restrict__ iperm, int32_t *__restrict__ perm) {
  const int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= m) return;
  const uint32_t j = order[s];
  xm[s] = pm[j];
  iperm[j] = (int32_t)s;
  perm[s] = (int32_t)j;
}

__device__ __forceinline__ int cpl(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  if (x == 0) return kMaxLevel;
  return (__clzll((long long)x) - 1) / 3;  // bit 63 is never used
}

// Nodes started by each member: cnt[p] = max(0, d_p - delta_p + 1). B + 1
// consecutive members share as many digits as their ends do, so the deepest
// node that holds p and must be split is the largest cpl(q, q + B) over the
// windows q = p - B .. p: one prefix length a member, shared through LDS, and a
// maximum over B + 1 of them.
constexpr int kMaxLeaf = 64;

__global__ __launch_bounds__(kBlock) void k_node_counts(const uint64_t *__restrict__ keys,
                                                        int64_t m,
                                                        const int32_t *__restrict__ soff,
                                                        int n_snap, int B,
                                                        uint32_t *__restrict__ cnt,
                                                        uint8_t *__restrict__ lev,
                                                        int32_t *__restrict__ maxlev) {
  // the block's keys with B neighbours on each side, and the windows' lengths
  __shared__ uint64_t win[kBlock + 2 * kMaxLeaf];
  __shared__ int8_t len[kBlock + kMaxLeaf];  // window of member b0 - B + k
  __shared__ int32_t block_max;  // deepest leaf level of the block
  if (threadIdx.x == 0) block_max = 0;
  const int64_t b0 = (int64_t)blockIdx.x * kBlock;
  for (int k = threadIdx.x; k < kBlock + 2 * B; k += kBlock) {
    const int64_t q = b0 - B + k;
    win[k] = (q >= 0 && q < m) ? keys[q] : 0ull;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < kBlock + B; k += kBlock) {
    const int64_t q = b0 - B + k;
    int v = -1;
    // members of other snapshots count as missing: each snapshot is a tree
    if (q >= 0 && q + B < m &&
        (n_snap == 1 || segment_of(soff, n_snap, q) == segment_of(soff, n_snap, q + B)))
      v = cpl(win[k], win[k + B]);
    len[k] = (int8_t)v;
  }
  __syncthreads();
  const int64_t p = b0 + threadIdx.x;
  if (p < m) {
    const int64_t s0 = n_snap > 1 ? soff[segment_of(soff, n_snap, p)] : 0;
    const int delta =
        (p == s0) ? 0 : cpl(win[B + threadIdx.x], win[B + threadIdx.x - 1]) + 1;
    int val = -1;
    for (int k = 0; k <= B; ++k) val = max(val, (int)len[threadIdx.x + k]);
    const int d = min(val + 1, kMaxLevel);
    cnt[p] = (d >= delta) ? (uint32_t)(d - delta + 1) : 0u;
    lev[2 * p] = (uint8_t)delta;
    lev[2 * p + 1] = (uint8_t)d;
    if (d >= delta) atomicMax(&block_max, d);
  }
  __syncthreads();
  // (most blocks find the depth reached already: 2^13 atomics on one word
  // took 80 us)
  if (threadIdx.x == 0 &&
      block_max > __hip_atomic_load(maxlev, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMax(maxlev, block_max);
}

// The nodes that start at member p: levels lev[2p]..lev[2p+1], each up to the
// first member that leaves its cell. A lane looks for a near end (kNearEnd
// members) itself; a far one is found by the whole wave, 64 probes a step.
// Bound by the longest chain of dependent loads: the first members of the
// largest cells start a node on every level, and with a lane's own doubling
// and halving search the chain was 170 loads on 2^21 particles: 60 us in the
// average octree of 2^21 and 2^20, 32 on 6e4, 12 on 4096 (52, 11 and 9 now).
constexpr int kNearEnd = 32;
__global__ __launch_bounds__(kBlock) void k_nodes(
    const uint64_t *__restrict__ keys, int64_t m, const int32_t *__restrict__ soff, int n_snap,
    const double4 *__restrict__ sbox, const uint32_t *__restrict__ off,
    const uint8_t *__restrict__ lev, int64_t nnodes, Node *__restrict__ nodes) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = lane_id();
  int delta = 1, d = 0;  // (none)
  if (p < m) {
    delta = lev[2 * p];
    d = lev[2 * p + 1];
  }
  uint64_t kp = 0;
  float side = 0.f;
  int end = 0;  // members of the level-l node: [p, end)
  uint32_t at = 0;
  if (d >= delta) {
    kp = keys[p];
    const int sn = n_snap > 1 ? segment_of(soff, n_snap, p) : 0;
    side = (float)sbox[sn].w;
    end = soff[sn + 1];
    at = off[p];
  }
  for (int l = delta; __ballot(l <= d) != 0ull; ++l) {
    const bool work = l <= d;
    // the first q in (p, end] with cpl(p, q) < l (end shrinks as l grows);
    // answer in [lo, hi]
    int lo = (int)p + 1, hi = end;
    bool far = false;
    if (work) {
      const int q = lo + kNearEnd - 1;
      if (q < hi) {
        if (cpl(kp, keys[q]) >= l) {
          lo = q + 1;
          far = true;
        } else {
          hi = q;
        }
      }
      while (!far && lo < hi) {
        const int mid = lo + (hi - lo) / 2;
        if (cpl(kp, keys[mid]) >= l) lo = mid + 1;
        else hi = mid;
      }
    }
    uint64_t fm = __ballot(far);
    while (fm) {
      const int b = (int)__builtin_ctzll(fm);
      fm &= fm - 1ull;
      const uint64_t kb = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(kp >> 32), b) << 32) |
                          (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)kp, b);
      const int lb = __builtin_amdgcn_readlane(l, b);
      int x = __builtin_amdgcn_readlane(lo, b), y = __builtin_amdgcn_readlane(hi, b);
      while (x < y) {
        const int step = (y - x + kWave - 1) / kWave;
        const int64_t q = (int64_t)x + (int64_t)step * (lane + 1) - 1;
        const int in = __popcll(__ballot(q < y && cpl(kb, keys[q < y ? q : x]) >= lb));
        y = (int)min((int64_t)y, (int64_t)x + (int64_t)step * (in + 1) - 1);
        x += step * in;
      }
      if (lane == b) lo = x;
    }
    if (work) {
      end = lo;
      Node nd;
      nd.lo_h = make_float4(0.f, 0.f, 0.f, 0.f);
      nd.hi_l = make_float4(0.f, 0.f, 0.f, ldexpf(side, -l));
      // (the moments fill com_m and the boxes)
      nd.meta = make_int4(end >= m ? (int)nnodes : (int)off[end], (int)p, end - (int)p,
                          l | (l == d ? kLeafBit : 0));
      Node &to = nodes[(int64_t)at + (l - delta)];
      to.lo_h = nd.lo_h;
      to.hi_l = nd.hi_l;
      to.meta = nd.meta;
    }
  }
}

// A node in four bytes for the terminal lists: its own member count (a leaf: 0)
// in the low half, its parent's in the high half, both cut off above what a
// walk_leaf can be. A root counts as inside an unbounded node.
constexpr uint32_t kRootCode = 0xffff0000u;
__device__ __forceinline__ uint32_t term_code(int4 meta, uint32_t parent) {
  return ((meta.w & kLeafBit) ? 0u : (uint32_t)min(meta.z, 65535)) | parent;
}
__device__ __forceinline__ bool is_terminal(uint32_t code, int walk_leaf) {
  return (int)(code & 0xffffu) <= walk_leaf && (int)(code >> 16) > walk_leaf;
}
__device__ __forceinline__ bool is_root(uint32_t code) { return code >= kRootCode; }

// The codes of all nodes; nch (nullable): the number of children of every node.
__global__ void k_parents(const Node *__restrict__ nodes, int64_t nnodes,
                          uint32_t *__restrict__ tcode, uint32_t *__restrict__ nch) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nnodes) return;
  const int4 meta = nodes[k].meta;
  if ((meta.w & 255) == 0) tcode[k] = term_code(meta, kRootCode);
  uint32_t nc = 0;
  if (!(meta.w & kLeafBit)) {
    const uint32_t pc = (uint32_t)min(meta.z, 65534) << 16;
    for (int64_t c = k + 1; c < meta.x; ++nc) {
      const int4 cm = nodes[c].meta;
      tcode[c] = term_code(cm, pc);
      c = cm.x;
    }
  }
  if (nch) nch[k] = nc;
}

// FP64 mass and first moments, tight box of one node, from its members or its
// children.
struct Moments {
  Node *__restrict__ nodes;
  double4 *__restrict__ mom;
  double4 *__restrict__ c64;
  const float4 *__restrict__ xm;
  const double4 *__restrict__ x64;
};
struct NodeSums {
  double M = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
  float3 lo = make_float3(INFINITY, INFINITY, INFINITY);
  float3 hi = make_float3(-INFINITY, -INFINITY, -INFINITY);
  __device__ __forceinline__ void add(double m, double x, double y, double z, float lx, float ly,
                                      float lz, float hx, float hy, float hz) {
    M += m;
    Sx += x;
    Sy += y;
    Sz += z;
    lo.x = fminf(lo.x, lx); lo.y = fminf(lo.y, ly); lo.z = fminf(lo.z, lz);
    hi.x = fmaxf(hi.x, hx); hi.y = fmaxf(hi.y, hy); hi.z = fmaxf(hi.z, hz);
  }
};

// A leaf's sums, four members' loads at a time.
__device__ __forceinline__ NodeSums leaf_sums(const Moments &A, int4 meta) {
  NodeSums r;
  const int end = meta.y + meta.z;
  for (int s = meta.y; s < end; s += 4) {
    float4 p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] = A.xm[min(s + q, end - 1)];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (s + q >= end) break;
      // moments from the exact positions (FP64 ones when the tree has them)
      const double4 v = A.x64 ? A.x64[s + q] : make_double4(p[q].x, p[q].y, p[q].z, p[q].w);
      r.add(v.w, v.w * v.x, v.w * v.y, v.w * v.z, p[q].x, p[q].y, p[q].z, p[q].x, p[q].y, p[q].z);
    }
  }
  return r;
}

// Node k's moments, centre and box (the fourth components of its box stay).
__device__ __forceinline__ void store_node(const Moments &A, int64_t k, const NodeSums &r) {
  A.mom[k] = make_double4(r.M, r.Sx, r.Sy, r.Sz);
  Node &nd = A.nodes[k];
  float4 cm;
  if (r.M > 0.0)
    cm = make_float4((float)(r.Sx / r.M), (float)(r.Sy / r.M), (float)(r.Sz / r.M), (float)r.M);
  else  // massless node: its geometric centre
    cm = make_float4(0.5f * (r.lo.x + r.hi.x), 0.5f * (r.lo.y + r.hi.y),
                     0.5f * (r.lo.z + r.hi.z), 0.f);
  nd.com_m = cm;
  if (A.c64)
    A.c64[k] = r.M > 0.0 ? make_double4(r.Sx / r.M, r.Sy / r.M, r.Sz / r.M, r.M)
                         : make_double4(cm.x, cm.y, cm.z, 0.0);
  nd.lo_h.x = r.lo.x; nd.lo_h.y = r.lo.y; nd.lo_h.z = r.lo.z;
  nd.hi_l.x = r.hi.x; nd.hi_l.y = r.hi.y; nd.hi_l.z = r.hi.z;
}

__device__ __forceinline__ void node_moments(const Moments &A, int64_t k, int4 meta) {
  if (meta.w & kLeafBit) {
    store_node(A, k, leaf_sums(A, meta));
    return;
  }
  NodeSums r;
  for (int64_t c = k + 1; c < meta.x; c = A.nodes[c].meta.x) {
    const double4 cm = A.mom[c];
    const float4 lo = A.nodes[c].lo_h, hi = A.nodes[c].hi_l;
    r.add(cm.x, cm.y, cm.z, cm.w, lo.x, lo.y, lo.z, hi.x, hi.y, hi.z);
  }
  store_node(A, k, r);
}

// The moments bottom up in two launches: the subtrees of at most kSubtree
// members (and larger leaves) whose parent holds more, a workgroup each, and
// then the nodes above them, one workgroup for all (one launch for trees of
// at most kSmallNodes nodes). Leaves need no order; inner nodes go level by
// level with a barrier between. Bound by latency: a level costs one step of
// its children's data. What a workgroup has summed stays in LDS for the
// parents, and the nodes above hold their children's indices (found once, by
// the build), so no step follows a chain of loads from one child to the next;
// that chain took 80 us for the subtrees and 50 for the nodes above in the
// average octree of 2^21 and 2^20 particles (57 and 46 now, the latter the
// request rate of the one CU), 14 and 23 on 6e4 (10.5 and 13), 23 on 4096 (19).
template <int kCap>
struct MomLds {
  double m[4][kCap];
  float lo[3][kCap], hi[3][kCap];
  int32_t skip[kCap];
  int32_t inner[kCap];  // (local index << 8) | level
  int32_t n_inner, max_level;
};

// The n nodes from k0 on (n <= kCap), whole subtrees.
template <int kCap>
__device__ __forceinline__ void lds_moments(const Moments &A, int k0, int n, MomLds<kCap> &S) {
  const int tid = (int)threadIdx.x, nthr = (int)blockDim.x;
  if (tid == 0) {
    S.n_inner = 0;
    S.max_level = -1;
  }
  __syncthreads();
  auto keep = [&](int q, const NodeSums &r) {
    S.m[0][q] = r.M; S.m[1][q] = r.Sx; S.m[2][q] = r.Sy; S.m[3][q] = r.Sz;
    S.lo[0][q] = r.lo.x; S.lo[1][q] = r.lo.y; S.lo[2][q] = r.lo.z;
    S.hi[0][q] = r.hi.x; S.hi[1][q] = r.hi.y; S.hi[2][q] = r.hi.z;
    store_node(A, k0 + q, r);
  };
  for (int q = tid; q < n; q += nthr) {
    const int4 meta = A.nodes[k0 + q].meta;
    S.skip[q] = meta.x - k0;
    if (meta.w & kLeafBit) {
      keep(q, leaf_sums(A, meta));
    } else {
      S.inner[atomicAdd(&S.n_inner, 1)] = q << 8 | (meta.w & 255);
      atomicMax(&S.max_level, meta.w & 255);
    }
  }
  __syncthreads();
  const int ni = S.n_inner;
  for (int l = S.max_level, left = ni; left > 0; --l) {
    int done = 0;
    for (int i0 = 0; i0 < ni; i0 += nthr) {
      const int e = i0 + tid < ni ? S.inner[i0 + tid] : -1;
      const bool mine = e >= 0 && (e & 255) == l;
      if (mine) {
        const int q = e >> 8, end = S.skip[q];
        NodeSums r;
        for (int c = q + 1; c < end; c = S.skip[c])
          r.add(S.m[0][c], S.m[1][c], S.m[2][c], S.m[3][c], S.lo[0][c], S.lo[1][c], S.lo[2][c],
                S.hi[0][c], S.hi[1][c], S.hi[2][c]);
        keep(q, r);
      }
      done += __syncthreads_count(mine);
    }
    left -= done;
  }
  __syncthreads();
}

constexpr int kTopBlock = 1024;
constexpr int kSmallNodes = 2048, kSubNodes = 512;
__global__ __launch_bounds__(kTopBlock) void k_moments_small(const Moments A, int nnodes) {
  __shared__ MomLds<kSmallNodes> S;
  lds_moments(A, 0, nnodes, S);
}

__global__ __launch_bounds__(kBlock) void k_moments_sub(const Moments A,
                                                        const int32_t *__restrict__ subs,
                                                        const int32_t *__restrict__ counts) {
  __shared__ MomLds<kSubNodes> S;
  const int nsub = counts[0];
  for (int b = (int)blockIdx.x; b < nsub; b += (int)gridDim.x) {
    const int k0 = subs[b];
    const int4 m0 = A.nodes[k0].meta;
    const int k1 = m0.x, lv0 = m0.w & 255;
    if (k1 - k0 <= kSubNodes) {
      lds_moments(A, k0, k1 - k0, S);
      continue;
    }
    // small leaves or long chains of single children: from memory
    if (threadIdx.x == 0) S.max_level = lv0;
    __syncthreads();
    for (int k = k0 + (int)threadIdx.x; k < k1; k += kBlock) {
      const int4 meta = A.nodes[k].meta;
      if (meta.w & kLeafBit) node_moments(A, k, meta);
      else atomicMax(&S.max_level, meta.w & 255);
    }
    __syncthreads();
    for (int l = S.max_level; l >= lv0; --l) {
      for (int k = k0 + (int)threadIdx.x; k < k1; k += kBlock) {
        const int4 meta = A.nodes[k].meta;
        if (!(meta.w & kLeafBit) && (meta.w & 255) == l) node_moments(A, k, meta);
      }
      __syncthreads();
    }
  }
}

// The nodes above the subtrees, level by level: eight threads a node read its
// children, one adds them up in their order.
constexpr int kTopList = 4096, kTopNodes = kTopBlock / 8;
__global__ __launch_bounds__(kTopBlock) void k_moments_top(const Moments A,
                                                           const TopNode *__restrict__ tops,
                                                           const int32_t *__restrict__ counts) {
  __shared__ int32_t order[kTopList];
  __shared__ int32_t start[kMaxLevel + 2], fill[kMaxLevel + 2];
  __shared__ double m[4][kTopBlock];
  __shared__ float lo[3][kTopBlock], hi[3][kTopBlock];
  __shared__ int32_t nchild[kTopNodes];
  const int n = counts[1], tid = (int)threadIdx.x;
  if (n > kTopList) {  // (trees of some 10^7 particles)
    for (int l = kMaxLevel; l >= 0; --l) {
      for (int i = tid; i < n; i += kTopBlock)
        if (tops[i].level == l) node_moments(A, tops[i].node, A.nodes[tops[i].node].meta);
      __syncthreads();
    }
    return;
  }
  if (tid < kMaxLevel + 2) fill[tid] = 0;
  __syncthreads();
  for (int i = tid; i < n; i += kTopBlock) atomicAdd(&fill[tops[i].level], 1);
  __syncthreads();
  if (tid == 0)
    for (int l = 0, at = 0; l < kMaxLevel + 2; ++l) {
      const int c = fill[l];
      start[l] = fill[l] = at;
      at += c;
    }
  __syncthreads();
  for (int i = tid; i < n; i += kTopBlock) order[atomicAdd(&fill[tops[i].level], 1)] = i;
  __syncthreads();
  for (int l = kMaxLevel; l >= 0; --l) {
    const int b = start[l], e = start[l + 1];
    for (int i0 = b; i0 < e; i0 += kTopNodes) {
      const int i = i0 + (tid >> 3);
      const int c = i < e ? tops[order[i]].child[tid & 7] : -1;
      if (c >= 0) {
        const double4 cm = A.mom[c];
        const float4 cl = A.nodes[c].lo_h, ch = A.nodes[c].hi_l;
        m[0][tid] = cm.x; m[1][tid] = cm.y; m[2][tid] = cm.z; m[3][tid] = cm.w;
        lo[0][tid] = cl.x; lo[1][tid] = cl.y; lo[2][tid] = cl.z;
        hi[0][tid] = ch.x; hi[1][tid] = ch.y; hi[2][tid] = ch.z;
      }
      const int have = __popcll(__ballot(c >= 0) & (0xffull << (tid & 56)));
      if ((tid & 7) == 0) nchild[tid >> 3] = have;
      __syncthreads();
      if (tid < kTopNodes && i0 + tid < e) {
        NodeSums r;
        for (int q = 8 * tid; q < 8 * tid + nchild[tid]; ++q)
          r.add(m[0][q], m[1][q], m[2][q], m[3][q], lo[0][q], lo[1][q], lo[2][q], hi[0][q],
                hi[1][q], hi[2][q]);
        store_node(A, tops[order[i0 + tid]].node, r);
      }
      __syncthreads();
    }
  }
}

// Bottom-up pass for one level: maximum h of the members (vh.w).
__global__ void k_hmax_level(Node *__restrict__ nodes, int64_t nnodes,
                             const float4 *__restrict__ vh, int level) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nnodes) return;
  const int4 meta = nodes[k].meta;
  if ((meta.w & 255) != level) return;
  float hm = 0.f;
  if (meta.w & kLeafBit) {
    for (int s = meta.y; s < meta.y + meta.z; ++s) hm = fmaxf(hm, vh[s].w);
  } else {
    int64_t c = k + 1;
    while (c < meta.x) {
      hm = fmaxf(hm, nodes[c].lo_h.w);
      c = nodes[c].meta.x;
    }
  }
  nodes[k].lo_h.w = hm;
}

inline unsigned nblk(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// The largest |coordinate| of the FP64 positions, as float bits (the FP32
// rounding upwards keeps it an upper bound); *out must start at zero. A
// grid-stride loop with one atomic per block: a few thousand atomics on the
// one word instead of one per wave.
constexpr int kAbsmaxBlocks = 2048;
__global__ __launch_bounds__(kBlock) void k_absmax(const double4 *__restrict__ x64, int64_t n,
                                                   unsigned *__restrict__ out) {
  __shared__ float part[kBlock / kWave];
  float m = 0.0f;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double4 v = x64[i];
    const double a = fmax(fabs(v.x), fmax(fabs(v.y), fabs(v.z)));
    float f = (float)a;
    if ((double)f < a) f = nextafterf(f, INFINITY);
    m = fmaxf(m, f);
  }
#pragma unroll
  for (int k = 1; k < kWave; k <<= 1) m = fmaxf(m, __shfl_xor(m, k));
  if ((threadIdx.x & 63u) == 0u) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kBlock / kWave; ++w) m = fmaxf(m, part[w]);
    if (m > 0.0f) atomicMax(out, __float_as_uint(m));
  }
}

__global__ void k_zero_one(unsigned *p) {
  if (threadIdx.x == 0) *p = 0u;
}

// ---- terminal lists (see Terms)

constexpr int kTermPer = 8;  // nodes per thread
constexpr int kTermTile = kBlock * kTermPer;

__device__ __forceinline__ int block_sum(int v, int *lds /* [kBlock / kWave] */) {
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) v += __shfl_xor(v, d);
  if ((threadIdx.x & 63u) == 0u) lds[threadIdx.x >> 6] = v;
  __syncthreads();
  int t = 0;
#pragma unroll
  for (int k = 0; k < kBlock / kWave; ++k) t += lds[k];
  __syncthreads();
  return t;
}

__global__ __launch_bounds__(kBlock) void k_term_count(const uint32_t *__restrict__ tcode,
                                                       int nn, int walk_leaf,
                                                       int32_t *__restrict__ bcount) {
  __shared__ int lds[kBlock / kWave];
  int c = 0;
  for (int q = 0; q < kTermPer; ++q) {
    const int k = (int)blockIdx.x * kTermTile + q * kBlock + (int)threadIdx.x;
    if (k < nn && is_terminal(tcode[k], walk_leaf)) ++c;
  }
  c = block_sum(c, lds);
  if (threadIdx.x == 0) bcount[blockIdx.x] = c;
}

// The indices of the terminals among the nodes [k0, k0 + kThreads kTermPer), in
// tree order from `base` on, and each snapshot's range of them: a snapshot's root
// sets its first one and the end of the snapshot before it. Returns the end.
template <int kThreads>
__device__ __forceinline__ int write_terms(const uint32_t *__restrict__ tcode, int nn,
                                           int walk_leaf, int k0, int base,
                                           const int32_t *__restrict__ nroot, int n_snap,
                                           int32_t *tnode, int32_t *__restrict__ tcount,
                                           int2 *__restrict__ range,
                                           int *lds /* [kThreads / kWave] */) {
  const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
  for (int q = 0; q < kTermPer && k0 + q * kThreads < nn; ++q) {
    const int k = k0 + q * kThreads + (int)threadIdx.x;
    const uint32_t code = k < nn ? tcode[k] : 0u;
    const bool f = k < nn && is_terminal(code, walk_leaf);
    const uint64_t m = __ballot(f);
    if (lane == 0) lds[w] = __popcll(m);
    __syncthreads();
    int at = base, tot = 0;
#pragma unroll
    for (int v = 0; v < kThreads / kWave; ++v) {
      if (v < w) at += lds[v];
      tot += lds[v];
    }
    at += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                         __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
    if (f) tnode[at] = k;
    if (is_root(code)) {
      if (n_snap == 1) {
        range[0].x = at;
      } else {
        range[segment_of(nroot, n_snap, k)].x = at;
        if (k > 0) range[segment_of(nroot, n_snap, k - 1)].y = at;
      }
    }
    if (k == nn - 1) {
      const int end = at + (f ? 1 : 0);
      *tcount = end;
      range[n_snap == 1 ? 0 : segment_of(nroot, n_snap, k)].y = end;
    }
    base += tot;
    __syncthreads();
  }
  return base;
}

__global__ __launch_bounds__(kBlock) void k_term_write(
    const uint32_t *__restrict__ tcode, int nn, int walk_leaf, const int32_t *__restrict__ bcount,
    const int32_t *__restrict__ nroot, int n_snap, int32_t *__restrict__ tnode,
    int32_t *__restrict__ tcount, int2 *__restrict__ range) {
  __shared__ int lds[kBlock / kWave];
  int pre = 0;
  for (int b = (int)threadIdx.x; b < (int)blockIdx.x; b += kBlock) pre += bcount[b];
  const int base = block_sum(pre, lds);
  (void)write_terms<kBlock>(tcode, nn, walk_leaf, (int)blockIdx.x * kTermTile, base, nroot, n_snap,
                            tnode, tcount, range, lds);
}

// The subtree roots and the (node, level) above them, in tree order; counts
// [0] and [1]. The same two passes as the terminals.
__global__ __launch_bounds__(kBlock) void k_split_count(const uint32_t *__restrict__ tcode,
                                                        int nn, int2 *__restrict__ bcount) {
  __shared__ int lds[kBlock / kWave];
  int a = 0, b = 0;
  for (int q = 0; q < kTermPer; ++q) {
    const int k = (int)blockIdx.x * kTermTile + q * kBlock + (int)threadIdx.x;
    if (k >= nn) continue;
    const uint32_t code = tcode[k];
    a += is_terminal(code, kSubtree);
    b += (int)(code & 0xffffu) > kSubtree;
  }
  a = block_sum(a, lds);
  b = block_sum(b, lds);
  if (threadIdx.x == 0) bcount[blockIdx.x] = make_int2(a, b);
}

__global__ __launch_bounds__(kBlock) void k_split_write(const Node *__restrict__ nodes,
                                                        const uint32_t *__restrict__ tcode, int nn,
                                                        const int2 *__restrict__ bcount,
                                                        int32_t *__restrict__ subs,
                                                        TopNode *__restrict__ tops,
                                                        int32_t *__restrict__ counts) {
  __shared__ int lds[kBlock / kWave];
  __shared__ int na, nb;  // appended by this block
  int a = 0, b = 0;
  for (int k = (int)threadIdx.x; k < (int)blockIdx.x; k += kBlock) {
    a += bcount[k].x;
    b += bcount[k].y;
  }
  a = block_sum(a, lds);
  b = block_sum(b, lds);
  if (threadIdx.x == 0) na = nb = 0;
  __syncthreads();
  // (the order within a block does not matter: each entry is worked alone)
  for (int q = 0; q < kTermPer; ++q) {
    const int k = (int)blockIdx.x * kTermTile + q * kBlock + (int)threadIdx.x;
    if (k >= nn) continue;
    const uint32_t code = tcode[k];
    if (is_terminal(code, kSubtree)) subs[a + atomicAdd(&na, 1)] = k;
    if ((int)(code & 0xffffu) > kSubtree) {
      const int4 meta = nodes[k].meta;
      TopNode t;
      t.node = k;
      t.level = meta.w & 255;
      int c = k + 1;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        t.child[j] = c < meta.x ? c : -1;
        if (c < meta.x) c = nodes[c].meta.x;
      }
      tops[b + atomicAdd(&nb, 1)] = t;
    }
  }
  __syncthreads();
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
    counts[0] = a + na;
    counts[1] = b + nb;
  }
}

// Boxes, first members and (vh given) largest h of the terminals and their
// windows: 16 lanes a terminal, a block a window. Bound by the latency of
// the members' loads; one launch, where a refit of every node's largest h
// takes one launch a level (11 of them, 5-6 us each, on 10^6 gas particles).
constexpr int kFillBlock = 1024;
struct WindowLds {
  float4 lo[kWave], hi[kWave];
};
__device__ __forceinline__ void fill_windows(const Node *__restrict__ nodes, const int32_t *tnode,
                                             int n, const float4 *__restrict__ vh, int m,
                                             float4 *__restrict__ lo, float4 *__restrict__ hi,
                                             float4 *__restrict__ wlo, float4 *__restrict__ whi,
                                             WindowLds &S) {
  const int sub = (int)(threadIdx.x & 15u), q = (int)(threadIdx.x >> 4);
  for (int b = (int)blockIdx.x; b * kWave < n; b += (int)gridDim.x) {
    const int t = b * kWave + q;
    float4 l = make_float4(INFINITY, INFINITY, INFINITY, 0.f);
    float4 h = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.f);
    if (t < n) {
      const Node &nd = nodes[tnode[t]];
      const int4 meta = nd.meta;
      l = nd.lo_h;
      h = nd.hi_l;
      float hm = 0.f;
      if (vh)
        for (int s = meta.y + sub; s < meta.y + meta.z; s += 16) hm = fmaxf(hm, vh[s].w);
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) hm = fmaxf(hm, __shfl_xor(hm, d));
      l.w = hm;
      h.w = __int_as_float(meta.y);
      if (sub == 0) {
        lo[t] = l;
        hi[t] = h;
        if (t == n - 1) hi[n] = make_float4(0.f, 0.f, 0.f, __int_as_float(m));
      }
    }
    if (sub == 0) {
      S.lo[q] = l;
      S.hi[q] = h;
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)kWave) {
      float4 a = S.lo[threadIdx.x], c = S.hi[threadIdx.x];
#pragma unroll
      for (int d = 1; d < kWave; d <<= 1) {
        a.x = fminf(a.x, __shfl_xor(a.x, d));
        a.y = fminf(a.y, __shfl_xor(a.y, d));
        a.z = fminf(a.z, __shfl_xor(a.z, d));
        a.w = fmaxf(a.w, __shfl_xor(a.w, d));
        c.x = fmaxf(c.x, __shfl_xor(c.x, d));
        c.y = fmaxf(c.y, __shfl_xor(c.y, d));
        c.z = fmaxf(c.z, __shfl_xor(c.z, d));
      }
      if (threadIdx.x == 0) {
        wlo[b] = a;
        whi[b] = c;
      }
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kFillBlock) void k_term_fill(
    const Node *__restrict__ nodes, const int32_t *__restrict__ tnode,
    const int32_t *__restrict__ tcount, const float4 *__restrict__ vh, int m,
    float4 *__restrict__ lo, float4 *__restrict__ hi, float4 *__restrict__ wlo,
    float4 *__restrict__ whi) {
  __shared__ WindowLds S;
  fill_windows(nodes, tnode, *tcount, vh, m, lo, hi, wlo, whi, S);
}

// The whole list of a small tree by one workgroup, one launch for three (us, with
// the tree walk that the lists replaced, with three launches, with one: velocity
// gradients of one particle 60, 75, 67, of 100 68, 77, 73; density of one particle
// 79, 88, 80).
constexpr int kSmallTerms = kSmallNodes;
__global__ __launch_bounds__(kFillBlock) void k_term_small(
    const Node *__restrict__ nodes, const uint32_t *__restrict__ tcode, int nn, int walk_leaf,
    const int32_t *__restrict__ nroot, int n_snap, const float4 *__restrict__ vh, int m,
    int32_t *__restrict__ tcount, int2 *__restrict__ range, float4 *__restrict__ lo,
    float4 *__restrict__ hi, float4 *__restrict__ wlo, float4 *__restrict__ whi) {
  static_assert(kSmallTerms <= kFillBlock * kTermPer, "one pass over the nodes");
  __shared__ int32_t tnode[kSmallTerms];
  __shared__ int lds[kFillBlock / kWave];
  __shared__ WindowLds S;
  const int n = write_terms<kFillBlock>(tcode, nn, walk_leaf, 0, 0, nroot, n_snap, tnode, tcount,
                                        range, lds);
  fill_windows(nodes, tnode, n, vh, m, lo, hi, wlo, whi, S);
}

// Boxes and largest h of the blocks, a wave each.
__global__ __launch_bounds__(kWave) void k_term_blocks(const int32_t *__restrict__ tcount,
                                                       const float4 *__restrict__ wlo,
                                                       const float4 *__restrict__ whi,
                                                       float4 *__restrict__ blo,
                                                       float4 *__restrict__ bhi) {
  const int nw = (*tcount + kWave - 1) / kWave, lane = (int)threadIdx.x;
  for (int b = (int)blockIdx.x; b * kWave < nw; b += (int)gridDim.x) {
    const int k = min(b * kWave + lane, nw - 1);
    float4 a = wlo[k], c = whi[k];
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      a.x = fminf(a.x, __shfl_xor(a.x, d));
      a.y = fminf(a.y, __shfl_xor(a.y, d));
      a.z = fminf(a.z, __shfl_xor(a.z, d));
      a.w = fmaxf(a.w, __shfl_xor(a.w, d));
      c.x = fmaxf(c.x, __shfl_xor(c.x, d));
      c.y = fmaxf(c.y, __shfl_xor(c.y, d));
      c.z = fmaxf(c.z, __shfl_xor(c.z, d));
    }
    if (lane == 0) {
      blo[b] = a;
      bhi[b] = c;
    }
  }
}

// The gravity walk's node copies (after the moments): every internal node
// writes its children's, a root also its own.
__global__ void k_cnodes(const Node *__restrict__ nodes, const double4 *__restrict__ c64,
                         const uint64_t *__restrict__ keys, int64_t nnodes,
                         const uint32_t *__restrict__ cbase, const int32_t *__restrict__ nroot,
                         int n_snap, CNode *__restrict__ cnodes, uint64_t *__restrict__ ckeys,
                         double4 *__restrict__ cc64) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= nnodes) return;
  const Node me = nodes[k];
  auto put = [&](int64_t at, int64_t c, const Node &nd) {
    CNode g;
    g.com_m = nd.com_m;
    const bool leaf = nd.meta.w & kLeafBit;
    g.meta = make_int4(leaf ? nd.meta.y : (int)(cbase[c] + (uint32_t)n_snap),
                       leaf ? -nd.meta.z : (int)(cbase[c + 1] - cbase[c]), (int)c,
                       __float_as_int(nd.hi_l.w));
    cnodes[at] = g;
    ckeys[at] = keys[nd.meta.y];
    if (cc64) cc64[at] = c64[c];
  };
  if ((me.meta.w & 255) == 0) put(n_snap == 1 ? 0 : segment_of(nroot, n_snap, k), k, me);
  if (me.meta.w & kLeafBit) return;
  int64_t at = (int64_t)cbase[k] + n_snap;
  for (int64_t c = k + 1; c < me.meta.x; ++at) {
    const Node nd = nodes[c];
    put(at, c, nd);
    c = nd.meta.x;
  }
}

}  // namespace

static void launch_moments(const g3_tree *t, const Octree &o, hipStream_t s) {
  const Moments A{o.nodes, o.mom, t->f64 ? o.c64 : nullptr, o.xm, t->f64 ? o.x64 : nullptr};
  if (o.nnodes <= kSmallNodes) {
    k_moments_small<<<1, kTopBlock, 0, s>>>(A, (int)o.nnodes);
    return;
  }
  const unsigned nb = (unsigned)std::min<int64_t>(o.nnodes, 4096);
  k_moments_sub<<<nb, kBlock, 0, s>>>(A, o.subs, o.nsplit);
  k_moments_top<<<1, kTopBlock, 0, s>>>(A, o.tops, o.nsplit);
}

static void fill_cnodes(const g3_tree *t, const Octree &o, hipStream_t s) {
  k_cnodes<<<nblk(o.nnodes), kBlock, 0, s>>>(o.nodes, t->f64 ? o.c64 : nullptr, o.keys, o.nnodes,
                                             o.cbase, o.nroot, t->n_snap, o.cnodes, o.ckeys,
                                             t->f64 ? o.cc64 : nullptr);
}

// The all-particle octree: keys, sort, topology, moments and gravity's node copies,
// and which members are gas. The gas octree, built next: those members in the same
// order, topology and moments. SYNCS once to read the node count.
int build_octree(g3_ctx *c, g3_tree *t, Octree &o, const void *pos, int f64,
                 const float *mass, int64_t m, hipStream_t s, const uint8_t *type,
                 int64_t *m_gas) {
  o.n = m;
  o.nnodes = 0;
  o.max_level = 0;
  if (m_gas) *m_gas = 0;
  if (m == 0) {  // no members: every snapshot's node range is empty
    const hipError_t e = fill_i32(o.nroot, 0, t->n_snap + 1, s);
    if (e != hipSuccess) { c->err = "fill launch failed"; return G3_EHIP; }
    return G3_OK;
  }
  if (f64 && (!o.x64 || o.cap_x64 < m)) {
    if (o.x64) (void)hipFree(o.x64);
    o.x64 = nullptr;
    o.cap_x64 = 0;
    if (dev_malloc(c, (void **)&o.x64, m * sizeof(double4)) != hipSuccess) {
      c->err = "device allocation of the FP64 positions failed";
      return G3_ENOMEM;
    }
    o.cap_x64 = m;
  }
  double4 *x64 = f64 ? o.x64 : nullptr;
  if (m > o.cap_n) {
    for (void *p : {(void *)o.keys, (void *)o.perm, (void *)o.xm, (void *)o.vh, (void *)o.aux})
      if (p) (void)hipFree(p);
    o.keys = nullptr; o.perm = nullptr; o.xm = nullptr; o.vh = nullptr; o.aux = nullptr;
    o.cap_n = 0;
    if (dev_malloc(c, (void **)&o.keys, m * sizeof(uint64_t)) != hipSuccess ||
        dev_malloc(c, (void **)&o.perm, m * sizeof(int32_t)) != hipSuccess ||
        dev_malloc(c, (void **)&o.xm, m * sizeof(float4)) != hipSuccess ||
        dev_malloc(c, (void **)&o.vh, m * sizeof(float4)) != hipSuccess ||
        dev_malloc(c, (void **)&o.aux, m * sizeof(float4)) != hipSuccess) {
      c->err = "device allocation of the sorted particle arrays failed";
      return G3_ENOMEM;
    }
    o.cap_n = m;
  }
  uint32_t *cnt = (uint32_t *)scratch(c, kCounts, (m + 1) * sizeof(uint32_t));
  uint32_t *off = (uint32_t *)scratch(c, kOffsets, (m + 1) * sizeof(uint32_t));
  uint8_t *lev = (uint8_t *)scratch(c, kLevel, 2 * m);
  uint32_t *stmp = (uint32_t *)scratch(c, kScanTmp, scan_tmp_elems(m) * sizeof(uint32_t));
  int32_t *maxlev = (int32_t *)scratch(c, kMisc, 64);
  if (!cnt || !off || !lev || !stmp || !maxlev) {
    c->err = "device allocation of build scratch failed";
    return G3_ENOMEM;
  }
  const bool gas = (&o == &t->gas);
  const int64_t n = t->n;
  uint32_t *flags = (uint32_t *)scratch(c, kGasFlags, (n + 1) * sizeof(uint32_t));
  uint32_t *slot = (uint32_t *)scratch(c, kGasSlot, (n + 1) * sizeof(uint32_t));
  uint32_t *stmp2 = (uint32_t *)scratch(c, kGasScan, scan_tmp_elems(n) * sizeof(uint32_t));
  if (!flags || !slot || !stmp2) { c->err = "device allocation of build scratch failed"; return G3_ENOMEM; }
  hipError_t e;
  if (gas) {
    // the all-particle octree's sorted members (built just before, with the
    // flags and slots of the gas ones)
    k_compact_sorted<<<nblk(n), kBlock, 0, s>>>(flags, slot, n, t->all, o.keys, o.perm, o.xm, x64,
                                                 t->iperm_gas);
  } else {
    uint64_t *kalt = (uint64_t *)scratch(c, kSortKeys, m * sizeof(uint64_t));
    uint32_t *valt = (uint32_t *)scratch(c, kSortVals, m * sizeof(uint32_t));
    void *rtmp = scratch(c, kSortTmp, radix_tmp_bytes(m));
    uint32_t *vals = (uint32_t *)scratch(c, kIds, m * sizeof(uint32_t));
    if (!kalt || !valt || !rtmp || !vals) {
      c->err = "device allocation of build scratch failed";
      return G3_ENOMEM;
    }
    if (f64)
      k_keys<double><<<nblk(m), kBlock, 0, s>>>((const double *)pos, m, t->coff, t->sbox,
                                                t->n_snap, mass, o.keys, vals, nullptr);
    else  // (this octree's vh is free: the SPH calls fill the gas octree's)
      k_keys<float><<<nblk(m), kBlock, 0, s>>>((const float *)pos, m, t->coff, t->sbox, t->n_snap,
                                               mass, o.keys, vals, o.vh);
    e = radix_sort_pairs(o.keys, vals, kalt, valt, m, 64, rtmp, s);
    if (e != hipSuccess) { c->err = "radix sort launch failed"; return G3_EHIP; }
    if (t->n_snap > 1) {
      // stable sort of the key-sorted members by snapshot: (snapshot, key) order
      uint64_t *skey = (uint64_t *)scratch(c, kSnapKeys, 2 * m * sizeof(uint64_t));
      uint64_t *skey_alt = (uint64_t *)scratch(c, kSnapKeysAlt, m * sizeof(uint64_t));
      if (!skey || !skey_alt) { c->err = "device allocation of build scratch failed"; return G3_ENOMEM; }
      uint32_t *sidx = (uint32_t *)(skey + m);
      int bits = 8;
      while (bits < 32 && (int64_t(1) << bits) < t->n_snap) bits += 8;
      k_snap_keys<<<nblk(m), kBlock, 0, s>>>(vals, m, t->coff, t->n_snap, skey, sidx);
      e = radix_sort_pairs(skey, sidx, skey_alt, cnt, m, bits, rtmp, s);
      if (e != hipSuccess) { c->err = "radix sort launch failed"; return G3_EHIP; }
      k_gather_sorted<<<nblk(m), kBlock, 0, s>>>(sidx, m, o.keys, vals, kalt, valt);
      e = hipMemcpyAsync(o.keys, kalt, m * sizeof(uint64_t), hipMemcpyDeviceToDevice, s);
      if (e == hipSuccess)
        e = hipMemcpyAsync(vals, valt, m * sizeof(uint32_t), hipMemcpyDeviceToDevice, s);
      if (e != hipSuccess) { c->err = "snapshot sort copy failed"; return G3_EHIP; }
    }
    if (f64)
      k_permute<double><<<nblk(m), kBlock, 0, s>>>(vals, m, (const double *)pos, mass, o.xm, x64,
                                                   t->iperm_all, o.perm);
    else
      k_permute_packed<<<nblk(m), kBlock, 0, s>>>(vals, m, o.vh, o.xm, t->iperm_all, o.perm);
    // the gas members among the sorted ones: their number comes back with the
    // node count
    k_gas_of_sorted<<<nblk(n), kBlock, 0, s>>>(o.perm, n, type, flags);
    e = scan_u32(flags, slot, n, stmp2, s);
    if (e != hipSuccess) { c->err = "scan launch failed"; return G3_EHIP; }
    k_gas_soff<<<nblk(t->n_snap + 1), kBlock, 0, s>>>(o.soff, t->n_snap, slot, t->gas.soff);
  }
  e = fill_i32(maxlev, 0, 1, s);
  if (e != hipSuccess) { c->err = "fill launch failed"; return G3_EHIP; }
  k_node_counts<<<nblk(m), kBlock, 0, s>>>(o.keys, m, o.soff, t->n_snap, t->leaf, cnt, lev,
                                           maxlev);
  e = scan_u32(cnt, off, m, stmp, s);
  if (e != hipSuccess) { c->err = "scan launch failed"; return G3_EHIP; }
  int64_t *pin = c->pinned;
  e = hipMemcpyAsync(&pin[0], off + m, sizeof(uint32_t), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipMemcpyAsync(&pin[1], maxlev, sizeof(int32_t), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess && !gas)
    e = hipMemcpyAsync(&pin[2], slot + n, sizeof(uint32_t), hipMemcpyDeviceToHost, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) { c->err = std::string("node count readback: ") + hipGetErrorString(e); return G3_EHIP; }
  const int64_t nnodes = (int64_t)(uint32_t)(pin[0] & 0xffffffffll);
  const int32_t maxl = (int32_t)(pin[1] & 0xffffffffll);
  if (m_gas) *m_gas = (int64_t)(uint32_t)(pin[2] & 0xffffffffll);
  if (nnodes <= 0 || nnodes >= (int64_t)INT32_MAX) { c->err = "node count out of range"; return G3_EHIP; }
  const bool grav = (&o == &t->all);
  if (nnodes > o.cap_nodes || o.cap_tops < max_tops(o.cap_n)) {
    for (void *p : {(void *)o.nodes, (void *)o.mom, (void *)o.tops})
      if (p) (void)hipFree(p);
    o.nodes = nullptr; o.mom = nullptr; o.tops = nullptr; o.cap_nodes = 0;
    const int64_t cap = nnodes + nnodes / 8 + 64;
    // (the lists of the moments and the terminal codes in one buffer)
    if (dev_malloc(c, (void **)&o.nodes, cap * sizeof(Node)) != hipSuccess ||
        dev_malloc(c, (void **)&o.mom, cap * sizeof(double4)) != hipSuccess ||
        dev_malloc(c, (void **)&o.tops, max_tops(o.cap_n) * sizeof(TopNode) +
                                            (2 * cap + 2) * sizeof(int32_t)) != hipSuccess) {
      c->err = "device allocation of the octree nodes failed";
      return G3_ENOMEM;
    }
    o.cap_nodes = cap;
    o.cap_tops = max_tops(o.cap_n);
  }
  uint32_t *nch = nullptr, *ctmp = nullptr;
  if (grav) {
    const int64_t need = t->n_snap + nnodes + kChildPad;
    if (need > o.cap_cnodes) {
      for (void *p : {(void *)o.cnodes, (void *)o.ckeys, (void *)o.cbase})
        if (p) (void)hipFree(p);
      o.cnodes = nullptr; o.ckeys = nullptr; o.cbase = nullptr; o.cap_cnodes = 0;
      const int64_t cap = need + nnodes / 8 + 64;
      if (dev_malloc(c, (void **)&o.cnodes, cap * sizeof(CNode)) != hipSuccess ||
          dev_malloc(c, (void **)&o.ckeys, cap * sizeof(uint64_t)) != hipSuccess ||
          dev_malloc(c, (void **)&o.cbase, (cap + 1) * sizeof(uint32_t)) != hipSuccess) {
        c->err = "device allocation of the gravity nodes failed";
        return G3_ENOMEM;
      }
      o.cap_cnodes = cap;
    }
    if (f64 && need > o.cap_cc64) {
      if (o.cc64) (void)hipFree(o.cc64);
      o.cc64 = nullptr;
      o.cap_cc64 = 0;
      const int64_t cap = need + nnodes / 8 + 64;
      if (dev_malloc(c, (void **)&o.cc64, cap * sizeof(double4)) != hipSuccess) {
        c->err = "device allocation of the gravity nodes failed";
        return G3_ENOMEM;
      }
      o.cap_cc64 = cap;
    }
    nch = (uint32_t *)scratch(c, kChildren,
                              (nnodes + 1 + scan_tmp_elems(nnodes)) * sizeof(uint32_t));
    if (!nch) { c->err = "device allocation of build scratch failed"; return G3_ENOMEM; }
    ctmp = nch + nnodes + 1;
  }
  if (f64 && (!o.c64 || o.cap_c64 < nnodes)) {
    if (o.c64) (void)hipFree(o.c64);
    o.c64 = nullptr;
    o.cap_c64 = 0;
    const int64_t cap = nnodes + nnodes / 8 + 64;
    if (dev_malloc(c, (void **)&o.c64, cap * sizeof(double4)) != hipSuccess) {
      c->err = "device allocation of the FP64 node centres failed";
      return G3_ENOMEM;
    }
    o.cap_c64 = cap;
  }
  o.subs = (int32_t *)(o.tops + o.cap_tops);
  o.nsplit = o.subs + o.cap_nodes;
  o.tcode = (uint32_t *)(o.nsplit + 2);
  // per-block counts of the list pass
  int2 *bcount = (int2 *)scratch(c, kMisc, 64 + (nnodes / kTermTile + 2) * sizeof(int2));
  if (!bcount) { c->err = "device allocation of build scratch failed"; return G3_ENOMEM; }
  bcount += 8;
  o.nnodes = nnodes;
  o.max_level = maxl;
  k_nodes<<<nblk(m), kBlock, 0, s>>>(o.keys, m, o.soff, t->n_snap, t->sbox, off, lev, nnodes,
                                     o.nodes);
  k_nroot<<<nblk(t->n_snap + 1), kBlock, 0, s>>>(off, o.soff, t->n_snap, o.nroot);
  k_parents<<<nblk(nnodes), kBlock, 0, s>>>(o.nodes, nnodes, o.tcode, nch);
  if (nnodes > kSmallNodes) {
    const unsigned nb = (unsigned)((nnodes + kTermTile - 1) / kTermTile);
    k_split_count<<<nb, kBlock, 0, s>>>(o.tcode, (int)nnodes, bcount);
    k_split_write<<<nb, kBlock, 0, s>>>(o.nodes, o.tcode, (int)nnodes, bcount, o.subs, o.tops,
                                        o.nsplit);
  }
  launch_moments(t, o, s);
  if (grav) {
    e = scan_u32(nch, o.cbase, nnodes, ctmp, s);
    if (e != hipSuccess) { c->err = "scan launch failed"; return G3_EHIP; }
    fill_cnodes(t, o, s);
  }
  e = hipGetLastError();
  if (e != hipSuccess) { c->err = std::string("tree build launch: ") + hipGetErrorString(e); return G3_EHIP; }
  return G3_OK;
}

int refit_octree(g3_ctx *c, g3_tree *t, Octree &o, const void *pos, const float *mass,
                 hipStream_t s) {
  if (o.n == 0 || o.nnodes == 0) return G3_OK;
  // (the order and its inverse stay)
  const uint32_t *order = (const uint32_t *)o.perm;
  if (t->f64)
    k_permute<double><<<nblk(o.n), kBlock, 0, s>>>(order, o.n, (const double *)pos, mass, o.xm,
                                                   o.x64, nullptr, nullptr);
  else
    k_permute<float><<<nblk(o.n), kBlock, 0, s>>>(order, o.n, (const float *)pos, mass, o.xm,
                                                  nullptr, nullptr, nullptr);
  launch_moments(t, o, s);
  if (&o == &t->all) fill_cnodes(t, o, s);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    c->err = std::string("tree refit launch: ") + hipGetErrorString(e);
    return G3_EHIP;
  }
  return G3_OK;
}

hipError_t update_absmax(g3_tree *t, hipStream_t s) {
  if (!t->f64 || !t->absmax) return hipSuccess;
  k_zero_one<<<1, 64, 0, s>>>(t->absmax);
  if (t->all.n > 0) {
    const unsigned nb = (unsigned)std::min<int64_t>(nblk(t->all.n), kAbsmaxBlocks);
    k_absmax<<<nb, kBlock, 0, s>>>(t->all.x64, t->all.n, t->absmax);
  }
  return hipGetLastError();
}

hipError_t refit_hmax(Octree &o, hipStream_t s) {
  for (int l = o.max_level; l >= 0 && o.nnodes > 0; --l)
    k_hmax_level<<<nblk(o.nnodes), kBlock, 0, s>>>(o.nodes, o.nnodes, o.vh, l);
  return hipGetLastError();
}

bool reserve_terms(g3_ctx *c, const Octree &o, int n_snap, TermBufs *b) {
  const size_t nn = (size_t)o.nnodes, nw = nn / kWave + 2, nb = nn / kTermTile + 2;
  const size_t nblocks = nw / kWave + 1, f4 = 2 * (nn + 1) + 2 * nw + 2 * nblocks;
  char *p = (char *)scratch(c, kTermBuf, f4 * sizeof(float4) + (size_t)n_snap * sizeof(int2) +
                                             (nn + nb + 4) * sizeof(int32_t));
  if (!p) return false;
  b->lo = (float4 *)p;
  b->hi = b->lo + nn + 1;
  b->wlo = b->hi + nn + 1;
  b->whi = b->wlo + nw;
  b->blo = b->whi + nw;
  b->bhi = b->blo + nblocks;
  b->range = (int2 *)(b->bhi + nblocks);
  b->node = (int32_t *)(b->range + n_snap);
  b->bcount = b->node + nn;
  b->count = b->bcount + nb;
  return true;
}

hipError_t build_terms(const Octree &o, int n_snap, int walk_leaf, bool with_h, const TermBufs &b,
                       hipStream_t s) {
  if (o.nnodes == 0) return hipSuccess;
  const int nn = (int)o.nnodes;
  if (nn <= kSmallTerms) {
    k_term_small<<<1, kFillBlock, 0, s>>>(o.nodes, o.tcode, nn, walk_leaf, o.nroot, n_snap,
                                          with_h ? o.vh : nullptr, (int)o.n, b.count, b.range,
                                          b.lo, b.hi, b.wlo, b.whi);
  } else {
    const unsigned nb = (unsigned)((nn + kTermTile - 1) / kTermTile);
    k_term_count<<<nb, kBlock, 0, s>>>(o.tcode, nn, walk_leaf, b.bcount);
    k_term_write<<<nb, kBlock, 0, s>>>(o.tcode, nn, walk_leaf, b.bcount, o.nroot, n_snap, b.node,
                                       b.count, b.range);
    const unsigned nf = (unsigned)std::min<int64_t>((nn + kWave - 1) / kWave, 512);
    k_term_fill<<<nf, kFillBlock, 0, s>>>(o.nodes, b.node, b.count, with_h ? o.vh : nullptr,
                                          (int)o.n, b.lo, b.hi, b.wlo, b.whi);
  }
  if (b.deep)
    k_term_blocks<<<(unsigned)(nn / (kWave * kWave) + 1), kWave, 0, s>>>(b.count, b.wlo, b.whi,
                                                                         b.blo, b.bhi);
  return hipGetLastError();
}

// The snapshot tables on the device. One snapshot's come from the launch's
// arguments; more are copied, and the copies waited for (the host staging is
// the caller's).
hipError_t upload_snapshots(g3_tree *t, const double4 *boxes, hipStream_t s) {
  if (t->n_snap == 1) {
    k_one_snap<<<1, 1, 0, s>>>(t->n, boxes[0], t->coff, t->sbox, t->all.soff);
    return hipGetLastError();
  }
  hipError_t e = hipMemcpyAsync(t->coff, t->snap_off.data(), (t->n_snap + 1) * sizeof(int64_t),
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess)
    e = hipMemcpyAsync(t->sbox, boxes, t->n_snap * sizeof(double4), hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  k_soff<<<nblk(t->n_snap + 1), kBlock, 0, s>>>(t->coff, t->n_snap, t->all.soff);
  return hipGetLastError();
}

}  // namespace g3
