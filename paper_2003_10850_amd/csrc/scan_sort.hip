// Device-wide exclusive scan and stable LSD radix sort of (u64 key, u32 value)
// pairs: the primitives of the octree build and the active-set compaction.
#include "g3_device.h"
#include "g3_internal.h"

namespace g3 {

namespace {

constexpr int kScanBlock = 256;
constexpr int kScanIpt = 8;
constexpr int kScanTile = kScanBlock * kScanIpt;

template <typename T>
__device__ T wave_incl_scan(T v) {
  const int lane = lane_id();
#pragma unroll
  for (int d = 1; d < kWave; d <<= 1) {
    T o = __shfl_up(v, (unsigned)d, kWave);
    if (lane >= d) v += o;
  }
  return v;
}

// Exclusive block scan of one value per thread; *total receives the sum.
template <typename T, int kBlock = kScanBlock>
__device__ T block_excl_scan(T v, T *total, T *lds /* [kBlock/64 + 1] */) {
  const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
  constexpr int kW = kBlock / kWave;
  T inc = wave_incl_scan(v);
  if (lane == kWave - 1) lds[w] = inc;
  __syncthreads();
  if (w == 0) {
    T t = lane < kW ? lds[lane] : T(0);
    T ti = wave_incl_scan(t);
    if (lane < kW) lds[lane] = ti - t;
    if (lane == kW - 1) lds[kW] = ti;
  }
  __syncthreads();
  const T res = lds[w] + inc - v;
  *total = lds[kW];
  __syncthreads();
  return res;
}

template <typename TI, typename TO>
__global__ __launch_bounds__(kScanBlock) void k_scan_reduce(const TI *__restrict__ in,
                                                            int64_t n, TO *__restrict__ part) {
  __shared__ TO lds[kScanBlock / kWave + 1];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanIpt;
  TO s = 0;
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k)
    if (base + k < n) s += (TO)in[base + k];
  TO tot;
  block_excl_scan<TO>(s, &tot, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

// The exclusive scan of one value per thread over all blocks. part: the blocks'
// sums (null for a single block), scanned already or (raw) added up here by
// every block for itself, in the barriers of its own scan. That takes a launch
// off a scan (4 us in a chain of small kernels); up to kRawParts blocks, 8e6
// items, it reads at most 16 values a thread.
constexpr int64_t kRawParts = 4096;
template <typename T>
__device__ T grid_excl_scan(T v, const T *__restrict__ part, int raw,
                            T *lds /* [2 kScanBlock/64 + 1] */) {
  const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
  constexpr int kW = kScanBlock / kWave;
  T before = 0;
  if (part) {
    if (raw)
      for (unsigned k = threadIdx.x; k < blockIdx.x; k += kScanBlock) before += part[k];
    else if (threadIdx.x == 0)
      before = part[blockIdx.x];
  }
  const T inc = wave_incl_scan(v), binc = wave_incl_scan(before);
  if (lane == kWave - 1) {
    lds[w] = inc;
    lds[kW + w] = binc;
  }
  __syncthreads();
  if (w == 0) {
    const T t = lane < 2 * kW ? lds[lane] : T(0);
    const T ti = wave_incl_scan(t);
    // all of the earlier blocks, the earlier waves of this one
    const T all = __shfl(ti, 2 * kW - 1, kWave) - __shfl(ti, kW - 1, kWave);
    if (lane < kW) lds[lane] = all + ti - t;
  }
  __syncthreads();
  return lds[w] + inc - v;
}

// Scans in[0..n) into out[0..n]; out may alias in (each thread reads its
// items before writing them). part: the blocks' sums (raw or scanned) or null.
template <typename TI, typename TO>
__global__ __launch_bounds__(kScanBlock) void k_scan_down(const TI *in, int64_t n, TO *out,
                                                          const TO *__restrict__ part, int raw) {
  __shared__ TO lds[2 * kScanBlock / kWave];
  const int64_t base = (int64_t)blockIdx.x * kScanTile + (int64_t)threadIdx.x * kScanIpt;
  TO v[kScanIpt];
  TO s = 0;
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) {
    v[k] = (base + k < n) ? (TO)in[base + k] : TO(0);
    s += v[k];
  }
  TO run = grid_excl_scan<TO>(s, part, raw, lds);
#pragma unroll
  for (int k = 0; k < kScanIpt; ++k) {
    if (base + k <= n) out[base + k] = run;
    run += v[k];
  }
}

// The whole scan by one workgroup of 1024, tile after tile: one launch.
constexpr int kOneBlock = 1024;
constexpr int64_t kOneItems = 2 * kOneBlock * kScanIpt;
template <typename TI, typename TO>
__global__ __launch_bounds__(kOneBlock) void k_scan_one(const TI *in, int n, TO *out) {
  __shared__ TO lds[kOneBlock / kWave + 1];
  TO carry = 0;
  for (int k0 = 0; k0 <= n; k0 += kOneBlock * kScanIpt) {
    const int base = k0 + (int)threadIdx.x * kScanIpt;
    TO v[kScanIpt];
    TO s = 0;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      v[k] = (base + k < n) ? (TO)in[base + k] : TO(0);
      s += v[k];
    }
    TO tot;
    TO run = carry + block_excl_scan<TO, kOneBlock>(s, &tot, lds);
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      if (base + k <= n) out[base + k] = run;
      run += v[k];
    }
    carry += tot;
  }
}

// One launch up to 2^14 items (two tiles of one workgroup: 5 us, as two
// launches of many cost 2 x 4), two up to kRawParts blocks.
template <typename TI, typename TO>
hipError_t scan_impl(const TI *in, TO *out, int64_t n, TO *tmp, hipStream_t s) {
  const int64_t nb = (n + 1 + kScanTile - 1) / kScanTile;
  if (nb == 1) {
    k_scan_down<TI, TO><<<1, kScanBlock, 0, s>>>(in, n, out, nullptr, 0);
    return hipGetLastError();
  }
  if (n < kOneItems) {
    k_scan_one<TI, TO><<<1, kOneBlock, 0, s>>>(in, (int)n, out);
    return hipGetLastError();
  }
  const int raw = nb <= kRawParts ? 1 : 0;
  k_scan_reduce<TI, TO><<<(unsigned)nb, kScanBlock, 0, s>>>(in, n, tmp);
  if (!raw) {
    hipError_t e = scan_impl<TO, TO>(tmp, tmp, nb, tmp + nb + 1, s);
    if (e != hipSuccess) return e;
  }
  k_scan_down<TI, TO><<<(unsigned)nb, kScanBlock, 0, s>>>(in, n, out, tmp, raw);
  return hipGetLastError();
}

// ------------------------------------------------------------ target lists

// Member s of an octree is a target when it is marked (mark[s], its row
// rowp1[s] - 1) or, with a time-bin rule, when the bin of its particle is at
// least kmin (its row is the caller id).
struct MarkRule {
  const int32_t *perm, *bins;
  int32_t kmin;
  const uint32_t *mark;
  const int32_t *rowp1;
  __device__ bool on(int64_t s) const { return bins ? bins[perm[s]] >= kmin : mark[s] != 0u; }
  __device__ int32_t row(int64_t s) const { return bins ? perm[s] : rowp1[s] - 1; }
};

// A wave takes kScanIpt runs of 64 members (coalesced), ranked by ballots.
// Counting and placing instead of marking, scanning and compacting: two
// launches for five (one below a tile).
__global__ __launch_bounds__(kScanBlock) void k_mark_count(const MarkRule r, int64_t m,
                                                           uint32_t *__restrict__ part) {
  __shared__ uint32_t lds[kScanBlock / kWave + 1];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)w * (kWave * kScanIpt) + lane;
  uint32_t cnt = 0;
#pragma unroll
  for (int c = 0; c < kScanIpt; ++c) {
    const int64_t s = t0 + (int64_t)c * kWave;
    cnt += s < m && r.on(s) ? 1u : 0u;
  }
  uint32_t tot;
  (void)block_excl_scan<uint32_t>(cnt, &tot, lds);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(kScanBlock) void k_mark_place(
    const MarkRule r, int64_t m, const uint32_t *__restrict__ part, int raw,
    uint32_t *__restrict__ slot, int32_t *__restrict__ targets, int32_t *__restrict__ rows) {
  __shared__ uint32_t lds[2 * kScanBlock / kWave];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  const int64_t t0 = (int64_t)blockIdx.x * kScanTile + (int64_t)w * (kWave * kScanIpt) + lane;
  uint64_t on[kScanIpt];
  uint32_t cnt = 0;  // the wave's
#pragma unroll
  for (int c = 0; c < kScanIpt; ++c) {
    const int64_t s = t0 + (int64_t)c * kWave;
    on[c] = __ballot(s < m && r.on(s));
    cnt += (uint32_t)__popcll(on[c]);
  }
  // (a wave's count once, by its first lane: the other lanes' prefix includes it)
  uint32_t at = __shfl(grid_excl_scan<uint32_t>(lane == 0 ? cnt : 0u, part, raw, lds), 0, kWave);
#pragma unroll
  for (int c = 0; c < kScanIpt; ++c) {
    const int64_t s = t0 + (int64_t)c * kWave;
    const uint32_t mine =
        at + __builtin_amdgcn_mbcnt_hi((uint32_t)(on[c] >> 32),
                                       __builtin_amdgcn_mbcnt_lo((uint32_t)on[c], 0u));
    if (s <= m) slot[s] = mine;
    if ((on[c] >> lane) & 1ull) {
      targets[mine] = (int32_t)s;
      rows[mine] = r.row(s);
    }
    at += (uint32_t)__popcll(on[c]);
  }
}

// ------------------------------------------------------------ radix sort

constexpr int kRsBlock = 512;
constexpr int kRsWaves = kRsBlock / kWave;
constexpr int kRsChunks = 8;  // 64-item chunks per wave
constexpr int kRsTile = kRsBlock * kRsChunks;
constexpr int kRsBits = 8;
constexpr int kRsBins = 1 << kRsBits;

__global__ __launch_bounds__(kRsBlock) void k_rs_hist(const uint64_t *__restrict__ keys,
                                                      int64_t n, int shift,
                                                      uint32_t *__restrict__ hist, int nb) {
  __shared__ uint32_t cnt[kRsBins];
  if (threadIdx.x < kRsBins) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * kRsTile;
  for (int k = threadIdx.x; k < kRsTile; k += kRsBlock) {
    const int64_t i = base + k;
    if (i < n) atomicAdd(&cnt[(keys[i] >> shift) & (kRsBins - 1)], 1u);
  }
  __syncthreads();
  if (threadIdx.x < kRsBins) hist[(int64_t)threadIdx.x * nb + blockIdx.x] = cnt[threadIdx.x];
}

// Exclusive scan of each digit's counts over the blocks (a block a digit, in
// place) and the digit's total. The scatter adds the totals of the smaller
// digits itself, so a pass is three launches; a device-wide scan of the
// counts took it to five.
__global__ __launch_bounds__(kScanBlock) void k_rs_rows(uint32_t *__restrict__ hist, int nb,
                                                        uint32_t *__restrict__ total) {
  __shared__ uint32_t lds[kScanBlock / kWave + 1];
  uint32_t *row = hist + (int64_t)blockIdx.x * nb;
  uint32_t run = 0;
  for (int k0 = 0; k0 < nb; k0 += kScanTile) {
    uint32_t v[kScanIpt], s = 0;
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      const int i = k0 + (int)threadIdx.x * kScanIpt + k;
      v[k] = i < nb ? row[i] : 0u;
      s += v[k];
    }
    uint32_t tot, at = run + block_excl_scan<uint32_t>(s, &tot, lds);
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
      const int i = k0 + (int)threadIdx.x * kScanIpt + k;
      if (i < nb) row[i] = at;
      at += v[k];
    }
    run += tot;
  }
  if (threadIdx.x == 0) total[blockIdx.x] = run;
}

// Stable scatter: wave w ranks its 512 items chunk by chunk (lanes with equal
// digits found by eight ballots), waves are ordered by a per-digit prefix; the
// tile is put in order in LDS and written out from there, a digit's items side
// by side (16 on average: 128 bytes of keys). Bound by those writes: straight
// from the registers, in tiles of 2048, a pass over 2^21 pairs took 29 us
// (17 now).
__global__ __launch_bounds__(kRsBlock) void k_rs_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, int64_t n, int shift,
    const uint32_t *__restrict__ offs, const uint32_t *__restrict__ total, int nb) {
  __shared__ uint64_t sk[kRsTile];
  __shared__ uint32_t sv[kRsTile];
  __shared__ uint32_t cnt[kRsWaves][kRsBins];
  __shared__ uint32_t base[kRsBins];  // where the tile's place 0 would go, by digit
  __shared__ uint32_t lds[kRsBlock / kWave + 1];
  static_assert(kRsBlock >= kRsBins, "a thread a digit");
  const int w = (int)(threadIdx.x >> 6), lane = lane_id(), tid = (int)threadIdx.x;
  for (int i = tid; i < kRsWaves * kRsBins; i += kRsBlock) (&cnt[0][0])[i] = 0;
  uint32_t all, gbase = 0;
  {
    const uint32_t smaller = block_excl_scan<uint32_t, kRsBlock>(
        tid < kRsBins ? total[tid] : 0u, &all, lds);
    if (tid < kRsBins) gbase = smaller + offs[(int64_t)tid * nb + blockIdx.x];
  }
  const int64_t t0 = (int64_t)blockIdx.x * kRsTile + (int64_t)w * (kWave * kRsChunks);
  uint64_t key[kRsChunks];
  uint32_t val[kRsChunks], rank[kRsChunks];
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int c = 0; c < kRsChunks; ++c) {
    const int64_t i = t0 + (int64_t)c * kWave + lane;
    const bool valid = i < n;
    key[c] = valid ? kin[i] : 0ull;
    val[c] = valid ? vin[i] : 0u;
  }
#pragma unroll
  for (int c = 0; c < kRsChunks; ++c) {
    const bool valid = t0 + (int64_t)c * kWave + lane < n;
    const uint32_t d = (uint32_t)(key[c] >> shift) & (kRsBins - 1);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < kRsBits; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t bb = __ballot(bit);
      peers &= bit ? bb : ~bb;
    }
    const uint32_t below = (uint32_t)__popcll(peers & lt);
    const uint32_t prev = cnt[w][d];
    rank[c] = prev + below;
    wave_sync();
    if (valid && below == 0) cnt[w][d] = prev + (uint32_t)__popcll(peers);
    wave_sync();
  }
  __syncthreads();
  uint32_t run = 0;
  if (tid < kRsBins) {
#pragma unroll
    for (int ww = 0; ww < kRsWaves; ++ww) run += cnt[ww][tid];
  }
  uint32_t at = block_excl_scan<uint32_t, kRsBlock>(run, &all, lds);  // the digit's place
  if (tid < kRsBins) {
    base[tid] = gbase - at;
#pragma unroll
    for (int ww = 0; ww < kRsWaves; ++ww) {
      const uint32_t t = cnt[ww][tid];
      cnt[ww][tid] = at;
      at += t;
    }
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < kRsChunks; ++c) {
    if (t0 + (int64_t)c * kWave + lane < n) {
      const uint32_t d = (uint32_t)(key[c] >> shift) & (kRsBins - 1);
      const uint32_t pos = cnt[w][d] + rank[c];
      sk[pos] = key[c];
      sv[pos] = val[c];
    }
  }
  __syncthreads();
  for (uint32_t p = (uint32_t)tid; p < all; p += kRsBlock) {
    const uint64_t k = sk[p];
    const uint32_t to = base[(uint32_t)(k >> shift) & (kRsBins - 1)] + p;
    kout[to] = k;
    vout[to] = sv[p];
  }
}

// Up to kSmallSort pairs by one workgroup in LDS: the same stable passes with
// the same ranks, without a launch in between (three launches of 3-8 us a
// pass and the gaps between them otherwise: 125 us for 4096 pairs, 37 here).
constexpr int kSmallBlock = 1024;
constexpr int kSmallWaves = kSmallBlock / kWave;
constexpr int kSmallIpt = 8;
constexpr int kSmallSort = kSmallBlock * kSmallIpt;

__global__ __launch_bounds__(kSmallBlock) void k_rs_small(uint64_t *__restrict__ keys,
                                                          uint32_t *__restrict__ vals, int n,
                                                          int bits) {
  __shared__ uint64_t sk[kSmallSort];
  __shared__ uint32_t sv[kSmallSort];
  __shared__ uint32_t cnt[kSmallWaves][kRsBins];
  __shared__ uint32_t lds[kRsBins / kWave];
  const int w = (int)(threadIdx.x >> 6), lane = lane_id();
  const int per = (n + kSmallBlock - 1) / kSmallBlock;  // 64-item chunks of a wave
  const int t0 = w * per * kWave;
  const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
  uint64_t key[kSmallIpt];
  uint32_t val[kSmallIpt], rank[kSmallIpt];
#pragma unroll
  for (int c = 0; c < kSmallIpt; ++c) {
    const int i = t0 + c * kWave + lane;
    const bool valid = c < per && i < n;
    key[c] = valid ? keys[i] : 0ull;
    val[c] = valid ? vals[i] : 0u;
  }
  for (int shift = 0; shift < bits; shift += kRsBits) {
    for (int i = (int)threadIdx.x; i < kSmallWaves * kRsBins; i += kSmallBlock)
      (&cnt[0][0])[i] = 0;
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kSmallIpt; ++c) {
      if (c >= per) break;
      const bool valid = t0 + c * kWave + lane < n;
      const uint32_t d = (uint32_t)(key[c] >> shift) & (kRsBins - 1);
      uint64_t peers = __ballot(valid);
#pragma unroll
      for (int b = 0; b < kRsBits; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        peers &= bit ? bb : ~bb;
      }
      const uint32_t below = (uint32_t)__popcll(peers & lt);
      const uint32_t prev = cnt[w][d];
      rank[c] = prev + below;
      wave_sync();
      if (valid && below == 0) cnt[w][d] = prev + (uint32_t)__popcll(peers);
      wave_sync();
    }
    __syncthreads();
    // per digit: exclusive over the waves, then over the smaller digits
    uint32_t run = 0, inc = 0;
    if (threadIdx.x < (unsigned)kRsBins) {
#pragma unroll
      for (int ww = 0; ww < kSmallWaves; ++ww) {
        const uint32_t t = cnt[ww][threadIdx.x];
        cnt[ww][threadIdx.x] = run;
        run += t;
      }
      inc = wave_incl_scan(run);
      if (lane == kWave - 1) lds[w] = inc;
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)kRsBins) {
      uint32_t base = inc - run;
      for (int ww = 0; ww < w; ++ww) base += lds[ww];
#pragma unroll
      for (int ww = 0; ww < kSmallWaves; ++ww) cnt[ww][threadIdx.x] += base;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kSmallIpt; ++c)
      if (c < per && t0 + c * kWave + lane < n) {
        const uint32_t at = cnt[w][(uint32_t)(key[c] >> shift) & (kRsBins - 1)] + rank[c];
        sk[at] = key[c];
        sv[at] = val[c];
      }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < kSmallIpt; ++c) {
      const int i = t0 + c * kWave + lane;
      if (c < per && i < n) {
        key[c] = sk[i];
        val[c] = sv[i];
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kSmallIpt; ++c) {
    const int i = t0 + c * kWave + lane;
    if (c < per && i < n) {
      keys[i] = key[c];
      vals[i] = val[c];
    }
  }
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace

int64_t scan_tmp_elems(int64_t n) {
  int64_t total = 0;
  int64_t m = n;
  for (;;) {
    const int64_t nb = (m + 1 + kScanTile - 1) / kScanTile;
    if (nb == 1) break;
    total += nb + 1;
    m = nb;
  }
  return total + 1;
}

hipError_t scan_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *tmp,
                    hipStream_t s) {
  return scan_impl<uint32_t, uint32_t>(in, out, n, tmp, s);
}

hipError_t scan_i32_to_i64(const int32_t *in, int64_t *out, int64_t n, int64_t *tmp,
                           hipStream_t s) {
  return scan_impl<int32_t, int64_t>(in, out, n, tmp, s);
}

hipError_t list_targets(const int32_t *perm, int64_t m, const int32_t *bins, int32_t kmin,
                        const uint32_t *mark, const int32_t *rowp1, uint32_t *slot,
                        int32_t *targets, int32_t *rows, uint32_t *tmp, hipStream_t s) {
  const MarkRule r{perm, bins, kmin, mark, rowp1};
  const int64_t nb = (m + 1 + kScanTile - 1) / kScanTile;
  const int raw = nb <= kRawParts ? 1 : 0;
  if (nb > 1) {
    k_mark_count<<<(unsigned)nb, kScanBlock, 0, s>>>(r, m, tmp);
    if (!raw) {
      const hipError_t e = scan_u32(tmp, tmp, nb, tmp + nb + 1, s);
      if (e != hipSuccess) return e;
    }
  }
  k_mark_place<<<(unsigned)nb, kScanBlock, 0, s>>>(r, m, nb > 1 ? tmp : nullptr, raw, slot,
                                                   targets, rows);
  return hipGetLastError();
}

size_t radix_tmp_bytes(int64_t n) {
  const int64_t nb = (n + kRsTile - 1) / kRsTile;
  const int64_t h = nb * kRsBins;
  return (size_t)(h + kRsBins) * sizeof(uint32_t);
}

hipError_t radix_sort_pairs(uint64_t *keys, uint32_t *vals, uint64_t *keys_alt,
                            uint32_t *vals_alt, int64_t n, int bits, void *tmp, hipStream_t s) {
  if (n <= 1) return hipSuccess;
  if (n <= kSmallSort) {
    k_rs_small<<<1, kSmallBlock, 0, s>>>(keys, vals, (int)n, bits);
    return hipGetLastError();
  }
  const int64_t nb = (n + kRsTile - 1) / kRsTile;
  const int64_t h = nb * kRsBins;
  uint32_t *hist = (uint32_t *)tmp;
  uint32_t *total = hist + h;
  uint64_t *ka = keys, *kb = keys_alt;
  uint32_t *va = vals, *vb = vals_alt;
  int passes = 0;
  for (int shift = 0; shift < bits; shift += kRsBits, ++passes) {
    k_rs_hist<<<(unsigned)nb, kRsBlock, 0, s>>>(ka, n, shift, hist, (int)nb);
    k_rs_rows<<<kRsBins, kScanBlock, 0, s>>>(hist, (int)nb, total);
    k_rs_scatter<<<(unsigned)nb, kRsBlock, 0, s>>>(ka, va, kb, vb, n, shift, hist, total, (int)nb);
    std::swap(ka, kb);
    std::swap(va, vb);
  }
  if (passes & 1) {  // the result is in the alternate buffers: copy it back
    hipError_t e = hipMemcpyAsync(keys, keys_alt, n * sizeof(uint64_t), hipMemcpyDeviceToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(vals, vals_alt, n * sizeof(uint32_t), hipMemcpyDeviceToDevice, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

hipError_t fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_fill_i32<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(p, v, n);
  return hipGetLastError();
}

}  // namespace g3
