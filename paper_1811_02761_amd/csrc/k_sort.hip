// k_sort.hip -- stable sort of (63-bit key, 32-bit index) pairs.
//
// The paper's tree build spends most of its time in a key/value radix sort
// (Sec. 4.1). Large sets take a reduce-then-scan LSD radix sort with 8-bit
// digits and 8 passes, written for wave64: every pass is a per-tile digit
// histogram (LDS atomics), a per-digit exclusive scan over tiles, and a scatter
// whose in-tile rank comes from a wave-level multisplit (eight ballots give the
// lanes sharing a digit; their popcount below the lane is the rank). Ranks
// follow input position, so each pass is stable and equal keys keep their
// input order. Smaller sets are sorted in tiles (by counting, or by all digits
// in LDS) and the tiles merged four at a time.
#include <utility>

#include "nbody_internal.h"

namespace nb {

constexpr int kWaves = kSortThreads / 64;
// the scatter of a 4096-key tile runs 8 wavefronts of 8 keys per lane: two
// tiles (58 KB of LDS each) per CU keep 16 wavefronts resident (4 with 16
// keys per lane waited on the rank chain; 59 vs 73 us per pass at 2^23)
constexpr int kScatterThreads = 512;
constexpr int kWaveKeys = kSortTile / kWaves;  // 1024 keys per wave

// Lanes whose digit equals this lane's digit (among `valid` lanes).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, uint64_t valid) {
  uint64_t peers = valid;
#pragma unroll
  for (int b = 0; b < kSortBits; ++b) {
    const bool bit = (d >> b) & 1u;
    const uint64_t m = __ballot(bit);
    peers &= bit ? m : ~m;
  }
  return peers;
}

// Per-tile digit counts by LDS atomics (one per key, into the wave's own
// counters; the order of the additions does not matter).
__global__ __launch_bounds__(kSortThreads) void k_sort_hist(
    const uint64_t *__restrict__ keys, int64_t n, int shift, uint32_t *__restrict__ hist,
    int64_t nblk, const uint32_t *__restrict__ n_dev) {
  if (n_dev) n = min(n, (int64_t)*n_dev);  // a count known on the device only
  __shared__ uint32_t cnt[kWaves][kSortRadix];
  for (int t = threadIdx.x; t < kWaves * kSortRadix; t += kSortThreads) (&cnt[0][0])[t] = 0;
  __syncthreads();
  const int w = threadIdx.x >> 6;
  const int64_t base = blockIdx.x * (int64_t)kSortTile + w * kWaveKeys + lane_id();
#pragma unroll
  for (int it = 0; it < kWaveKeys / 64; ++it) {
    const int64_t i = base + it * 64;
    if (i < n) atomicAdd(&cnt[w][(uint32_t)(keys[i] >> shift) & (kSortRadix - 1)], 1u);
  }
  __syncthreads();
  for (int d = threadIdx.x; d < kSortRadix; d += kSortThreads) {
    uint32_t s = 0;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) s += cnt[q][d];
    hist[d * nblk + blockIdx.x] = s;
  }
}

// Block-wide exclusive scan of one value per thread (blockDim = kSortThreads).
__device__ __forceinline__ uint32_t block_excl_scan(uint32_t v, uint32_t *tot,
                                                    uint32_t *wsum) {
  const uint32_t inc = wave_incl_scan(v);
  const int w = threadIdx.x >> 6;
  if (lane_id() == 63) wsum[w] = inc;
  __syncthreads();
  uint32_t off = 0, all = 0;
  for (int q = 0; q < (int)(blockDim.x >> 6); ++q) {
    if (q < w) off += wsum[q];
    all += wsum[q];
  }
  if (tot) *tot = all;
  __syncthreads();
  return off + inc - v;
}

// One workgroup per digit: exclusive scan of hist[d][0..nblk) in place and
// the digit total.
__global__ __launch_bounds__(kSortThreads) void k_sort_scan(uint32_t *__restrict__ hist,
                                                             int64_t nblk,
                                                             uint32_t *__restrict__ totals) {
  __shared__ uint32_t wsum[kWaves];
  uint32_t *row = hist + blockIdx.x * nblk;
  const int64_t per = cdiv(nblk, kSortThreads);
  const int64_t b0 = threadIdx.x * per;
  uint32_t s = 0;
  for (int64_t k = b0; k < b0 + per && k < nblk; ++k) s += row[k];
  uint32_t tot;
  uint32_t run = block_excl_scan(s, &tot, wsum);
  for (int64_t k = b0; k < b0 + per && k < nblk; ++k) {
    const uint32_t v = row[k];
    row[k] = run;
    run += v;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = tot;
}

// Scatter of one tile: ranks as in the histogram pass (stable: wave, item,
// lane = input order), then the tile is reordered by digit in LDS and
// written out from there, so consecutive threads store consecutive
// addresses of each digit's run instead of 256 scattered runs per wave.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void k_sort_scatter(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin, int64_t n,
    int shift, const uint32_t *__restrict__ hist, int64_t nblk,
    const uint32_t *__restrict__ totals, uint64_t *__restrict__ kout,
    uint32_t *__restrict__ vout, const uint32_t *__restrict__ n_dev) {
  constexpr int kW = kThreads / 64;
  constexpr int kItems = kSortTile / kThreads;
  constexpr int kWK = kSortTile / kW;
  static_assert(kThreads >= kSortRadix, "one thread per digit");
  if (n_dev) n = min(n, (int64_t)*n_dev);
  __shared__ uint32_t cnt[kW][kSortRadix];
  __shared__ uint32_t dbase[kSortRadix];   // global start of each digit's run of this tile
  __shared__ uint32_t lstart[kSortRadix];  // tile-local start of each digit
  __shared__ uint32_t wsum[kW];
  __shared__ uint64_t sk[kSortTile];
  __shared__ uint32_t sv[kSortTile];
  for (int t = threadIdx.x; t < kW * kSortRadix; t += kThreads) (&cnt[0][0])[t] = 0;
  // digit start = exclusive scan of totals; plus this tile's offset
  {
    const bool dig = threadIdx.x < (unsigned)kSortRadix;
    const uint32_t tv = dig ? totals[threadIdx.x] : 0u;
    const uint32_t ex = block_excl_scan(tv, nullptr, wsum);
    if (dig) dbase[threadIdx.x] = ex + hist[threadIdx.x * nblk + blockIdx.x];
  }
  __syncthreads();
  const int w = threadIdx.x >> 6;
  const int64_t tile0 = blockIdx.x * (int64_t)kSortTile;
  const int64_t base = tile0 + w * kWK;
  uint64_t k[kItems];
  uint32_t v[kItems];
  uint32_t r[kItems];
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int64_t i = base + it * 64 + lane_id();
    const bool valid = i < n;
    const uint64_t vmask = __ballot(valid);
    k[it] = valid ? kin[i] : 0ull;
    v[it] = valid ? vin[i] : 0u;
    const uint32_t d = (uint32_t)(k[it] >> shift) & (kSortRadix - 1);
    const uint64_t peers = match_digit(d, vmask);
    const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
    uint32_t c0 = 0;
    if (valid) c0 = cnt[w][d];
    r[it] = c0 + below;
    // every lane has read the counter before the digit's first lane bumps it
    __builtin_amdgcn_wave_barrier();
    if (valid && below == 0) cnt[w][d] = c0 + (uint32_t)__popcll(peers);
  }
  __syncthreads();
  // per digit: offsets of the waves within the tile's digit, then the
  // digit's start within the tile
  uint32_t tot = 0;
  if (threadIdx.x < (unsigned)kSortRadix) {
    const int d = threadIdx.x;
    uint32_t o = 0;
#pragma unroll
    for (int q = 0; q < kW; ++q) {
      const uint32_t t = cnt[q][d];
      cnt[q][d] = o;
      o += t;
    }
    tot = o;
  }
  const uint32_t ls = block_excl_scan(tot, nullptr, wsum);
  if (threadIdx.x < (unsigned)kSortRadix) lstart[threadIdx.x] = ls;
  __syncthreads();
#pragma unroll
  for (int it = 0; it < kItems; ++it) {
    const int64_t i = base + it * 64 + lane_id();
    if (i < n) {
      const uint32_t d = (uint32_t)(k[it] >> shift) & (kSortRadix - 1);
      const uint32_t lp = lstart[d] + cnt[w][d] + r[it];
      sk[lp] = k[it];
      sv[lp] = v[it];
    }
  }
  __syncthreads();
  const int64_t m = min((int64_t)kSortTile, n - tile0);  // valid items of the tile
  for (int j = threadIdx.x; j < m; j += kThreads) {
    const uint64_t key = sk[j];
    const uint32_t d = (uint32_t)(key >> shift) & (kSortRadix - 1);
    const uint32_t pos = dbase[d] + ((uint32_t)j - lstart[d]);
    kout[pos] = key;
    vout[pos] = sv[j];
  }
}

void launch_digit_sort(int64_t n, const uint32_t *n_dev, int shift, const uint64_t *kin,
                       const uint32_t *vin, uint64_t *kout, uint32_t *vout, uint32_t *hist,
                       hipStream_t st) {
  const int64_t nblk = cdiv(n, kSortTile);
  uint32_t *totals = hist + (int64_t)kSortRadix * nblk;
  hipLaunchKernelGGL(k_sort_hist, dim3(nblk), dim3(kSortThreads), 0, st, kin, n, shift, hist,
                     nblk, n_dev);
  hipLaunchKernelGGL(k_sort_scan, dim3(kSortRadix), dim3(kSortThreads), 0, st, hist, nblk,
                     totals);
  hipLaunchKernelGGL(k_sort_scatter<kScatterThreads>, dim3(nblk), dim3(kScatterThreads), 0, st,
                     kin, vin, n, shift, hist, nblk, totals, kout, vout, n_dev);
}

// One tile of kSortTile pairs sorted in LDS by all eight digits; 1024 threads,
// item `it` of thread t at position (t / 64) 256 + 64 it + t mod 64, so ranks in
// (wave, item, lane) order are stable. Values move as 16-bit tile positions.
constexpr int kTileThreads = 1024;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kTileItems = kSortTile / kTileThreads;
__global__ __launch_bounds__(kTileThreads) void k_sort_tile(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin, int64_t n,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout) {
  __shared__ uint64_t sk[kSortTile];
  __shared__ uint16_t si[kSortTile];
  __shared__ uint32_t cnt[kTileWaves][kSortRadix];
  __shared__ uint32_t wsum[kSortRadix / 64];
  const int64_t tile0 = blockIdx.x * (int64_t)kSortTile;
  const int m = (int)min((int64_t)kSortTile, n - tile0);
  const int w = threadIdx.x >> 6;
  const int p0 = w * (64 * kTileItems) + (int)lane_id();
  uint64_t k[kTileItems];
  uint32_t v[kTileItems], r[kTileItems];
#pragma unroll
  for (int it = 0; it < kTileItems; ++it) {
    const int p = p0 + 64 * it;
    k[it] = p < m ? kin[tile0 + p] : 0ull;
    v[it] = (uint32_t)p;
  }
  for (int shift = 0; shift < 64; shift += kSortBits) {
    for (int t = threadIdx.x; t < kTileWaves * kSortRadix; t += kTileThreads)
      (&cnt[0][0])[t] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kTileItems; ++it) {
      const bool valid = p0 + 64 * it < m;  // valid pairs stay in [0, m)
      const uint64_t vmask = __ballot(valid);
      const uint32_t d = (uint32_t)(k[it] >> shift) & (kSortRadix - 1);
      const uint64_t peers = match_digit(d, vmask);
      const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
      uint32_t c0 = 0;
      if (valid) c0 = cnt[w][d];
      r[it] = c0 + below;
      __builtin_amdgcn_wave_barrier();
      if (valid && below == 0) cnt[w][d] = c0 + (uint32_t)__popcll(peers);
    }
    __syncthreads();
    // per digit: the waves' offsets, then the digit's start in the tile
    uint32_t o = 0, inc = 0;
    if (threadIdx.x < (unsigned)kSortRadix) {
      const int d = threadIdx.x;
      uint32_t c[kTileWaves];
#pragma unroll
      for (int q = 0; q < kTileWaves; ++q) c[q] = cnt[q][d];
#pragma unroll
      for (int q = 0; q < kTileWaves; ++q) o += c[q];
      inc = wave_incl_scan_dpp(o);
      if (lane_id() == 63) wsum[w] = inc;
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)kSortRadix) {
      const int d = threadIdx.x;
      uint32_t at = inc - o;
      for (int q = 0; q < w; ++q) at += wsum[q];
#pragma unroll
      for (int q = 0; q < kTileWaves; ++q) {
        const uint32_t t = cnt[q][d];
        cnt[q][d] = at;
        at += t;
      }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kTileItems; ++it)
      if (p0 + 64 * it < m) {
        const uint32_t lp = cnt[w][(uint32_t)(k[it] >> shift) & (kSortRadix - 1)] + r[it];
        sk[lp] = k[it];
        si[lp] = (uint16_t)v[it];
      }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kTileItems; ++it) {
      const int p = p0 + 64 * it;
      if (p < m) {
        k[it] = sk[p];
        v[it] = si[p];
      }
    }
  }
#pragma unroll
  for (int it = 0; it < kTileItems; ++it) {
    const int p = p0 + 64 * it;
    if (p < m) {
      kout[tile0 + p] = k[it];
      vout[tile0 + p] = vin[tile0 + v[it]];
    }
  }
}

// Tiles of kTile pairs sorted by counting: a pair's place in its tile is the
// number of pairs there that come before it. A workgroup places 64 pairs (one per
// lane, the same ones in each wavefront), each wavefront counting over 256 pairs
// of the tile, staged in LDS (as scalar loads the keys came one latency after the
// other: 15 us instead of 8).
constexpr uint32_t kRankSlice = 256;
template <uint32_t kTile>
__global__ __launch_bounds__(kTile / kRankSlice * 64) void k_sort_rank(
    const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin, uint32_t n,
    uint64_t *__restrict__ kout, uint32_t *__restrict__ vout) {
  constexpr uint32_t kW = kTile / kRankSlice;
  __shared__ uint64_t slice[kW][kRankSlice];
  __shared__ uint32_t part[kW][64];
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = lane_id();
  const uint32_t i0 = blockIdx.x * 64u, tile0 = i0 / kTile * kTile;
  const uint32_t i = i0 + lane;
  const uint64_t key = i < n ? kin[i] : 0ull;
  const uint32_t b = tile0 + w * kRankSlice, e = min(max(n, b), b + kRankSlice);
  uint64_t *o = slice[w];
#pragma unroll
  for (uint32_t u = 0; u < kRankSlice / 64u; ++u) {
    const uint32_t j = b + 64u * u + lane;
    o[64u * u + lane] = j < e ? kin[j] : ~0ull;  // (before no key)
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  uint32_t c = 0;
  // 64 at a time: those of an earlier 64 come before equal keys, those of a later
  // one do not
  for (uint32_t q = 0; q < kRankSlice; q += 64u) {
    const uint32_t at = b + q;
    if (at >= e) break;
    if (at < i0) {
#pragma unroll 16
      for (uint32_t j = 0; j < 64u; ++j) c += o[q + j] <= key ? 1u : 0u;
    } else if (at > i0) {
#pragma unroll 16
      for (uint32_t j = 0; j < 64u; ++j) c += o[q + j] < key ? 1u : 0u;
    } else {
#pragma unroll 16
      for (uint32_t j = 0; j < 64u; ++j)
        c += (j < lane ? o[q + j] <= key : o[q + j] < key) ? 1u : 0u;
    }
  }
  if constexpr (kW > 1) {
    part[w][lane] = c;
    __syncthreads();
    if (w != 0u) return;
#pragma unroll
    for (uint32_t q = 1; q < kW; ++q) c += part[q][lane];
  }
  if (i < n) {
    kout[tile0 + c] = key;
    vout[tile0 + c] = vin[i];
  }
}

// Pairs of a run of len keys at r that come before `key` (equal keys too, if le),
// for two keys at once, found by a whole wavefront: 64 probes a round, three
// rounds for 2^18 keys.
__device__ __forceinline__ void wave_count_before(const uint64_t *__restrict__ r, uint32_t len,
                                                  const uint64_t (&key)[2], bool le,
                                                  uint32_t (&lo)[2]) {
  uint32_t m[2] = {len, len};
  lo[0] = lo[1] = 0u;
  while ((m[0] | m[1]) != 0u) {
    uint32_t step[2], c[2];
    uint64_t o[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      step[k] = (m[k] + 63u) / 64u;
      c[k] = (lane_id() + 1u) * step[k];
      o[k] = r[max(lo[k] + min(c[k], m[k]), 1u) - 1u];  // (in the run, which is not empty)
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const bool yes = c[k] <= m[k] && (le ? o[k] <= key[k] : o[k] < key[k]);
      const uint32_t t = m[k] ? (uint32_t)__popcll(__ballot(yes)) : 0u;
      lo[k] += t * step[k];
      m[k] = m[k] ? min(step[k] - 1u, m[k] - t * step[k]) : 0u;
    }
  }
}

// Merges groups of four sorted runs of `run` pairs (a power of two, 1024 or more):
// a pair's place is its place in its own run plus, for each other run of the
// group, the pairs there that come before it (equal keys: those of earlier runs,
// which keeps the sort stable). A workgroup's 256 pairs are neighbours in one run,
// so their answers lie between those of its first and its last pair: three
// wavefronts find these, the keys between go to LDS (or, if they are too many, are
// searched in memory), and every pair searches there. (A search of a whole run
// by every pair was a chain of up to 17 loads: 8.8, 11.2 and 15.0 us per merge at
// 16411, 50000 and 200003 pairs, 7.1, 10.1 and 12.0 this way.)
constexpr uint32_t kMergeStage = 2048;
__global__ __launch_bounds__(256) void k_sort_merge(const uint64_t *__restrict__ kin,
                                                    const uint32_t *__restrict__ vin, uint32_t n,
                                                    uint32_t run, uint64_t *__restrict__ kout,
                                                    uint32_t *__restrict__ vout) {
  __shared__ uint64_t stage[kMergeStage];
  __shared__ uint32_t s_lo[3], s_hi[3];
  const uint32_t i0 = blockIdx.x * 256u, i = i0 + threadIdx.x;  // (i0 < n)
  const uint32_t g0 = i0 / (4u * run) * (4u * run);
  const uint32_t mine = (i0 - g0) / run;
  const uint64_t key = kin[min(i, n - 1u)];
  const uint32_t vi = vin[min(i, n - 1u)];
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t b[3], len[3];
  bool le[3];
#pragma unroll
  for (uint32_t q = 0; q < 3; ++q) {
    const uint32_t s = q + (q >= mine ? 1u : 0u);
    b[q] = g0 + s * run;
    len[q] = b[q] < n ? min(n - b[q], run) : 0u;
    le[q] = s < mine;
  }
  const uint64_t ends[2] = {kin[i0], kin[min(i0 + 255u, n - 1u)]};
#pragma unroll
  for (uint32_t q = 0; q < 3; ++q)
    if (w == q) {
      uint32_t at[2];
      wave_count_before(kin + b[q], len[q], ends, le[q], at);
      s_lo[q] = at[0];
      s_hi[q] = at[1];
    }
  __syncthreads();
  uint32_t off[4] = {0u, 0u, 0u, 0u};
#pragma unroll
  for (uint32_t q = 0; q < 3; ++q) {
    b[q] += s_lo[q];
    len[q] = s_hi[q] - s_lo[q];
    off[q + 1] = off[q] + len[q];
  }
  const bool staged = off[3] <= kMergeStage;
  if (staged) {
#pragma unroll
    for (uint32_t q = 0; q < 3; ++q)
      for (uint32_t k = threadIdx.x; k < len[q]; k += 256u) stage[off[q] + k] = kin[b[q] + k];
    __syncthreads();
  }
  if (i >= n) return;
  const uint32_t most = max(max(len[0], len[1]), len[2]);
  uint32_t lo[3] = {0u, 0u, 0u};
  for (uint32_t step = most ? 1u << (31 - __builtin_clz(most)) : 0u; step >= 1u; step >>= 1) {
#pragma unroll
    for (uint32_t q = 0; q < 3; ++q) {
      const uint32_t c = lo[q] + step;  // are the first c pairs before mine?
      if (c <= len[q]) {
        const uint64_t o = staged ? stage[off[q] + c - 1u] : kin[b[q] + c - 1u];
        if (le[q] ? o <= key : o < key) lo[q] = c;
      }
    }
  }
  uint32_t at = i - mine * run;
#pragma unroll
  for (uint32_t q = 0; q < 3; ++q) at += s_lo[q] + lo[q];
  kout[at] = key;
  vout[at] = vi;
}

// Sorts by tiles and merges up to kMergeSort pairs. Tiles sorted by digits (a
// serial chain of eight passes, 30 to 35 us for any n) leave most of the chip
// idle below about 2*10^5 pairs; counting grows with n times the tile: 8 us for
// 1000 pairs, 11 for 16411 in tiles of 4096; at 2*10^5, 24 in tiles of 1024 and
// a merge of 10. All of a call's forces, us, digits / 4096 / 1024 wide tiles:
// 1000 particles 168 / 151 / 147, 16411 272 / 248 / 253, 32000 282 / 261 / 264,
// 65000 317 / 306 / 303, 130000 418 / 425 / 411, 200000 587 / 617 / 588.
constexpr int64_t kMergeSort = 1 << 20, kRankWide = 32768, kRankNarrow = 131072;

void launch_sort(int64_t n, uint64_t *keysA, uint32_t *valsA, uint64_t *keysB,
                 uint32_t *valsB, uint32_t *hist, hipStream_t st, uint64_t **keys_out,
                 uint32_t **vals_out) {
  uint64_t *ki = keysA, *ko = keysB;
  uint32_t *vi = valsA, *vo = valsB;
  if (n <= kMergeSort) {
    uint32_t run = kSortTile;
    const dim3 g64((unsigned)cdiv(n, 64));
    if (n <= 1024 || (n > kRankWide && n <= kRankNarrow)) {
      run = 1024;
      hipLaunchKernelGGL(k_sort_rank<1024>, g64, dim3(256), 0, st, ki, vi, (uint32_t)n, ko, vo);
    } else if (n <= kRankWide) {
      hipLaunchKernelGGL(k_sort_rank<4096>, g64, dim3(1024), 0, st, ki, vi, (uint32_t)n, ko, vo);
    } else {
      hipLaunchKernelGGL(k_sort_tile, dim3((unsigned)cdiv(n, kSortTile)), dim3(kTileThreads), 0,
                         st, ki, vi, n, ko, vo);
    }
    for (; run < n; run *= 4) {
      std::swap(ki, ko);
      std::swap(vi, vo);
      hipLaunchKernelGGL(k_sort_merge, dim3((unsigned)cdiv(n, 256)), dim3(256), 0, st, ki, vi,
                         (uint32_t)n, run, ko, vo);
    }
    *keys_out = ko;
    *vals_out = vo;
    return;
  }
  for (int pass = 0; pass < 8; ++pass) {
    launch_digit_sort(n, nullptr, pass * kSortBits, ki, vi, ko, vo, hist, st);
    std::swap(ki, ko);
    std::swap(vi, vo);
  }
  *keys_out = ki;
  *vals_out = vi;
}

}  // namespace nb
