// Stable sort of 32,769 and more (uint32 key, int32 index) pairs in three steps,
// of which two ride on other launches: keys and counts of their top nine bits per
// tile of 2,048, a stable scatter into 512 buckets, and a sort of each bucket in
// LDS by the remaining bits.
//
// What bounds it: the number of launches.  Two radix passes over 264,192 keys of
// 18 bits were eight launches (histogram, two of a scan, scatter, twice), 45 us of
// kernels; here 4 and 9 us more in the launches it rides on (8 and 16 us), and 9
// for the buckets.
//
// A bucket holds at most kBucketKeys keys.  On roots of up to 512 cells one of
// nodes holds 512 (and 2^19 targets make 1,024 on average); on a root of 1,024 it
// holds 2,048, and a body's targets come on top.  So 2,048 are sorted at once, and
// what is above (few buckets) as two runs that are then merged.  (A workgroup of
// 1,024 threads for 4,096 keys at once: a 600^2 node field 230 us, 219 so.)  A
// bucket that does not fit (targets crowded into a few cells) raises `skew`, and
// its keys come out as its lowest key, in order: the host then repeats the first
// segment with radix passes.
#pragma once

#include "blockscan.h"
#include "internal.h"
#include "runsort.h"

namespace pp {

constexpr int kBucketBlock = 256;
constexpr int kBucketRows = kBucketTile / kBucketBlock;
constexpr int kBucketWaves = kBucketBlock / kWave;
constexpr int kBucketSortBlock = 512;
constexpr int kBucketRun = kBucketSortBlock * kRunItems;
constexpr int kBucketKeys = 2 * kBucketRun;
static_assert(kBuckets == 2 * kBucketBlock, "two buckets per thread");

// Keys key_of(i), i in [0, n), of the tile at `first`, stored, and the tile's
// counts (h: kBuckets ints of LDS).
template <class KeyOf>
__device__ inline void bucket_count(int* h, KeyOf key_of, int first, int n, int shift, uint32_t* __restrict__ keys,
                                    int* __restrict__ hist) {
  const int t = threadIdx.x;
  h[2 * t] = h[2 * t + 1] = 0;
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kBucketRows; ++r) {
    const int i = r * kBucketBlock + t;
    if (i < n) {
      const uint32_t key = key_of(i);
      keys[first + i] = key;
      atomicAdd(&h[key >> shift], 1);
    }
  }
  __syncthreads();
  reinterpret_cast<int2*>(hist)[t] = make_int2(h[2 * t], h[2 * t + 1]);
}

// The tile's keys to their buckets, in input order within each.  hist: the
// tiles' counts; cnt: kBucketWaves * kBuckets ints of LDS; scan: kBucketWaves +
// 1.  Tile 0 stores the buckets' starts (kBuckets + 1) and *skew.
__device__ inline void bucket_scatter(int* cnt, int* scan, const uint32_t* __restrict__ keys, int total, int tile,
                                      int ntiles, int shift, const int* __restrict__ hist, int* __restrict__ starts,
                                      int* __restrict__ skew, uint32_t* __restrict__ kout, int* __restrict__ vout) {
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const uint64_t below = lane == 0 ? 0ull : (~0ull) >> (kWave - lane);
  const int first = tile * kBucketTile, n = min(kBucketTile, total - first);
  const int at = w * (kBucketRows * kWave) + lane;  // a wave owns kBucketRows consecutive rows of 64 keys
  uint32_t k[kBucketRows];
#pragma unroll
  for (int r = 0; r < kBucketRows; ++r) k[r] = keys[first + min(at + r * kWave, n - 1)];
  // the thread's two buckets: keys in all tiles, and in the tiles before this one
  int2 all = make_int2(0, 0), pre = make_int2(0, 0);
  constexpr int kReads = 16;
  for (int b0 = 0; b0 < ntiles; b0 += kReads) {
    int2 c[kReads];
#pragma unroll
    for (int u = 0; u < kReads; ++u)
      c[u] = reinterpret_cast<const int2*>(hist + (int64_t)min(b0 + u, ntiles - 1) * kBuckets)[t];
#pragma unroll
    for (int u = 0; u < kReads; ++u) {
      const bool in = b0 + u < ntiles, before = b0 + u < tile;
      all.x += in ? c[u].x : 0;
      all.y += in ? c[u].y : 0;
      pre.x += before ? c[u].x : 0;
      pre.y += before ? c[u].y : 0;
    }
  }
#pragma unroll
  for (int q = 0; q < kBucketWaves; ++q) *reinterpret_cast<int2*>(cnt + q * kBuckets + 2 * t) = make_int2(0, 0);
  int sum;
  const int base = block_excl_scan<kBucketBlock>(all.x + all.y, scan, &sum);  // ends with a barrier
  if (tile == 0) {
    reinterpret_cast<int2*>(starts)[t] = make_int2(base, base + all.x);
    if (t == 0) starts[kBuckets] = total;
    if (all.x > kBucketKeys || all.y > kBucketKeys) *skew = 1;
  }
  // equal buckets of a row in lane order, then rows and waves in order (as in sort_run)
  uint64_t peers[kBucketRows];
  int rank[kBucketRows];
#pragma unroll
  for (int r = 0; r < kBucketRows; ++r) {
    const uint32_t d = k[r] >> shift;
    uint64_t p = __ballot(at + r * kWave < n);
#pragma unroll
    for (int b = 0; b < kBucketBits; ++b) {
      const bool bit = (d >> b) & 1;
      const uint64_t m = __ballot(bit);
      p &= bit ? m : ~m;
    }
    peers[r] = p;
  }
#pragma unroll
  for (int r = 0; r < kBucketRows; ++r) {
    rank[r] = 0;
    if (at + r * kWave < n && (peers[r] & below) == 0)
      rank[r] = atomicAdd(&cnt[w * kBuckets + (k[r] >> shift)], __popcll(peers[r]));
  }
#pragma unroll
  for (int r = 0; r < kBucketRows; ++r) {
    const int leader = peers[r] ? __builtin_ctzll(peers[r]) : 0;
    rank[r] = __shfl(rank[r], leader, kWave) + __popcll(peers[r] & below);
  }
  __syncthreads();
  int2 o = make_int2(base + pre.x, base + all.x + pre.y);
#pragma unroll
  for (int q = 0; q < kBucketWaves; ++q) {
    int2* c = reinterpret_cast<int2*>(cnt + q * kBuckets + 2 * t);
    const int2 v = *c;
    *c = o;
    o.x += v.x;
    o.y += v.y;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kBucketRows; ++r) {
    const int i = at + r * kWave;
    if (i < n) {
      const int pos = cnt[w * kBuckets + (k[r] >> shift)] + rank[r];
      kout[pos] = k[r];
      vout[pos] = first + i;
    }
  }
}

// One workgroup per bucket: its keys by their low `shift` bits.
__global__ __launch_bounds__(kBucketSortBlock) void k_bucket_sort(const uint32_t* __restrict__ kin,
                                                                   const int* __restrict__ vin,
                                                                   const int* __restrict__ starts, int shift,
                                                                   uint32_t* kout, int* vout) {
  __shared__ RunLds<kBucketSortBlock> lds;
  const int first = starts[blockIdx.x], n = starts[blockIdx.x + 1] - first;
  if (n <= 0) return;
  if (n > kBucketKeys) {  // uniform
    for (int i = threadIdx.x; i < n; i += kBucketSortBlock) {
      kout[first + i] = (uint32_t)blockIdx.x << shift;
      vout[first + i] = vin[first + i];
    }
    return;
  }
  for (int r = 0; r < n; r += kBucketRun) {
    const int at = first + r;
    sort_run(lds, [&](int i) { return kin[at + i]; }, min(kBucketRun, n - r), [&](int i) { return vin[at + i]; },
             shift, kout + at, vout + at);
    __syncthreads();  // (also the second run's results, for the merge)
  }
  if (n <= kBucketRun) return;  // uniform
  // every key's place: its own in its run, and the keys before it in the other
  // (of equal keys the first run's come first)
  constexpr int kItems = kBucketKeys / kBucketSortBlock;
  uint32_t key[kItems];
  int val[kItems], pos[kItems];
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    const int i = q * kBucketSortBlock + (int)threadIdx.x;
    if (i >= n) continue;
    const bool second = i >= kBucketRun;
    key[q] = kout[first + i];
    val[q] = vout[first + i];
    const uint32_t* other = kout + first + (second ? 0 : kBucketRun);
    int lo = 0, hi = second ? kBucketRun : n - kBucketRun;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (other[mid] < key[q] || (second && other[mid] == key[q]))
        lo = mid + 1;
      else
        hi = mid;
    }
    pos[q] = lo + (second ? i - kBucketRun : i);
  }
  __syncthreads();  // the runs are read
#pragma unroll
  for (int q = 0; q < kItems; ++q) {
    if (q * kBucketSortBlock + (int)threadIdx.x >= n) continue;
    kout[first + pos[q]] = key[q];
    vout[first + pos[q]] = val[q];
  }
}

}  // namespace pp
