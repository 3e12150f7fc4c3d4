// Stable sort of (uint32 key, int32 index) pairs in two steps that can ride on
// other launches: runs of 1,024 keys sorted in LDS (one workgroup each), then
// one merge in which every key finds its place by counting the keys before it
// in the other runs.  The result is the stable order (ties keep their input
// order) whatever the keys' distribution.
//
// What bounds it: latency.  At the sizes it is used for (up to kMergeRuns
// runs) a radix sort over the device is a chain of 4 to 6 launches of a few
// workgroups each, 5-9 us per launch with the gap before it (32,768 keys of
// 24 bits: 38 us; 8,192 keys of 20 bits: 31 us).  Here the runs are sorted
// beside the first ingest launch and merged beside the second.
#pragma once

#include "blockscan.h"
#include "internal.h"

namespace pp {

constexpr int kRunItems = 4;       // keys per thread
constexpr int kRunDigit = 8;       // bits per pass, one counter per thread
constexpr int kRunBlock = 256;     // threads of a merge, and of a short run's sort
constexpr int kRunKeys = kRunBlock * kRunItems;  // keys per short run
constexpr int kLongRunBlock = 1024;
constexpr int kLongRunKeys = kLongRunBlock * kRunItems;

// A run is sorted by a workgroup of BLOCK threads, RUN = BLOCK kRunItems keys.
// Short runs ride on other launches; long ones keep the number of runs that a
// key is searched in small (65,536 keys in short runs: 14 us to sort, 53 to
// merge; in long ones 25 and 21).
template <int BLOCK>
struct RunLds {
  uint32_t key[BLOCK * kRunItems];
  uint16_t val[BLOCK * kRunItems];
  int cnt[BLOCK / kWave][1 << kRunDigit];
  int scan[BLOCK / kWave + 1];
};

// One workgroup sorts the n <= RUN keys that `key_of(i)` gives for i in
// [0, n) by their low `bits` bits and stores the sorted keys at kout[0, n) and
// val_of(i) at vout[0, n).  LSD passes of up to 8 bits inside LDS; a wave owns
// kRunItems consecutive rows of 64 keys, ranks equal digits of a row with one
// ballot per digit bit, and counts rows in its own column of cnt.
template <int BLOCK, class KeyOf, class ValOf>
__device__ inline void sort_run(RunLds<BLOCK>& s, KeyOf key_of, int n, ValOf val_of, int bits,
                                uint32_t* __restrict__ kout, int* __restrict__ vout) {
  constexpr int kRunWaves = BLOCK / kWave, kDigits = 1 << kRunDigit;
  static_assert(BLOCK >= kDigits, "one counter per thread");
  const int t = threadIdx.x, lane = t % kWave, w = t / kWave;
  const uint64_t below = lane == 0 ? 0ull : (~0ull) >> (kWave - lane);
  const int at = w * (kRunItems * kWave) + lane;  // the lane's key of row 0
  uint32_t k[kRunItems];
  int v[kRunItems], rank[kRunItems];
#pragma unroll
  for (int r = 0; r < kRunItems; ++r) {
    const int i = at + r * kWave;
    k[r] = i < n ? key_of(i) : 0u;
    v[r] = i;
  }
  const int passes = (bits + kRunDigit - 1) / kRunDigit;
  const int width = passes ? (bits + passes - 1) / passes : 0;
  const uint32_t mask = (1u << width) - 1;
  for (int ps = 0; ps < passes; ++ps) {
    const int shift = ps * width;
    for (int q = t; q < kRunWaves * kDigits; q += BLOCK) s.cnt[q / kDigits][q % kDigits] = 0;
    __syncthreads();
    // each row's lanes with equal digits, in lane order (the rows are
    // independent, so their ballots interleave)
    uint64_t peers[kRunItems];
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {
      const int d = (int)((k[r] >> shift) & mask);
      uint64_t p = __ballot(at + r * kWave < n);
#pragma unroll
      for (int b = 0; b < kRunDigit; ++b) {
        if (b < width) {
          const bool bit = (d >> b) & 1;
          const uint64_t m = __ballot(bit);
          p &= bit ? m : ~m;
        }
      }
      peers[r] = p;
    }
    // the first lane of each digit adds the row's count; a wave's LDS
    // operations are carried out in order, so a row sees the rows before it
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {
      rank[r] = 0;
      if (at + r * kWave < n && (peers[r] & below) == 0)
        rank[r] = atomicAdd(&s.cnt[w][(k[r] >> shift) & mask], __popcll(peers[r]));
    }
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {
      const int leader = peers[r] ? __builtin_ctzll(peers[r]) : 0;
      rank[r] = __shfl(rank[r], leader, kWave) + __popcll(peers[r] & below);
    }
    __syncthreads();
    // thread t owns digit t: offsets of its keys in each wave
    int c[kRunWaves], sum = 0;
#pragma unroll
    for (int q = 0; q < kRunWaves; ++q) {
      c[q] = t < kDigits ? s.cnt[q][t] : 0;
      sum += c[q];
    }
    int total;
    int o = block_excl_scan<BLOCK>(sum, s.scan, &total);  // ends with a barrier
#pragma unroll
    for (int q = 0; q < kRunWaves; ++q) {
      if (t < kDigits) s.cnt[q][t] = o;
      o += c[q];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {
      if (at + r * kWave < n) {
        const int pos = s.cnt[w][(k[r] >> shift) & mask] + rank[r];
        s.key[pos] = k[r];
        s.val[pos] = (uint16_t)v[r];
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRunItems; ++r) {
      const int i = at + r * kWave;
      if (i < n) {
        k[r] = s.key[i];
        v[r] = s.val[i];
      }
    }
    // (the next pass writes key and val only after its own barriers)
  }
#pragma unroll
  for (int r = 0; r < kRunItems; ++r) {
    const int i = at + r * kWave;
    if (i < n) {
      kout[i] = k[r];
      vout[i] = val_of(v[r]);
    }
  }
}

// Sorted position of key i of the n keys kin (runs of RUN, each sorted;
// 16-byte aligned): its place in its own run, plus the keys <= it in the runs
// before and the keys < it in the runs after.  The whole workgroup calls it
// (threads with i >= n too): kMergeStage runs at a time are staged in `stage`
// (kMergeStage RUN keys of LDS), the next ones' loads in flight, and
// the binary searches of a stage's runs advance together.  (Searched in global
// memory, each of the 11 steps waited on an L2 round trip: 11-14 us for up to
// 8,192 keys.)
constexpr int kMergeStage = 4;
template <int RUN>
__device__ inline int merged_position(const uint32_t* __restrict__ kin, int n, int i, uint32_t key, uint32_t* stage) {
  constexpr int kReads = kMergeStage * RUN / (4 * kRunBlock);  // 16-byte loads per thread and stage
  const int t = threadIdx.x;
  const int own = i / RUN;
  const int nr = (n + RUN - 1) / RUN;
  uint4 nxt[kReads];
  auto fetch = [&](int r0) {
#pragma unroll
    for (int q = 0; q < kReads; ++q) {
      const int j = r0 * RUN + 4 * (t + q * kRunBlock);
      nxt[q] = make_uint4(0u, 0u, 0u, 0u);
      if (j + 4 <= n) {
        nxt[q] = *reinterpret_cast<const uint4*>(kin + j);
      } else {
        if (j < n) nxt[q].x = kin[j];
        if (j + 1 < n) nxt[q].y = kin[j + 1];
        if (j + 2 < n) nxt[q].z = kin[j + 2];
      }
    }
  };
  int pos = i - own * RUN;
  fetch(0);
  for (int r0 = 0; r0 < nr; r0 += kMergeStage) {
    __syncthreads();  // the last stage's searches are done
#pragma unroll
    for (int q = 0; q < kReads; ++q) *reinterpret_cast<uint4*>(stage + 4 * (t + q * kRunBlock)) = nxt[q];
    __syncthreads();
    if (r0 + kMergeStage < nr) fetch(r0 + kMergeStage);
    int lo[kMergeStage], len[kMergeStage];
#pragma unroll
    for (int u = 0; u < kMergeStage; ++u) {
      const int r = r0 + u;
      lo[u] = 0;
      len[u] = (r < nr && r != own) ? min(RUN, n - r * RUN) : 0;
    }
#pragma unroll 1
    for (int half = RUN; half > 0; half >>= 1) {
      uint32_t kv[kMergeStage];
#pragma unroll
      for (int u = 0; u < kMergeStage; ++u)  // (an index past the run's end is clamped: its key is not used)
        kv[u] = stage[u * RUN + min(lo[u] + half, RUN) - 1];
#pragma unroll
      for (int u = 0; u < kMergeStage; ++u)
        if (lo[u] + half <= len[u] && (kv[u] < key || (kv[u] == key && r0 + u < own))) lo[u] += half;
    }
#pragma unroll
    for (int u = 0; u < kMergeStage; ++u) pos += lo[u];
  }
  return pos;
}

}  // namespace pp
