// Wave64 / workgroup prefix-sum helpers (device only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pp {

constexpr int kWave = 64;

// Orders the LDS writes of a wave's lanes before the wave's reads that follow, and
// its reads before writes that follow.  (The hardware carries a wave's LDS
// operations out in order; this keeps the compiler from moving them.)
__device__ inline void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ inline int lane_id() { return __lane_id(); }

// v plus the value that the DPP move CTRL brings from another lane (rows of
// ROWS; 0 where the move has no source lane).
template <int CTRL, int ROWS>
__device__ inline int dpp_plus(int v) {
  return v + __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xF, false);
}

// Inclusive prefix sum across the 64 lanes of a wave, by DPP moves (plain VALU
// instructions; a cross-lane exchange through LDS per step took several times
// as long): shifts by 1, 2, 4 and 8 inside the rows of 16 lanes, then the last
// lane of row 0 into row 1 and of row 2 into row 3, then lane 31 into rows 2, 3.
// Every lane of the wave must be active.
__device__ inline int wave_incl_scan(int v) {
  v = dpp_plus<0x111, 0xF>(v);  // row_shr:1
  v = dpp_plus<0x112, 0xF>(v);  // row_shr:2
  v = dpp_plus<0x114, 0xF>(v);  // row_shr:4
  v = dpp_plus<0x118, 0xF>(v);  // row_shr:8
  v = dpp_plus<0x142, 0xA>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_plus<0x143, 0xC>(v);  // row_bcast:31 into rows 2 and 3
  return v;
}

// Sum over the 64 lanes, in every lane.
__device__ inline int wave_sum(int v) { return __builtin_amdgcn_readlane(wave_incl_scan(v), kWave - 1); }

// Exclusive prefix sum over a workgroup of BLOCK threads; returns the
// exclusive value for this thread and writes the block total to *total.
// `lds` must hold BLOCK/64 ints.  Contains __syncthreads() and ends with one
// (lds may be reused at once).
template <int BLOCK>
__device__ inline int block_excl_scan(int v, int* lds, int* total) {
  constexpr int NW = BLOCK / kWave;
  const int lane = lane_id();
  const int w = threadIdx.x / kWave;
  const int incl = wave_incl_scan(v);
  if (lane == kWave - 1) lds[w] = incl;
  __syncthreads();
  // every thread adds up the few wave totals itself (broadcast reads, one
  // barrier fewer than a serial prefix by one thread)
  int before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int t = lds[i];
    before += i < w ? t : 0;
    all += t;
  }
  *total = all;
  __syncthreads();
  return before + incl - v;
}

}  // namespace pp
