// Forces summed per body (segment of consecutive panels): device code of the
// pressure forces (forces.hip) and the viscous forces (assembly.hip).
//
// One workgroup per slice of a segment: thread i of slice q takes the panels i
// + kSumBlock (q + slices j), j = 0, 1, ..., in order with a compensated FP64
// sum; the compensated sums are combined by fixed trees (wave, workgroup,
// slices), so the result does not depend on the hardware's scheduling.  The
// slices' sums meet in device memory, and the workgroup of a segment that
// arrives last adds them up.
//
// What bounds it: the latency of a thread's loads, panel after panel.  4,096
// panels take 6 us (pressure) and 8 us (viscous) in 16 slices; one workgroup for
// the whole segment took 13 and 39 us.
#pragma once

#include "blockscan.h"
#include "internal.h"

namespace pp {

struct Comp {  // Neumaier-compensated sum
  double s, c;
  __device__ void add(double x) {
#pragma clang fp contract(off)
    const double t = s + x;
    c += fabs(s) >= fabs(x) ? (s - t) + x : (x - t) + s;
    s = t;
  }
  // (a sum that overflows here stays infinite, as plain sums do)
  __device__ void merge(const Comp& o) {
    if (isfinite(s + o.s)) add(o.s);
    else s += o.s;
    c += o.c;
  }
  __device__ Comp down(int o) const {
    Comp r = {};
    r.s = __shfl_down(s, o, kWave);
    r.c = __shfl_down(c, o, kWave);
    return r;
  }
};

struct ForcePair {
  Comp x, y;
  __device__ void merge(const ForcePair& o) {
    x.merge(o.x);
    y.merge(o.y);
  }
  // lane 0: the wave's sum
  __device__ void wave_sum() {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      ForcePair r = {};
      r.x = x.down(o);
      r.y = y.down(o);
      merge(r);
    }
  }
};
static_assert(sizeof(ForcePair) == kSlicePairBytes, "the slices' sums in device memory");

// panel(j, fx, fy): the force on panel j, stored too where the caller wants it.
template <class Panel>
__device__ inline void sum_segment(const ForceSegments& segs, double ux, double uy, double rho, double area,
                                   pp_force* __restrict__ out, Panel panel) {
  constexpr int kWaves = kSumBlock / kWave;
  __shared__ ForcePair part[kWaves];
  __shared__ int last;
  const int seg = blockIdx.x / segs.slices, slice = blockIdx.x % segs.slices;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int64_t a = segs.dev ? segs.dev[seg] : segs.start[seg];
  const int64_t b = segs.dev ? segs.dev[seg + 1] : segs.start[seg + 1];
  ForcePair sum = {};
  for (int64_t j = a + (int64_t)slice * kSumBlock + tid; j < b; j += (int64_t)segs.slices * kSumBlock) {
    double fx, fy;
    panel(j, fx, fy);
    sum.x.add(fx);
    sum.y.add(fy);
  }
  sum.wave_sum();
  if (lane == 0) part[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kWaves; ++w) sum.merge(part[w]);
    last = 1;
    if (segs.slices > 1) {
      static_cast<ForcePair*>(segs.part)[blockIdx.x] = sum;
      // release this slice's sum, acquire the others' (the ticket is back at
      // zero for the next launch)
      last = __hip_atomic_fetch_add(segs.ticket + seg, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
             segs.slices - 1;
      if (last) __hip_atomic_store(segs.ticket + seg, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  __syncthreads();
  if (!last || wave != 0) return;
  if (segs.slices > 1) {
    sum = lane < segs.slices ? static_cast<const ForcePair*>(segs.part)[seg * segs.slices + lane] : ForcePair{};
    sum.wave_sum();
  }
  if (lane == 0) {
    const double fx = sum.x.s + sum.x.c, fy = sum.y.s + sum.y.c;
    const double speed = sqrt(ux * ux + uy * uy);
    const double drag = (fx * ux + fy * uy) / speed;
    pp_force f;
    f.fx = fx;
    f.fy = fy;
    f.drag = drag;
    f.cd = 2.0 * drag / (rho * speed * speed * area);
    out[seg] = f;
  }
}

}  // namespace pp
