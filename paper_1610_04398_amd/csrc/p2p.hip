// Near field (P2P): the direct part of the group superposition, Appendix A,
// eq. greenSum restricted to the source leaves that are not accepted for an
// expansion.  Also serves as the all-pairs direct sum when every source leaf
// is listed for every target leaf.
//
// Work item: one wave per (target leaf, part of its source list); lane j owns
// target j of each 64-target chunk.  Every lane of a wave needs the same
// source at the same time, so sources are read with wave-uniform addresses
// (scalar loads, no LDS staging) and each source costs one pass of ~7 VALU
// instructions over the 64 lanes.
//
// Coordinates are offsets in units of h: sources relative to their own leaf
// corner (exact half-integers for grid nodes), targets relative to their leaf
// corner, shifted per source leaf by the integer corner difference.  This keeps
// FP32 positions accurate to ~1e-6 h however large the grid.  The kernel sums
// w log2(r^2 / h^2); per target and list part it then stores, in FP64, half
// that sum times ln 2 plus ln(h) times the part's near weight W = sum w, which
// is the part's share of sum w ln r.
//
// Mixed precision: FP32 with Kahan-compensated accumulation in a fixed order.
// The pair of a target with a coincident node only occurs inside its own leaf;
// that leaf is processed by a guarded loop where r^2 = 0 contributes 0.
#include <algorithm>

#include "blockscan.h"
#include "internal.h"
#include "near.h"

namespace pp {

namespace {
constexpr int kP2PWaves = 4;

// Work: wave w (workgroups spread over the XCDs in contiguous runs, so an
// XCD's L2 holds the sources of a compact region) handles target leaf
// tleaves[w / nparts] and the list part
// w % nparts (entries [part * nb / nparts, (part + 1) * nb / nparts)), looping
// over the leaf's targets 64 at a time.  Partial sums go to
// near_sum[part * m + k] and are added in a fixed order by the finalize step;
// pair_counts[w] receives the number of (target, source) pairs the wave
// evaluated.
// The source planes come in as separate __restrict__ arguments: with no
// possible aliasing the compiler keeps their wave-uniform loads on the scalar
// path although the kernel stores partial sums between chunks.
template <bool DIRECT>
__global__ __launch_bounds__(kP2PWaves* kWave) __attribute__((amdgpu_waves_per_eu(7, 8))) void k_p2p32(
    P2PArgs a, const float* __restrict__ sx, const float* __restrict__ sy, const float* __restrict__ sw) {
  __shared__ Staged stage[kP2PWaves][kWave];
  const Planes q{sx, sy, sw};
  // wave-uniform work index (keeps all per-item data in scalar registers)
  const int wid = __builtin_amdgcn_readfirstlane(xcd_contiguous(blockIdx.x, gridDim.x) * kP2PWaves +
                                                    threadIdx.x / kWave);
  if (wid >= a.ntleaves * a.nparts) return;
  const int part = wid % a.nparts;
  const int lane = threadIdx.x % kWave;
  const TreeView& t = a.t;
  const int A = a.tleaves[wid / a.nparts];
  const int nb = DIRECT ? a.nsleaves : a.list_cnt[A];
  const int* lst = DIRECT ? a.sleaves : a.list_src + a.list_off[A];
  const int e0 = (int)((int64_t)part * nb / a.nparts);
  const int e1 = (int)((int64_t)(part + 1) * nb / a.nparts);
  const int tb = t.tb[A], te = t.te[A];
  if (te - tb <= kSparseTargets) {  // wave-uniform
    near32_sparse<false>(a, stage[threadIdx.x / kWave], A, part, e0, e1, lst, wid);
    return;
  }
  const int shA = t.D - t.lvl[A];
  const int cax = t.ix[A] << shA, cay = t.iy[A] << shA;
  int64_t pairs = 0;
  bool bad = false;
  for (int chunk = tb; chunk < te; chunk += kWave) {
    const int k = chunk + lane;
    const bool active = k < te;
    const float2 r = active ? a.rel32[k] : make_float2(0.0f, 0.0f);
    float sum = 0.0f, comp = 0.0f;
    double wn = 0.0;
    int nsrc = 0;
    for (int e = e0; e < e1; e += kWave) {
      ListPart lp;
      const int n = load_part(a, lst, e, e1, cax, cay, lp, nsrc, bad);
      for (int j = 0; j < n; ++j) {
        const float tx = r.x + (float)__builtin_amdgcn_readlane(lp.dx, j);
        const float ty = r.y + (float)__builtin_amdgcn_readlane(lp.dy, j);
        const int s0 = __builtin_amdgcn_readlane(lp.s0, j), s1 = __builtin_amdgcn_readlane(lp.s1, j);
        near_weight(a.w64, s0, s1, wn);
        if (__builtin_amdgcn_readlane(lp.B, j) == A)
          p2p32_leaf<true>(q, s0, s1, tx, ty, sum, comp);
        else
          p2p32_leaf<false>(q, s0, s1, tx, ty, sum, comp);
      }
    }
    wn = wave_sum_f64(wn);
    if (active) a.near_sum[(int64_t)part * a.m + k] = 0.5 * (((double)sum - (double)comp) * kLn2) + a.lnh * wn;
    pairs += (int64_t)min(kWave, te - chunk) * wave_sum(nsrc);
  }
  if (lane == 0 && a.pair_counts) a.pair_counts[wid] = pairs;
  if (bad && a.flags) atomicOr(a.flags, kFlagBadIndex);
}

// The near field from sources staged in LDS (near32_staged), for launches of
// few target leaves; work and result layout as k_p2p32.
template <bool RAW>
__global__ __launch_bounds__(kP2PWaves* kWave) void k_near32(P2PArgs a) {
  __shared__ Staged stage[kP2PWaves][kWave];
  const int wid = __builtin_amdgcn_readfirstlane(xcd_contiguous(blockIdx.x, gridDim.x) * kP2PWaves +
                                                    threadIdx.x / kWave);
  if (wid >= a.ntleaves * a.nparts) return;
  near32_wave<RAW>(a, stage[threadIdx.x / kWave], wid);
}

__global__ void k_log_table(double* __restrict__ tab) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n < kLogTable) tab[n] = n > 0 ? log((double)n) : 0.0;
}

__global__ __launch_bounds__(kP2PWaves* kWave) void k_p2p64(P2PArgs a) {
  __shared__ double tab[kLogTable];
  load_log_table(tab, a.log_tab);
  const int wid = __builtin_amdgcn_readfirstlane(xcd_contiguous(blockIdx.x, gridDim.x) * kP2PWaves +
                                                    threadIdx.x / kWave);
  if (wid < a.ntleaves * a.nparts) near64_wave(a, tab, wid);
}

}  // namespace

void log_table(double* tab, hipStream_t s) { k_log_table<<<(kLogTable + 255) / 256, 256, 0, s>>>(tab); }

void p2p(const P2PArgs& a, int fp64, hipStream_t s) {
  const int64_t waves = (int64_t)a.ntleaves * a.nparts;
  if (waves <= 0) return;
  const unsigned g = (unsigned)((waves + kP2PWaves - 1) / kP2PWaves);
  const bool direct = a.list_cnt == nullptr;
  if (fp64) {
    k_p2p64<<<g, kP2PWaves * kWave, 0, s>>>(a);
  } else if (a.staged && !direct) {
    if (a.ij)
      k_near32<true><<<g, kP2PWaves * kWave, 0, s>>>(a);
    else
      k_near32<false><<<g, kP2PWaves * kWave, 0, s>>>(a);
  } else {
    if (direct)
      k_p2p32<true><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
    else
      k_p2p32<false><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
  }
}

}  // namespace pp
