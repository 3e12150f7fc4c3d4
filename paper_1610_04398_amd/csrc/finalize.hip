// Final assembly of P at each target (Appendix A, superposition of the group
// contributions): far field from the local expansion (read, or evaluated here
// by L2P) plus the near field, with the 1/(2 pi) of eq. green2D, scattered back
// to the caller's target order.
//
// The near-field kernel leaves, per target and list part, sum w ln r over the
// part's near sources (its own leaf included).  A target that coincides with a
// grid node (exact FP64 equality with x0 + (i + 1/2) h) contributed 0 for that
// node's pair inside the near-field kernel, but w ln h through the near weight
// term: the self rule then subtracts w ln h (skip) or w kappa (cell average:
// w (ln h - kappa) in total).  In mixed precision a target within 2^-20 h of a
// node was snapped onto it (FP32 cannot resolve that distance); the exact FP64
// term w ln d is restored here.  Scattered sources that coincide exactly with a
// target were skipped by the near-field kernel the same way; their share w ln h
// is removed here (G(0) := 0).
#include <algorithm>

#include "blockscan.h"
#include "downward.h"
#include "internal.h"

namespace pp {

namespace {
constexpr int kFinBlock = 256;
constexpr int kFinWaves = kFinBlock / kWave;

__device__ inline long long wave_sum(long long v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// One item per thread of the statistics (per-wave pair counts, per-cell list
// lengths; item i of the launch), wave sums, one atomic per workgroup and
// counter, into zeroed slots: no launch of their own, and little added to the
// launch's critical path.
__device__ inline void add_totals(const FinalizeTotals& tot, int64_t i) {
  __shared__ long long part[3][kFinWaves];
  long long acc = 0, am = 0, ap = 0;
  if (tot.pairs && i < tot.nwaves) acc = tot.pair_counts[i];
  if (tot.cnt_m && i < tot.ncells) {
    am = tot.cnt_m[i];
    ap = tot.cnt_p[i];
  }
  acc = wave_sum(acc);
  am = wave_sum(am);
  ap = wave_sum(ap);
  const int w = threadIdx.x / kWave;
  if (threadIdx.x % kWave == 0) {
    part[0][w] = acc;
    part[1][w] = am;
    part[2][w] = ap;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    long long t = 0;
    for (int q = 0; q < kFinWaves; ++q) t += part[threadIdx.x][q];
    if (t) {
      if (threadIdx.x == 0 && tot.pairs) atomicAdd(tot.pairs, (unsigned long long)t);
      if (threadIdx.x == 1 && tot.cnt_m) atomicAdd(tot.tot_m, (int)t);
      if (threadIdx.x == 2 && tot.cnt_m) atomicAdd(tot.tot_p, (int)t);
    }
  }
}
__host__ __device__ inline int64_t totals_items(const FinalizeTotals& tot) {
  return std::max<int64_t>(tot.pairs ? tot.nwaves : 0, tot.cnt_m ? tot.ncells : 0);
}

// What finishes a target besides its far field, requested together: the
// near-field parts' sum (in part order), the self rule's data and its place in
// the caller's order.
struct Finish {
  double near, w, lg;
  int o;
};
struct FinishArgs {
  int64_t m;
  int nparts;
  const int* __restrict__ perm;
  const double* __restrict__ near_sum;
  const double* __restrict__ self_w;
  const double* __restrict__ self_logd;
  double lnh;
  int self_mode;
  double* __restrict__ out;
  const GridBatch* __restrict__ bt;
};
__device__ inline Finish finish_load(const FinishArgs& a, int64_t k) {
  double nsq[kMaxNearParts];
#pragma unroll
  for (int q = 0; q < kMaxNearParts; ++q) nsq[q] = q < a.nparts ? a.near_sum[(int64_t)q * a.m + k] : 0.0;
  Finish r;
  r.w = a.self_w ? a.self_w[k] : 0.0;
  r.lg = a.self_logd ? a.self_logd[k] : -INFINITY;
  r.o = a.perm[k];
  r.near = nsq[0];
#pragma unroll
  for (int q = 1; q < kMaxNearParts; ++q)
    if (q < a.nparts) r.near += nsq[q];
  return r;
}
__device__ inline void finish_store(const FinishArgs& a, const Finish& r, double far) {
  double v = far + r.near;
  if (a.self_w) {
    if (isinf(r.lg)) {
      v -= (a.self_mode == 1) ? r.w * kKappa : r.w * a.lnh;
    } else {
      v += r.w * (r.lg - a.lnh);
    }
  }
  if (a.bt) {  // a forest of requests: target o - toff[r] of request r
    const int q = batch_request(*a.bt, r.o);
    a.bt->out[q][r.o - a.bt->toff[q]] = v * kInv2Pi;
  } else {
    a.out[r.o] = v * kInv2Pi;
  }
}

__global__ __launch_bounds__(kFinBlock) void k_finalize(FinishArgs a, double* __restrict__ far,
                                                         const int* __restrict__ flags, FinalizeTotals tot,
                                                         FarEval fe) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if ((int64_t)blockIdx.x * kFinBlock < totals_items(tot)) add_totals(tot, k);  // uniform per workgroup
  if (k >= a.m) return;
  if (*flags != 0) return;
  const Finish r = finish_load(a, k);
  double fv;
  if (fe.loc) {
    const int c = fe.tleaf[k];
    fv = l2p_eval(fe.loc + (int64_t)c * (fe.p + 1), fe.p, fe.rel64[k], fe.D, fe.lvl[c], fe.fp32 != 0);
    if (far) far[k] = fv;  // kept for the far-field array read-back
  } else {
    fv = far ? far[k] : 0.0;
    if (far && fe.far_parts > 1) {
      for (int q = 1; q < fe.far_parts; ++q) fv += far[(int64_t)q * a.m + k];
      far[k] = fv;  // the total, for the far-field array read-back
    }
  }
  finish_store(a, r, fv);
}

// The way from the M2L locals to the targets in one launch, for small solves:
// workgroup b takes target leaves 4 b .. 4 b + 3.  Its first wave forms their
// locals (16 lanes each, the downward pass's terms and order) while every
// wave's loads for its own leaf's targets are in flight; then each wave
// evaluates its leaf's local at the targets and finishes them.  (Apart, the
// downward pass and the finalize step were two launches of 5-7 and 7-9 us at
// up to 1024^2, both of them latency.)  The workgroups after the leaves' add
// up the statistics.
template <int PM>
__global__ __launch_bounds__(kFinBlock) void k_far_finalize(TreeView t, const int* __restrict__ tleaves, int n, int p,
                                                            const double2* __restrict__ own,
                                                            const int* __restrict__ dense_off, int dense_levels,
                                                            int top, const double2* __restrict__ rel64, int fp32,
                                                            FinishArgs a, double* __restrict__ far,
                                                            const int* __restrict__ flags, FinalizeTotals tot) {
  __shared__ double2 red[kWave][PM + 1];
  __shared__ double2 loc[kFinWaves][PM + 1];
  static_assert(kFinWaves * kDownLanes == kWave, "one wave forms the locals of a workgroup's leaves");
  const int leaf_blocks = (n + kFinWaves - 1) / kFinWaves;
  if ((int)blockIdx.x >= leaf_blocks) {  // uniform per workgroup
    add_totals(tot, (int64_t)(blockIdx.x - leaf_blocks) * kFinBlock + threadIdx.x);
    return;
  }
  const int w = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const int i = (int)blockIdx.x * kFinWaves + w;
  const int c = i < n ? tleaves[i] : -1;
  const int lvl = c >= 0 ? t.lvl[c] : 0;
  const int tb = c >= 0 ? t.tb[c] : 0, te = c >= 0 ? t.te[c] : 0;
  const bool bad = *flags != 0;
  const int k0 = tb + lane;
  Finish r{};
  double2 rel = make_double2(0.0, 0.0);
  if (k0 < te) {
    r = finish_load(a, k0);
    rel = rel64[k0];
  }
  if (w == 0) {
    const int sub = lane % kDownLanes, grp = lane / kDownLanes;
    const int ic = (int)blockIdx.x * kFinWaves + grp;
    cplx acc[PM + 1];
    down_terms<PM>(t, ic < n ? tleaves[ic] : -1, sub, p, own, dense_off, dense_levels, top, acc);
#pragma unroll
    for (int k = 0; k <= PM; ++k) red[lane][k] = make_double2(acc[k].x, acc[k].y);
    wave_lds_fence();
    for (int m = sub; m <= p; m += kDownLanes) {
      const cplx s = down_sum<PM>(red + grp * kDownLanes, m);
      loc[grp][m] = make_double2(s.x, s.y);
    }
  }
  __syncthreads();
  if (bad) return;
  for (int k = k0; k < te; k += kWave) {
    if (k != k0) {
      r = finish_load(a, k);
      rel = rel64[k];
    }
    const double fv = l2p_eval(loc[w], p, rel, t.D, lvl, fp32 != 0);
    far[k] = fv;  // kept for the far-field array read-back
    finish_store(a, r, fv);
  }
}
}  // namespace

void finalize(int64_t m, int nparts, const int* perm, double* far, const double* near_sum,
              const double* self_w, const double* self_logd, double h, int self_mode, const int* flags, double* out,
              const FinalizeTotals& tot, const FarEval& fe, const GridBatch* bt, hipStream_t s) {
  const int64_t blocks = (std::max(m, totals_items(tot)) + kFinBlock - 1) / kFinBlock;
  if (blocks <= 0) return;
  const FinishArgs a{m, nparts, perm, near_sum, self_w, self_logd, log(h), self_mode, out, bt ? bt->dev : nullptr};
  k_finalize<<<(unsigned)blocks, kFinBlock, 0, s>>>(a, far, flags, tot, fe);
}

void far_finalize(TreeView t, const int* tleaves, int ntleaves, int64_t m, int nparts, const int* perm,
                  const double2* own, const int* dense_off, int dense_levels, int top, const double2* rel64, int p,
                  int fp32, double* far, const double* near_sum, const double* self_w, const double* self_logd,
                  double h, int self_mode, const int* flags, double* out, const FinalizeTotals& tot,
                  const GridBatch* bt, hipStream_t s) {
  const int64_t leaves = (ntleaves + kFinWaves - 1) / kFinWaves;
  const int64_t blocks = leaves + (totals_items(tot) + kFinBlock - 1) / kFinBlock;
  if (blocks <= 0) return;
  const unsigned g = (unsigned)blocks;
  const FinishArgs a{m, nparts, perm, near_sum, self_w, self_logd, log(h), self_mode, out, bt ? bt->dev : nullptr};
#define PP_FAR_FINALIZE(PM)                                                                                       \
  k_far_finalize<PM><<<g, kFinBlock, 0, s>>>(t, tleaves, ntleaves, p, own, dense_off, dense_levels, top, rel64, fp32, \
                                             a, far, flags, tot)
  if (p <= 4)
    PP_FAR_FINALIZE(4);
  else if (p <= 8)
    PP_FAR_FINALIZE(8);
  else if (p <= 12)
    PP_FAR_FINALIZE(12);
  else if (p <= 16)
    PP_FAR_FINALIZE(16);
  else
    PP_FAR_FINALIZE(20);
#undef PP_FAR_FINALIZE
}

}  // namespace pp
