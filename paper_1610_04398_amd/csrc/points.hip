// Ingest of scattered sources (w_i = f_i h_i^2 given per source, so a source
// may carry its own cell area, eq. greenSum with a varying h) and the per-leaf
// packing of those sources and of the targets.
//
// The root square is anchored at the lower-left corner (x0, y0) of the
// bounding box of the weighted sources and the targets, and its finest cells
// have the power-of-two side u for which 2^D u first exceeds the box's extent
// (D = kPointsDepth).  Keys are floor((x - x0) / u) interleaved, the same FP64
// operations as for grid targets, so every point falls inside the root.
// Sources with w = 0 take the key 0xFFFFFFFF, above every cell key, and sort
// to the end where the tree does not see them.
#include <cfloat>
#include <cmath>

#include "blockscan.h"
#include "internal.h"
#include "leafpass.h"
#include "runsort.h"

namespace pp {

namespace {
constexpr int kBoxBlock = 256;
constexpr int kBoxItems = 8;  // points per thread, up to kBoxBlocks workgroups
constexpr int kBoxBlocks = 1024;
constexpr int kBoxReads = 4;  // requested together
constexpr int kBoxCountBits = 24;  // a workgroup's count (at most 2^31 / kBoxBlocks sources), its flags above

// Extremes of a set of points (x.. as minima: x0, -x1, y0, -y1), the number of
// weighted sources in it, and its flags.
struct Box {
  double v[4];
  int count, flags;
};
__device__ inline Box empty_box() { return {{INFINITY, INFINITY, INFINITY, INFINITY}, 0, 0}; }
__device__ inline void join(Box& a, const Box& b) {
#pragma unroll
  for (int q = 0; q < 4; ++q) a.v[q] = fmin(a.v[q], b.v[q]);
  a.count += b.count;
  a.flags |= b.flags;
}
// Thread 0: the workgroup's box.
__device__ inline void block_box(Box& b, Box* lds) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    Box r;
#pragma unroll
    for (int q = 0; q < 4; ++q) r.v[q] = __shfl_down(b.v[q], o, kWave);
    r.count = __shfl_down(b.count, o, kWave);
    r.flags = __shfl_down(b.flags, o, kWave);
    join(b, r);
  }
  if (threadIdx.x % kWave == 0) lds[threadIdx.x / kWave] = b;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < kBoxBlock / kWave; ++w) join(b, lds[w]);
}

// Per-workgroup bounding box of the weighted sources and the targets, the number
// of weighted sources, and flags for non-finite input.
__global__ __launch_bounds__(kBoxBlock) void k_box_partial(const double* __restrict__ sx,
                                                            const double* __restrict__ sy,
                                                            const double* __restrict__ w, int64_t n,
                                                            const double* __restrict__ tx,
                                                            const double* __restrict__ ty, int64_t m,
                                                            double4* __restrict__ part, int* __restrict__ cnt) {
  __shared__ Box lds[kBoxBlock / kWave];
  Box b = empty_box();
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < n + m; i0 += kBoxReads * stride) {
    double x[kBoxReads], y[kBoxReads], wi[kBoxReads];
#pragma unroll
    for (int q = 0; q < kBoxReads; ++q) {  // (no branch around the loads: past the end, the last point again)
      const int64_t i = min(i0 + q * stride, n + m - 1);
      const bool source = i < n;
      x[q] = *(source ? sx + i : tx + (i - n));
      y[q] = *(source ? sy + i : ty + (i - n));
      wi[q] = *(source ? w + i : tx + (i - n));
    }
#pragma unroll
    for (int q = 0; q < kBoxReads; ++q) {
      const int64_t i = i0 + q * stride;
      const bool source = i < n;
      if (i >= n + m) continue;
      if (!isfinite(wi[q]) || !isfinite(x[q]) || !isfinite(y[q])) {
        b.flags |= source ? kFlagNonFiniteSource : kFlagNonFiniteTarget;
      } else if (!source || wi[q] != 0.0) {
        join(b, {{x[q], -x[q], y[q], -y[q]}, source ? 1 : 0, 0});
      }
    }
  }
  block_box(b, lds);
  if (threadIdx.x == 0) {
    part[blockIdx.x] = make_double4(b.v[0], b.v[1], b.v[2], b.v[3]);
    cnt[blockIdx.x] = b.count | (b.flags << kBoxCountBits);
  }
}

// One workgroup: the whole box; every other word of the call's counters starts
// at zero here.  The root square follows from the box on the device (the key
// launches read it from `frame`: corner and finest cell side) and, by the same
// steps, on the host (points_unit).
__global__ __launch_bounds__(kBoxBlock) void k_box_final(const double4* __restrict__ part,
                                                          const int* __restrict__ cnt, int nparts, int D,
                                                          PointCounters pc) {
  __shared__ Box lds[kBoxBlock / kWave];
  const int t = threadIdx.x;
  Box b = empty_box();
  for (int i = t; i < nparts; i += kBoxBlock) {
    const double4 p = part[i];
    const int c = cnt[i];
    join(b, {{p.x, p.y, p.z, p.w}, c & ((1 << kBoxCountBits) - 1), c >> kBoxCountBits});
  }
  for (int i = t; i < pc.nwords; i += kBoxBlock) pc.words[i] = 0;
  block_box(b, lds);  // (its barrier orders the zeros before the values)
  if (t == 0) {
    const double x0 = b.v[0], x1 = -b.v[1], y0 = b.v[2], y1 = -b.v[3];
    pc.box[0] = x0;
    pc.box[1] = x1;
    pc.box[2] = y0;
    pc.box[3] = y1;
    pc.frame[0] = x0;
    pc.frame[1] = y0;
    pc.frame[2] = points_unit(fmax(x1 - x0, y1 - y0), D);
    *pc.nsrc = b.count;
    *pc.flags = b.flags;
  }
}

__device__ inline uint32_t source_key(double x, double y, double w, double x0, double y0, double u, int D) {
#pragma clang fp contract(off)
  if (w == 0.0) return 0xFFFFFFFFu;
  const double lim = (double)(1u << D);
  const double qx = floor((x - x0) / u);
  const double qy = floor((y - y0) / u);
  // inside by construction of the root; clamp defensively
  return morton((uint32_t)fmin(fmax(qx, 0.0), lim - 1.0), (uint32_t)fmin(fmax(qy, 0.0), lim - 1.0));
}

// Both sorts in two launches: runs of kLongRunKeys sources, then of targets, sorted
// in LDS; then every key finds its place among all runs, and a source's sorted
// copy is written there (runsort.h).
__global__ __launch_bounds__(kLongRunBlock) void k_point_runs(PointSort a) {
  __shared__ RunLds<kLongRunBlock> lds;
  const int sruns = (a.n + kLongRunKeys - 1) / kLongRunKeys;
  const double x0 = a.frame[0], y0 = a.frame[1], u = a.frame[2];
  if ((int)blockIdx.x < sruns) {
    const int first = blockIdx.x * kLongRunKeys;
    auto key_of = [&](int i) { return source_key(a.sx[first + i], a.sy[first + i], a.w[first + i], x0, y0, u, a.D); };
    sort_run(lds, key_of, min(kLongRunKeys, a.n - first), [&](int i) { return first + i; }, 32, a.skey_run + first, a.sval_run + first);
  } else {
    const int first = (blockIdx.x - sruns) * kLongRunKeys;
    int errs = 0;
    NodeCount nodes{0.0};  // (not used: there are no nodes)
    auto key_of = [&](int i) {
      int err = 0;
      const uint32_t key = target_key(a.tx[first + i], a.ty[first + i], x0, y0, u, a.D, &err, nodes);
      errs |= err;
      return key;
    };
    sort_run(lds, key_of, min(kLongRunKeys, a.m - first), [&](int i) { return first + i; }, 2 * a.D, a.tkey_run + first, a.tval_run + first);
    if (errs & 1) atomicOr(a.flags, kFlagNonFiniteTarget);
    if (errs & 2) atomicOr(a.flags, kFlagTargetOutside);
  }
}
__global__ __launch_bounds__(kRunBlock) void k_point_merge(PointSort a) {
  __shared__ __align__(16) uint32_t stage[kMergeStage * kLongRunKeys];
  const int sblocks = (a.n + kRunBlock - 1) / kRunBlock;
  const bool source = (int)blockIdx.x < sblocks;  // uniform
  const int i = ((int)blockIdx.x - (source ? 0 : sblocks)) * kRunBlock + threadIdx.x;
  const int n = source ? a.n : a.m;
  const uint32_t* kin = source ? a.skey_run : a.tkey_run;
  const uint32_t key = i < n ? kin[i] : 0u;
  const int val = i < n ? (source ? a.sval_run : a.tval_run)[i] : 0;
  double x = 0.0, y = 0.0, w = 0.0;
  if (source && i < n) {
    x = a.sx[val];
    y = a.sy[val];
    w = a.w[val];
  }
  const int pos = merged_position<kLongRunKeys>(kin, n, i, key, stage);
  if (i >= n) return;
  if (!source) {
    a.tkey[pos] = key;
    a.tperm[pos] = val;
    return;
  }
  a.skey[pos] = key;
  a.sval[pos] = val;
  if (pos < *a.nsrc) {
    a.xs[pos] = x;
    a.ys[pos] = y;
    a.ws[pos] = w;
  }
}

__global__ void k_point_keys(const double* __restrict__ sx, const double* __restrict__ sy,
                             const double* __restrict__ w, int64_t n, double x0, double y0, double u, int D,
                             uint32_t* __restrict__ key, int* __restrict__ idx) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  key[i] = source_key(sx[i], sy[i], w[i], x0, y0, u, D);
  idx[i] = (int)i;
}

__global__ void k_gather_points(const int* __restrict__ perm, const int* __restrict__ nsrc_dev,
                                const double* __restrict__ sx, const double* __restrict__ sy,
                                const double* __restrict__ w, double* __restrict__ xs, double* __restrict__ ys,
                                double* __restrict__ ws) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= *nsrc_dev) return;
  const int o = perm[i];
  xs[i] = sx[o];
  ys[i] = sy[o];
  ws[i] = w[o];
}

// Both per-leaf passes in one launch: the first workgroups pack the source
// leaves, the rest prepare the target leaves.
__global__ __launch_bounds__(256) void k_pack_prep_points(TreeArrays t, int D, PointFrame fr,
                                                           const int* __restrict__ sleaves, int ns,
                                                           float* __restrict__ s32, int64_t stride,
                                                           double2* __restrict__ s64,
                                                           int pack_blocks, const int* __restrict__ tleaves, int nt,
                                                           const double* __restrict__ tx,
                                                           const double* __restrict__ ty,
                                                           const int* __restrict__ perm, float2* __restrict__ rel32,
                                                           double2* __restrict__ rel64, int* __restrict__ tleaf,
                                                           double* __restrict__ self_w) {
  const int lane = threadIdx.x % kWave;
  if ((int)blockIdx.x < pack_blocks) {
    const int wid = blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (wid < ns)
      pack_point_leaf(wid, lane, t, sleaves, D, fr.xs, fr.ys, fr.ws, fr.x0, fr.y0, fr.u, s32, stride, s64);
  } else {
    const int wid = (blockIdx.x - pack_blocks) * (blockDim.x / kWave) + threadIdx.x / kWave;
    if (wid < nt)
      prep_point_leaf(wid, lane, t, tleaves, D, tx, ty, perm, fr.x0, fr.y0, fr.u, fr.xs, fr.ys, fr.ws, rel32, rel64,
                      tleaf, self_w);
  }
}
}  // namespace

int points_box_blocks(int64_t n_total) {
  const int64_t b = (n_total + kBoxBlock * kBoxItems - 1) / (kBoxBlock * kBoxItems);
  return (int)std::min<int64_t>(std::max<int64_t>(b, 1), kBoxBlocks);
}

void points_box(const double* sx, const double* sy, const double* w, int64_t n, const double* tx, const double* ty,
                int64_t m, int D, double4* part, int* cnt, const PointCounters& pc, hipStream_t s) {
  const int g = points_box_blocks(n + m);
  k_box_partial<<<g, kBoxBlock, 0, s>>>(sx, sy, w, n, tx, ty, m, part, cnt);
  k_box_final<<<1, kBoxBlock, 0, s>>>(part, cnt, g, D, pc);
}

bool points_sort_joint(int64_t n, int64_t m) {
  const int64_t most = (int64_t)kPointRuns * kLongRunKeys;
  return n <= most && m <= most;
}
void points_sort(const PointSort& a, hipStream_t s) {
  auto parts = [](int n, int per) { return (unsigned)((n + per - 1) / per); };
  const unsigned runs = parts(a.n, kLongRunKeys) + parts(a.m, kLongRunKeys);
  if (!runs) return;
  k_point_runs<<<runs, kLongRunBlock, 0, s>>>(a);
  k_point_merge<<<parts(a.n, kRunBlock) + parts(a.m, kRunBlock), kRunBlock, 0, s>>>(a);
}

void points_keys(const double* sx, const double* sy, const double* w, int64_t n, double x0, double y0, double u,
                 int D, uint32_t* key, int* idx, hipStream_t s) {
  if (n <= 0) return;
  k_point_keys<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(sx, sy, w, n, x0, y0, u, D, key, idx);
}

void points_gather(const int* perm, const int* nsrc_dev, int64_t nmax, const double* sx, const double* sy,
                   const double* w, double* xs, double* ys, double* ws, hipStream_t s) {
  if (nmax <= 0) return;
  k_gather_points<<<(unsigned)((nmax + 255) / 256), 256, 0, s>>>(perm, nsrc_dev, sx, sy, w, xs, ys, ws);
}

LeafPass leaf_pass_points(TreeArrays t, int D, double x0, double y0, double u, const double* xs, const double* ys,
                          const double* ws, const int* sleaves, int nsleaves, float* s32, int64_t stride,
                          double2* s64, const int* tleaves, int ntleaves, const double* tx,
                          const double* ty, const int* perm, float2* rel32, double2* rel64, int* tleaf,
                          double* self_w) {
  LeafPass lp;
  lp.kind = 2;
  lp.pack_blocks = std::max(nsleaves, 0) / 4 + (nsleaves % 4 > 0);
  lp.prep_blocks = std::max(ntleaves, 0) / 4 + (ntleaves % 4 > 0);
  lp.t = t;
  lp.D = D;
  lp.pa = PointArgs{PointFrame{x0, y0, u, xs, ys, ws}, sleaves, nsleaves, s32, stride, s64, tleaves, ntleaves,
                    tx, ty, perm, rel32, rel64, tleaf, self_w};
  return lp;
}

void leaf_pack_prep_points(TreeArrays t, int D, double x0, double y0, double u, const double* xs, const double* ys,
                           const double* ws, const int* sleaves, int nsleaves, float* s32, int64_t stride,
                           double2* s64, const int* tleaves, int ntleaves, const double* tx,
                           const double* ty, const int* perm, float2* rel32, double2* rel64, int* tleaf,
                           double* self_w, hipStream_t s) {
  const int gp = std::max(nsleaves, 0) / 4 + (nsleaves % 4 > 0);
  const int gt = std::max(ntleaves, 0) / 4 + (ntleaves % 4 > 0);
  if (gp + gt <= 0) return;
  const PointFrame fr{x0, y0, u, xs, ys, ws};
  k_pack_prep_points<<<gp + gt, 256, 0, s>>>(t, D, fr, sleaves, nsleaves, s32, stride, s64, gp, tleaves,
                                             ntleaves, tx, ty, perm, rel32, rel64, tleaf, self_w);
}

}  // namespace pp
