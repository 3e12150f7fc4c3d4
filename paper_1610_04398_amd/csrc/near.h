// Near field of one (target leaf, list part), by one wave: device code shared
// by the near-field launches (p2p.hip).
#pragma once

#include "blockscan.h"
#include "internal.h"

namespace pp {

// Kahan step with the group's partial sum y (which already carries -comp).
__device__ inline void kahan_fold(float y, float& sum, float& comp) {
  const float tt = sum + y;
  comp = (tt - sum) - y;
  sum = tt;
}

__device__ inline float pair_log2(float tx, float ty, float qx, float qy, bool guard) {
  const float dx = tx - qx;
  const float dy = ty - qy;
  float r2 = fmaf(dy, dy, dx * dx);
  if (guard) r2 = (r2 == 0.0f) ? 1.0f : r2;
  return __builtin_amdgcn_logf(r2);  // v_log_f32: log2
}

// Source planes (offsets x, y and weights w of the sorted sources).
struct Planes {
  const float* __restrict__ x;
  const float* __restrict__ y;
  const float* __restrict__ w;
};

// G consecutive sources from s: their terms are summed in order (the first
// product starts from -comp) and the group is folded into the running sum with
// Kahan compensation.
template <int G, bool GUARD>
__device__ inline void p2p32_group(const Planes& q, int s, float tx, float ty, float& sum, float& comp) {
  float qx[G], qy[G], qw[G], l[G];
#pragma unroll
  for (int i = 0; i < G; ++i) {
    qx[i] = q.x[s + i];
    qy[i] = q.y[s + i];
    qw[i] = q.w[s + i];
  }
#pragma unroll
  for (int i = 0; i < G; ++i) l[i] = pair_log2(tx, ty, qx[i], qy[i], GUARD);
  float y = fmaf(qw[0], l[0], -comp);
#pragma unroll
  for (int i = 1; i < G; ++i) y = fmaf(qw[i], l[i], y);
  kahan_fold(y, sum, comp);
}

// Sources [s0, s1) of one leaf against this lane's target: groups of eight
// (3 VALU of compensation per 8 pairs), then the ragged tail as at most one
// group each of four, two and one.
template <bool GUARD>
__device__ inline void p2p32_leaf(const Planes& q, int s0, int s1, float tx, float ty, float& sum, float& comp) {
  int s = s0;
  for (; s + 8 <= s1; s += 8) p2p32_group<8, GUARD>(q, s, tx, ty, sum, comp);
  if (s + 4 <= s1) {
    p2p32_group<4, GUARD>(q, s, tx, ty, sum, comp);
    s += 4;
  }
  if (s + 2 <= s1) {
    p2p32_group<2, GUARD>(q, s, tx, ty, sum, comp);
    s += 2;
  }
  if (s < s1) p2p32_group<1, GUARD>(q, s, tx, ty, sum, comp);
}

// A wave's list part [e0, e1), 64 entries at a time: lane j holds entry
// e + j's leaf, its corner relative to the target leaf's (finest cells) and
// its source range, so that the loop over the entries reads them from
// registers.  (Read per entry, the cell, its record and its range were two
// dependent round trips to L2 before the first source of every leaf.)
struct ListPart {
  int B, dx, dy, s0, s1;
  int sh;  // the leaf is 2^sh finest cells wide
};

// Entries [e, min(e + 64, e1)) of the part; returns their number.  nsrc
// gathers the lane's share of the part's source count.
__device__ inline int load_part(const P2PArgs& a, const int* lst, int e, int e1, int cax, int cay, ListPart& q,
                                int& nsrc, bool& bad) {
  const TreeView& t = a.t;
  const int n = min(kWave, e1 - e);
  const int lane = threadIdx.x % kWave;
  q = ListPart{-1, 0, 0, 0, 0, 0};
  if (lane < n) {
    const int B = lst[e + lane];
    if ((unsigned)B < (unsigned)t.ncells) {
      const int sh = t.D - t.lvl[B], ix = t.ix[B], iy = t.iy[B], s0 = t.sb[B], s1 = t.se[B];
      q = ListPart{B, cax - (ix << sh), cay - (iy << sh), s0, s1, sh};
      nsrc += s1 - s0;
    } else {
      bad = true;
    }
  }
  return n;
}

__device__ inline double wave_sum_f64(double v) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// The lane's share of the near weight sum w of sources [s0, s1): lane l adds
// sources s0 + l, s0 + l + 64, ...  Every near-field path gathers the weight
// this way (and sums the lanes by the same butterfly), so the paths' results
// are bitwise equal.
__device__ inline void near_weight(const double* __restrict__ w64, int s0, int s1, double& wn) {
  for (int s = s0 + (int)(threadIdx.x % kWave); s < s1; s += kWave) wn += w64[s];
}

// Sparse target leaves (at most kSparseTargets targets, e.g. surface points
// crossing a leaf): one lane per (target, source slot), Q source slots per
// target (Q = 4, 8 or 16 for up to 16, 8 or 4 targets), so that Q times
// more lanes do useful work than with one lane per target.  (Two slots for
// up to 32 targets were measured slower than one lane per target.)  Lane (t, q) takes the
// sources q, q + Q, q + 2Q, ... of every source leaf of its list part, sums
// their terms four at a time in FP32 and folds each group into a Kahan-
// compensated running sum; the Q slots' compensated totals are then added in
// FP64 in a fixed order (a butterfly over the Q lanes).
constexpr int kSparseTargets = 16;

// A source as the waves read it from LDS: offsets from its leaf's corner and
// weight, in FP32.
struct alignas(16) Staged {
  float x, y, w, pad;
};

// G consecutive staged sources: as p2p32_group.
template <int G, bool GUARD>
__device__ inline void staged_group(const Staged* b, float tx, float ty, float& sum, float& comp) {
  Staged q[G];
  float l[G];
#pragma unroll
  for (int i = 0; i < G; ++i) q[i] = b[i];
#pragma unroll
  for (int i = 0; i < G; ++i) l[i] = pair_log2(tx, ty, q[i].x, q[i].y, GUARD);
  float y = fmaf(q[0].w, l[0], -comp);
#pragma unroll
  for (int i = 1; i < G; ++i) y = fmaf(q[i].w, l[i], y);
  kahan_fold(y, sum, comp);
}

// cnt <= 64 staged sources of one leaf against the lane's target: Q == 1, all
// of them in groups of eight and a tail of four, two and one (as
// p2p32_leaf); Q > 1, those of the lane's slot, four at a time.
template <int Q, bool GUARD>
__device__ inline void staged_batch(const Staged* b, int cnt, int slot, float tx, float ty, float& sum, float& comp) {
  if constexpr (Q == 1) {
    int i = 0;
    for (; i + 8 <= cnt; i += 8) staged_group<8, GUARD>(b + i, tx, ty, sum, comp);
    if (i + 4 <= cnt) {
      staged_group<4, GUARD>(b + i, tx, ty, sum, comp);
      i += 4;
    }
    if (i + 2 <= cnt) {
      staged_group<2, GUARD>(b + i, tx, ty, sum, comp);
      i += 2;
    }
    if (i < cnt) staged_group<1, GUARD>(b + i, tx, ty, sum, comp);
  } else {
    for (int i0 = slot; i0 - slot < cnt; i0 += 4 * Q) {  // (uniform trip count)
      Staged q[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) q[i] = b[min(i0 + i * Q, kWave - 1)];
      if (i0 < cnt) {
        float y = -comp;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i0 + i * Q < cnt) y = fmaf(q[i].w, pair_log2(tx, ty, q[i].x, q[i].y, GUARD), y);
        kahan_fold(y, sum, comp);
      }
    }
  }
}

// The near field of (target leaf A, list part) in FP32 from sources staged in
// LDS 64 at a time (buf: the wave's 64 slots), for launches too small to hide
// latency behind other waves: one coalesced load per plane and batch, the next
// batch's in flight while this one is summed.  RAW: grid sources straight
// from their node indices and FP64 weights (the packing step's values bit for
// bit, so nothing has to be packed for it); else from the packed planes.
template <int Q, bool RAW>
__device__ inline void near32_staged(const P2PArgs& a, Staged* buf, int A, int part, int e0, int e1, const int* lst,
                                     int wid) {
  const TreeView& t = a.t;
  const int lane = threadIdx.x % kWave;
  const int tb = t.tb[A], te = t.te[A];
  const int shA = t.D - t.lvl[A];
  const int cax = t.ix[A] << shA, cay = t.iy[A] << shA;
  const int ti = lane / Q, slot = lane % Q;
  constexpr int kTargets = kWave / Q;
  int64_t pairs = 0;
  bool bad = false;
  for (int chunk = tb; chunk < te; chunk += kTargets) {
    const int k = chunk + ti;
    const bool active = k < te;
    const float2 r = a.rel32[active ? k : chunk];
    float sum = 0.0f, comp = 0.0f;
    double wn = 0.0;
    int nsrc = 0;
    for (int e = e0; e < e1; e += kWave) {
      ListPart lp;
      const int n = load_part(a, lst, e, e1, cax, cay, lp, nsrc, bad);
      // batch (j, s): entry j's sources [s, s + 64) (uniform)
      uint32_t v = 0;
      float fx = 0.0f, fy = 0.0f, fw = 0.0f;
      double w = 0.0;
      auto fetch = [&](int j, int s) {
        const int at = s + lane;
        const bool ok = at < __builtin_amdgcn_readlane(lp.s1, j);
        w = ok ? a.w64[at] : 0.0;
        if constexpr (RAW) {
          v = ok ? a.ij[at] : 0u;
        } else {
          fx = ok ? a.sx[at] : 0.0f;
          fy = ok ? a.sy[at] : 0.0f;
          fw = ok ? a.sw[at] : 0.0f;
        }
      };
      // the first batch at or after (j, s); j == n: none
      auto settle = [&](int& j, int& s) {
        while (j < n && s >= __builtin_amdgcn_readlane(lp.s1, j)) {
          ++j;
          if (j < n) s = __builtin_amdgcn_readlane(lp.s0, j);
        }
      };
      int j = 0, s = n > 0 ? __builtin_amdgcn_readlane(lp.s0, 0) : 0;
      settle(j, s);
      if (j < n) fetch(j, s);
      while (j < n) {
        const int dx = __builtin_amdgcn_readlane(lp.dx, j), dy = __builtin_amdgcn_readlane(lp.dy, j);
        const int cnt = min(kWave, __builtin_amdgcn_readlane(lp.s1, j) - s);
        const bool own = __builtin_amdgcn_readlane(lp.B, j) == A;
        Staged q;
        if constexpr (RAW) {
          q.x = (float)((int)(v & 0xFFFFu) - (cax - dx)) + 0.5f;
          q.y = (float)((int)(v >> 16) - (cay - dy)) + 0.5f;
          q.w = (float)w;
        } else {
          q.x = fx;
          q.y = fy;
          q.w = fw;
        }
        q.pad = 0.0f;
        wn += w;
        wave_lds_fence();
        buf[lane] = q;
        wave_lds_fence();
        s += kWave;
        settle(j, s);
        if (j < n) fetch(j, s);
        const float tx = r.x + (float)dx, ty = r.y + (float)dy;
        if (own)
          staged_batch<Q, true>(buf, cnt, slot, tx, ty, sum, comp);
        else
          staged_batch<Q, false>(buf, cnt, slot, tx, ty, sum, comp);
      }
    }
    double val = (double)sum - (double)comp;
    for (int o = 1; o < Q; o <<= 1) val += __shfl_xor(val, o, kWave);
    wn = wave_sum_f64(wn);
    if (active && slot == 0) a.near_sum[(int64_t)part * a.m + k] = 0.5 * (val * kLn2) + a.lnh * wn;
    pairs += (int64_t)min(kTargets, te - chunk) * wave_sum(nsrc);
  }
  if (lane == 0 && a.pair_counts) a.pair_counts[wid] = pairs;
  if (bad && a.flags) atomicOr(a.flags, kFlagBadIndex);
}

// Sparse leaf: Q from the leaf's number of targets.
template <bool RAW>
__device__ inline void near32_sparse(const P2PArgs& a, Staged* buf, int A, int part, int e0, int e1, const int* lst,
                                     int wid) {
  const int nt = a.t.te[A] - a.t.tb[A];
  if (nt <= 4)
    near32_staged<16, RAW>(a, buf, A, part, e0, e1, lst, wid);
  else if (nt <= 8)
    near32_staged<8, RAW>(a, buf, A, part, e0, e1, lst, wid);
  else
    near32_staged<4, RAW>(a, buf, A, part, e0, e1, lst, wid);
}

// Wave wid of a launch over (target leaf, list part): FP32 from staged sources.
template <bool RAW>
__device__ inline void near32_wave(const P2PArgs& a, Staged* buf, int wid) {
  const int part = wid % a.nparts;
  const int A = a.tleaves[wid / a.nparts];
  const int nb = a.list_cnt[A];
  const int* lst = a.list_src + a.list_off[A];
  const int e0 = (int)((int64_t)part * nb / a.nparts);
  const int e1 = (int)((int64_t)(part + 1) * nb / a.nparts);
  if (a.t.te[A] - a.t.tb[A] <= kSparseTargets)  // wave-uniform
    near32_sparse<RAW>(a, buf, A, part, e0, e1, lst, wid);
  else
    near32_staged<1, RAW>(a, buf, A, part, e0, e1, lst, wid);
}

// FP64 near field, one wave per (target leaf, list part) as above.
//
// Grid-node targets and grid sources sit at exact half-integer offsets, so r^2
// is a whole number there; below kLogTable it is looked up in a table of ln n
// computed on the device with the same log (bitwise the same term), any other
// r^2 calls log.  The table is kept in LDS: a gather of 64 doubles from L1
// bound the kernel (109.5M pairs of a 301 x 243 node field in 158 us, about
// 23 cycles per CU and wave-pair).  Where a whole leaf of targets lies on the
// nodes and the entry is near enough for every r^2 to be in the table (the
// usual pair of a node field), r^2 is formed in integers: 6 instructions and
// one LDS gather per wave-pair.
//
// Few targets (at most 32 in the leaf): Q source slots per target, lane
// (target, slot) taking every Q-th source, and the slots' sums added in a
// fixed order, so that the lanes are filled.
template <bool GUARD>
__device__ inline double log_term(const double* tab, double r2) {
  if (GUARD && r2 == 0.0) return 0.0;
  return r2 < (double)kLogTable && r2 == floor(r2) ? tab[(int)r2] : log(r2);
}

struct Sources64 {
  const uint32_t* __restrict__ ij;  // grid nodes: packed node indices (else null)
  const double2* __restrict__ s64;  // scattered sources: FP64 offsets from the leaf corner
  const double* __restrict__ w64;
};

// (cx, cy): the source leaf's corner, for grid nodes.
template <int STEP, bool GUARD>
__device__ inline void p2p64_leaf(const Sources64& q, const double* tab, int s0, int s1, int slot, int cx, int cy,
                                  double tx, double ty, double& sum) {
  auto term = [&](int s) {
    double ox, oy;
    if (q.ij) {
      const uint32_t v = q.ij[s];
      ox = (double)((int)(v & 0xFFFFu) - cx) + 0.5;
      oy = (double)((int)(v >> 16) - cy) + 0.5;
    } else {
      const double2 o = q.s64[s];
      ox = o.x;
      oy = o.y;
    }
    const double dx = tx - ox, dy = ty - oy;
    sum = fma(q.w64[s], log_term<GUARD>(tab, fma(dy, dy, dx * dx)), sum);
  };
  if constexpr (STEP == 1) {
#pragma unroll 2
    for (int s = s0; s < s1; ++s) term(s);
  } else {
    for (int s = s0 + slot; s < s1; s += STEP) term(s);
  }
}

// Every target on a node (itx, ity), every r^2 in the table.
template <int STEP>
__device__ inline void p2p64_lattice(const Sources64& q, const double* tab, int s0, int s1, int slot, int itx, int ity,
                                     double& sum) {
  int s = s0 + (STEP == 1 ? 0 : slot);
  for (; s + 3 * STEP < s1; s += 4 * STEP) {
    double lg[4], w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = s + i * STEP;
      const uint32_t v = q.ij[at];
      const int dx = itx - (int)(v & 0xFFFFu), dy = ity - (int)(v >> 16);
      lg[i] = tab[__mul24(dx, dx) + __mul24(dy, dy)];
      w[i] = q.w64[at];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = fma(w[i], lg[i], sum);
  }
  for (; s < s1; s += STEP) {
    const uint32_t v = q.ij[s];
    const int dx = itx - (int)(v & 0xFFFFu), dy = ity - (int)(v >> 16);
    sum = fma(q.w64[s], tab[__mul24(dx, dx) + __mul24(dy, dy)], sum);
  }
}

// Full leaves of 8 x 8 nodes against targets on the nodes: ln(r^2) by the nodes'
// offset, as in the FP32 kernel of node fields (p2p.hip), from a table filled
// from tab.  (A pitch of 56 doubles puts the 32 lanes of a half-wave's read on
// different banks.)
constexpr int kNodeSide = 8, kNodeShift = 3;
constexpr int kNodeReach64 = 23, kNodePitch64 = 56, kNodeRows64 = 2 * kNodeReach64 + 1;
__host__ __device__ constexpr int morton_x(int s) { return (s & 1) | ((s >> 1) & 2) | ((s >> 2) & 4); }
__device__ inline void node_leaf64(const double* T, const double* __restrict__ w, double& sum) {
#pragma unroll
  for (int g = 0; g < 8; ++g) {
    double l[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int s = 8 * g + i;
      l[i] = T[(kNodeSide - 1 - morton_x(s)) + kNodePitch64 * (kNodeSide - 1 - morton_x(s >> 1))];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) sum = fma(w[8 * g + i], l[i], sum);
  }
}

// nodes (NODES): the table by node offset.
template <int Q, bool NODES = false>
__device__ inline void near64(const P2PArgs& a, const Sources64& q, const double* tab, int A, int slot0, int e0, int e1,
                              const int* lst, int wid, const double* nodes = nullptr) {
  const TreeView& t = a.t;
  const int lane = threadIdx.x % kWave;
  const int tb = t.tb[A], te = t.te[A];
  const int shA = t.D - t.lvl[A];
  const int cax = t.ix[A] << shA, cay = t.iy[A] << shA;
  const int ti = lane / Q, slot = lane % Q;
  constexpr int kTargets = kWave / Q;
  int64_t pairs = 0;
  bool bad = false;
  for (int chunk = tb; chunk < te; chunk += kTargets) {
    const int k = chunk + ti;
    const bool active = k < te;
    const double2 r = a.rel64[active ? k : te - 1];
    // on a node: the offset is a whole number plus 1/2
    const double fx = r.x - 0.5, fy = r.y - 0.5;
    const bool lattice = q.ij && __ballot(fx == floor(fx) && fy == floor(fy)) == ~0ull;
    double sum = 0.0, wn = 0.0;
    int nsrc = 0;
    for (int e = e0; e < e1; e += kWave) {
      ListPart lp;
      const int n = load_part(a, lst, e, e1, cax, cay, lp, nsrc, bad);
      // the largest r^2 of an entry's pairs: both leaves' squares
      int far2 = kLogTable;
      if (lp.B >= 0) {
        const int wA = 1 << shA, wB = 1 << (t.D - t.lvl[lp.B]);
        const int mx = max(lp.dx + wA, wB - lp.dx), my = max(lp.dy + wA, wB - lp.dy);
        far2 = max(mx, my) < 2048 ? mx * mx + my * my : kLogTable;
      }
      uint64_t full = 0;  // the entries that the table by node offset serves, one bit each
      constexpr int kLast = kNodeSide - 1, low = kLast - kNodeReach64;
      if constexpr (NODES) {
        const int wA = 1 << shA, high = kNodeReach64 - wA + 1;
        const bool inside = shA <= kNodeShift && __all(fx >= 0.0 && fy >= 0.0 && fx < (double)wA && fy < (double)wA);
        full = __ballot(lattice && inside && lane < n && lp.s1 - lp.s0 == kNodeSide * kNodeSide &&
                        lp.sh == kNodeShift && lp.dx >= low && lp.dx <= high && lp.dy >= low && lp.dy <= high);
      }
      for (int j = 0; j < n; ++j) {
        const int dx = __builtin_amdgcn_readlane(lp.dx, j), dy = __builtin_amdgcn_readlane(lp.dy, j);
        const int s0 = __builtin_amdgcn_readlane(lp.s0, j), s1 = __builtin_amdgcn_readlane(lp.s1, j);
        near_weight(q.w64, s0, s1, wn);
        if (NODES && ((full >> j) & 1))
          node_leaf64(nodes + ((int)fx + dx - low) + kNodePitch64 * ((int)fy + dy - low), q.w64 + s0, sum);
        else if (lattice && __builtin_amdgcn_readlane(far2, j) < kLogTable)
          p2p64_lattice<Q>(q, tab, s0, s1, slot, cax + (int)fx, cay + (int)fy, sum);
        else if (__builtin_amdgcn_readlane(lp.B, j) == A)
          p2p64_leaf<Q, true>(q, tab, s0, s1, slot, cax - dx, cay - dy, r.x + (double)dx, r.y + (double)dy, sum);
        else
          p2p64_leaf<Q, false>(q, tab, s0, s1, slot, cax - dx, cay - dy, r.x + (double)dx, r.y + (double)dy, sum);
      }
    }
    for (int o = 1; o < Q; o <<= 1) sum += __shfl_xor(sum, o, kWave);
    wn = wave_sum_f64(wn);
    if (active && slot == 0) a.near_sum[(int64_t)slot0 * a.m + k] = 0.5 * sum + a.lnh * wn;
    pairs += (int64_t)min(kTargets, te - chunk) * wave_sum(nsrc);
  }
  if (lane == 0 && a.pair_counts) a.pair_counts[wid] = pairs + (a.more ? a.pair_counts[wid] : 0);
  if (bad && a.flags) atomicOr(a.flags, kFlagBadIndex);
}

// The workgroup's copy of the table (kLogTable doubles of LDS).
__device__ inline void load_log_table(double* tab, const double* __restrict__ log_tab) {
  for (int i = 2 * threadIdx.x; i < kLogTable; i += 2 * blockDim.x)
    *reinterpret_cast<double2*>(tab + i) = *reinterpret_cast<const double2*>(log_tab + i);
  __syncthreads();
}

// Wave wid of a launch over (target leaf, list part); list_cnt null: every
// source leaf is listed (the all-pairs sum).
template <bool NODES = false>
__device__ inline void near64_wave(const P2PArgs& a, const double* tab, int wid, const double* nodes = nullptr) {
  const Sources64 q{a.ij, a.s64, a.w64};
  const int part = a.first + wid % a.count, at = a.slot + wid % a.count;
  const TreeView& t = a.t;
  const int A = a.tleaves[wid / a.count];
  const int nb = a.list_cnt ? a.list_cnt[A] : a.nsleaves;
  const int* lst = a.list_cnt ? a.list_src + a.list_off[A] : a.sleaves;
  const int e0 = (int)((int64_t)part * nb / a.nparts);
  const int e1 = (int)((int64_t)(part + 1) * nb / a.nparts);
  const int nt = t.te[A] - t.tb[A];  // (wave-uniform)
  if (nt > 32)
    near64<1, NODES>(a, q, tab, A, at, e0, e1, lst, wid, nodes);
  else if (nt > 16)
    near64<2>(a, q, tab, A, at, e0, e1, lst, wid);
  else if (nt > 8)
    near64<4>(a, q, tab, A, at, e0, e1, lst, wid);
  else
    near64<8>(a, q, tab, A, at, e0, e1, lst, wid);
}

}  // namespace pp
