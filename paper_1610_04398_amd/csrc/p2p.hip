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

namespace pp {

namespace {
constexpr int kP2PWaves = 4;

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

// A wave's list part [e0, e1), 64 entries at a time: lane j holds entry
// e + j's leaf, its corner relative to the target leaf's (finest cells) and
// its source range, so that the loop over the entries reads them from
// registers.  (Read per entry, the cell, its record and its range were two
// dependent round trips to L2 before the first source of every leaf.)
struct ListPart {
  int B, dx, dy, s0, s1;
};

// Entries [e, min(e + 64, e1)) of the part; returns their number.  wn and
// nsrc gather the lane's share of the part's near weight and source count.
__device__ inline int load_part(const P2PArgs& a, const int* lst, int e, int e1, int cax, int cay, ListPart& q,
                                double& wn, int& nsrc, bool& bad) {
  const TreeView& t = a.t;
  const int n = min(kWave, e1 - e);
  const int lane = threadIdx.x % kWave;
  q = ListPart{-1, 0, 0, 0, 0};
  if (lane < n) {
    const int B = lst[e + lane];
    if ((unsigned)B < (unsigned)t.ncells) {
      const int sh = t.D - t.lvl[B], ix = t.ix[B], iy = t.iy[B], s0 = t.sb[B], s1 = t.se[B];
      wn += a.leaf_w[B];
      q = ListPart{B, cax - (ix << sh), cay - (iy << sh), s0, s1};
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

// The sparse leaves' loop.  One step is up to four sources of one list entry
// per lane; the next step's sources are requested before this one's terms are
// formed, across the entries.  Order and rounding per lane: the entry's
// sources q, q + Q, q + 2Q, ... four at a time, each four folded once.
struct SparseStep {
  float x[4], y[4], w[4];
  float tx, ty;
  int cnt;  // of the four, how many exist for this lane
  bool guard;
};

template <int Q>
__device__ inline void p2p32_sparse(const P2PArgs& a, const Planes& q, int A, int part, int e0, int e1, const int* lst,
                                    int wid) {
  const TreeView& t = a.t;
  const int lane = threadIdx.x % kWave;
  const int tb = t.tb[A], nt = t.te[A] - tb;
  const int ti = lane / Q, qi = lane % Q;
  const bool active = ti < nt;
  const int k = tb + (active ? ti : 0);
  const int shA = t.D - t.lvl[A];
  const int cax = t.ix[A] << shA, cay = t.iy[A] << shA;
  const float2 r = a.rel32[k];
  float sum = 0.0f, comp = 0.0f;
  double wn = 0.0;
  int nsrc = 0;
  bool bad = false;
  for (int e = e0; e < e1; e += kWave) {
    ListPart lp;
    const int n = load_part(a, lst, e, e1, cax, cay, lp, wn, nsrc, bad);
    // step (j, s): entry j's sources from s on (uniform); entries without sources have none
    auto fetch = [&](int j, int s, SparseStep& st) {
      const int s1 = __builtin_amdgcn_readlane(lp.s1, j);
      st.tx = r.x + (float)__builtin_amdgcn_readlane(lp.dx, j);
      st.ty = r.y + (float)__builtin_amdgcn_readlane(lp.dy, j);
      st.guard = __builtin_amdgcn_readlane(lp.B, j) == A;
      st.cnt = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int si = s + qi + i * Q;
        st.cnt += si < s1 ? 1 : 0;
        const int at = si < s1 ? si : s;  // (s is a source of the entry)
        st.x[i] = q.x[at];
        st.y[i] = q.y[at];
        st.w[i] = q.w[at];
      }
    };
    // the first step at or after (j, s); j == n: none
    auto settle = [&](int& j, int& s) {
      while (j < n && s >= __builtin_amdgcn_readlane(lp.s1, j)) {
        ++j;
        if (j < n) s = __builtin_amdgcn_readlane(lp.s0, j);
      }
    };
    int j = 0, s = n > 0 ? __builtin_amdgcn_readlane(lp.s0, 0) : 0;
    settle(j, s);
    SparseStep cur, nxt;
    if (j < n) fetch(j, s, cur);
    while (j < n) {
      s += 4 * Q;
      settle(j, s);
      if (j < n) fetch(j, s, nxt);
      if (cur.cnt > 0) {
        float y = -comp;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (i < cur.cnt) y = fmaf(cur.w[i], pair_log2(cur.tx, cur.ty, cur.x[i], cur.y[i], cur.guard), y);
        kahan_fold(y, sum, comp);
      }
      cur = nxt;
    }
  }
  double v = (double)sum - (double)comp;
  for (int o = 1; o < Q; o <<= 1) v += __shfl_xor(v, o, kWave);
  wn = wave_sum_f64(wn);
  const int total = wave_sum(nsrc);
  if (active && qi == 0) a.near_sum[(int64_t)part * a.m + k] = 0.5 * (v * kLn2) + a.lnh * wn;
  if (lane == 0 && a.pair_counts) a.pair_counts[wid] = (int64_t)nt * total;
  if (bad && a.flags) atomicOr(a.flags, kFlagBadIndex);
}

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
__global__ __launch_bounds__(kP2PWaves* kWave) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_p2p32(
    P2PArgs a, const float* __restrict__ sx, const float* __restrict__ sy, const float* __restrict__ sw) {
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
    if (te - tb <= 4)
      p2p32_sparse<16>(a, q, A, part, e0, e1, lst, wid);
    else if (te - tb <= 8)
      p2p32_sparse<8>(a, q, A, part, e0, e1, lst, wid);
    else
      p2p32_sparse<4>(a, q, A, part, e0, e1, lst, wid);
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
      const int n = load_part(a, lst, e, e1, cax, cay, lp, wn, nsrc, bad);
      for (int j = 0; j < n; ++j) {
        const float tx = r.x + (float)__builtin_amdgcn_readlane(lp.dx, j);
        const float ty = r.y + (float)__builtin_amdgcn_readlane(lp.dy, j);
        const int s0 = __builtin_amdgcn_readlane(lp.s0, j), s1 = __builtin_amdgcn_readlane(lp.s1, j);
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
  const float* __restrict__ sx;  // grid nodes: offsets from the leaf corner (exact)
  const float* __restrict__ sy;
  const double2* __restrict__ s64;  // scattered sources: FP64 offsets (else null)
  const double* __restrict__ w64;
};

template <int STEP, bool GUARD>
__device__ inline void p2p64_leaf(const Sources64& q, const double* tab, int s0, int s1, int slot, double tx, double ty,
                                  double& sum) {
  auto term = [&](int s) {
    double ox, oy;
    if (q.s64) {
      const double2 o = q.s64[s];
      ox = o.x;
      oy = o.y;
    } else {
      ox = (double)q.sx[s];
      oy = (double)q.sy[s];
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

// Every target on a node, every r^2 in the table: whole-number arithmetic
// (tx2, ty2 and the sources' doubled offsets are odd, their differences even).
template <int STEP>
__device__ inline void p2p64_lattice(const Sources64& q, const double* tab, int s0, int s1, int slot, int itx, int ity,
                                     double& sum) {
  int s = s0 + (STEP == 1 ? 0 : slot);
  for (; s + 3 * STEP < s1; s += 4 * STEP) {
    double lg[4], w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int at = s + i * STEP;
      const int dx = itx - (int)q.sx[at], dy = ity - (int)q.sy[at];  // (the halves cancel)
      lg[i] = tab[__mul24(dx, dx) + __mul24(dy, dy)];
      w[i] = q.w64[at];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) sum = fma(w[i], lg[i], sum);
  }
  for (; s < s1; s += STEP) {
    const int dx = itx - (int)q.sx[s], dy = ity - (int)q.sy[s];
    sum = fma(q.w64[s], tab[__mul24(dx, dx) + __mul24(dy, dy)], sum);
  }
}

template <int Q, bool DIRECT>
__device__ inline void near64(const P2PArgs& a, const Sources64& q, const double* tab, int A, int part, int e0, int e1,
                              const int* lst, int wid) {
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
    const bool lattice = !q.s64 && __ballot(fx == floor(fx) && fy == floor(fy)) == ~0ull;
    double sum = 0.0, wn = 0.0;
    int nsrc = 0;
    for (int e = e0; e < e1; e += kWave) {
      ListPart lp;
      const int n = load_part(a, lst, e, e1, cax, cay, lp, wn, nsrc, bad);
      // the largest r^2 of an entry's pairs: both leaves' squares
      int far2 = kLogTable;
      if (lp.B >= 0) {
        const int wA = 1 << shA, wB = 1 << (t.D - t.lvl[lp.B]);
        const int mx = max(lp.dx + wA, wB - lp.dx), my = max(lp.dy + wA, wB - lp.dy);
        far2 = max(mx, my) < 2048 ? mx * mx + my * my : kLogTable;
      }
      for (int j = 0; j < n; ++j) {
        const int dx = __builtin_amdgcn_readlane(lp.dx, j), dy = __builtin_amdgcn_readlane(lp.dy, j);
        const int s0 = __builtin_amdgcn_readlane(lp.s0, j), s1 = __builtin_amdgcn_readlane(lp.s1, j);
        if (lattice && __builtin_amdgcn_readlane(far2, j) < kLogTable)
          p2p64_lattice<Q>(q, tab, s0, s1, slot, dx + (int)fx, dy + (int)fy, sum);
        else if (__builtin_amdgcn_readlane(lp.B, j) == A)
          p2p64_leaf<Q, true>(q, tab, s0, s1, slot, r.x + (double)dx, r.y + (double)dy, sum);
        else
          p2p64_leaf<Q, false>(q, tab, s0, s1, slot, r.x + (double)dx, r.y + (double)dy, sum);
      }
    }
    for (int o = 1; o < Q; o <<= 1) sum += __shfl_xor(sum, o, kWave);
    wn = wave_sum_f64(wn);
    if (active && slot == 0) a.near_sum[(int64_t)part * a.m + k] = 0.5 * sum + a.lnh * wn;
    pairs += (int64_t)min(kTargets, te - chunk) * wave_sum(nsrc);
  }
  if (lane == 0 && a.pair_counts) a.pair_counts[wid] = pairs;
  if (bad && a.flags) atomicOr(a.flags, kFlagBadIndex);
}

__global__ void k_log_table(double* __restrict__ tab) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n < kLogTable) tab[n] = n > 0 ? log((double)n) : 0.0;
}

template <bool DIRECT>
__global__ __launch_bounds__(kP2PWaves* kWave) void k_p2p64(P2PArgs a, const float* __restrict__ sx,
                                                             const float* __restrict__ sy,
                                                             const double2* __restrict__ s64,
                                                             const double* __restrict__ w64,
                                                             const double* __restrict__ log_tab) {
  __shared__ double tab[kLogTable];
  for (int i = 2 * threadIdx.x; i < kLogTable; i += 2 * kP2PWaves * kWave)
    *reinterpret_cast<double2*>(tab + i) = *reinterpret_cast<const double2*>(log_tab + i);
  __syncthreads();
  const Sources64 q{sx, sy, s64, w64};
  const int wid = __builtin_amdgcn_readfirstlane(xcd_contiguous(blockIdx.x, gridDim.x) * kP2PWaves +
                                                    threadIdx.x / kWave);
  if (wid >= a.ntleaves * a.nparts) return;
  const int part = wid % a.nparts;
  const TreeView& t = a.t;
  const int A = a.tleaves[wid / a.nparts];
  const int nb = DIRECT ? a.nsleaves : a.list_cnt[A];
  const int* lst = DIRECT ? a.sleaves : a.list_src + a.list_off[A];
  const int e0 = (int)((int64_t)part * nb / a.nparts);
  const int e1 = (int)((int64_t)(part + 1) * nb / a.nparts);
  const int nt = t.te[A] - t.tb[A];  // (wave-uniform)
  if (nt > 32)
    near64<1, DIRECT>(a, q, tab, A, part, e0, e1, lst, wid);
  else if (nt > 16)
    near64<2, DIRECT>(a, q, tab, A, part, e0, e1, lst, wid);
  else if (nt > 8)
    near64<4, DIRECT>(a, q, tab, A, part, e0, e1, lst, wid);
  else
    near64<8, DIRECT>(a, q, tab, A, part, e0, e1, lst, wid);
}

}  // namespace

void log_table(double* tab, hipStream_t s) { k_log_table<<<(kLogTable + 255) / 256, 256, 0, s>>>(tab); }

void p2p(const P2PArgs& a, int fp64, hipStream_t s) {
  const int64_t waves = (int64_t)a.ntleaves * a.nparts;
  if (waves <= 0) return;
  const unsigned g = (unsigned)((waves + kP2PWaves - 1) / kP2PWaves);
  const bool direct = a.list_cnt == nullptr;
  if (fp64) {
    if (direct)
      k_p2p64<true><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.s64, a.w64, a.log_tab);
    else
      k_p2p64<false><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.s64, a.w64, a.log_tab);
  } else {
    if (direct)
      k_p2p32<true><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
    else
      k_p2p32<false><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
  }
}

}  // namespace pp
