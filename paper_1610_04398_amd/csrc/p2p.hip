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

// Workgroup b's place in the order of the work when each XCD takes runs of kRun
// workgroups in turn (a bijection of [0, G), as xcd_contiguous).  Waves differ in
// length with the level of their target leaf (64 or 16 targets against like lists),
// and leaves are numbered level by level: an XCD that takes a contiguous eighth of
// them may get long ones only.  Targets off the nodes split leaves here and there:
// 512^2 with 262,144 of them 148 us in runs, 213 in eighths; 256^2 with 65,536 in
// FP64 330 and 847.  Leaves of one size (nodes) and scattered sources in FP32 keep
// the eighths, for their L2 (256^2 nodes with leaf_max 256: 189 against 196).
constexpr int kRun = 16;
__device__ inline int xcd_runs(int b, int G) {
  constexpr int span = kXcds * kRun;
  if (b >= G / span * span) return b;
  return b / span * span + (b % kXcds) * kRun + b % span / kXcds;
}
// Whether the launch is the one for where the targets lie.
__device__ inline bool unasked(const P2PArgs& a) { return a.votes && (*a.votes > 0) != (a.nodes != 0); }

// Work: wave w (workgroups spread over the XCDs in contiguous eighths, so an
// XCD's L2 holds the sources of a compact region, or in runs) handles target leaf
// tleaves[w / nparts] and the list part w % nparts (entries [part * nb / nparts,
// (part + 1) * nb / nparts)), looping over the leaf's targets 64 at a time.
// Partial sums go to
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
  if (!DIRECT && unasked(a)) return;
  const Planes q{sx, sy, sw};
  // wave-uniform work index (keeps all per-item data in scalar registers)
  const bool runs = !DIRECT && a.ij && !a.nodes;
  const int wid = __builtin_amdgcn_readfirstlane(
      (runs ? xcd_runs(blockIdx.x, gridDim.x) : xcd_contiguous(blockIdx.x, gridDim.x)) * kP2PWaves +
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

// The near field of node fields: targets on the grid's nodes against leaves of
// 8 x 8 nodes, none of them culled.  There r^2 is a whole number that depends on
// the nodes' offset only, and the sources of a leaf lie in Morton order, so that
// source s of every such leaf is the same step away from source 0: a table of
// log2(r^2) by offset in LDS (the same instruction's results, so the same terms
// bit for bit) replaces the arithmetic of a pair by one read at a compile-time
// distance from the lane's base.  The table's pitch puts an 8 x 8 block of
// targets on 64 different banks.
//
// What bounds it: LDS, 2 cycles of a compute unit per wave-pair (8 of a SIMD's);
// with r^2 and v_log_f32 a pair took 36 cycles of the SIMD.  399M pairs of a
// 512^2 node field with 2,048 other targets: 48 us alone (LDS busy for 22, the
// vector units for 30), 50 beside M2L, where k_p2p32 took 96; the whole solve 260
// -> 216 us.  Pairs of rows at a pitch of 80 collide on the banks: 66 us.
//
// It is taken where the table can serve: most targets on nodes, and 64 <= leaf_max
// < 256 (smaller leaves hold fewer than 64 sources, larger ones of a full field
// are 16 nodes wide and more).  Elsewhere its general loop, in fewer and longer
// waves, loses to k_p2p32: 301 against 205 us at 512^2 with 262,144 targets off the
// nodes, 207 against 137 with leaf_max 32, 405 against 351 with 256.
//
// Workgroups stay for several items each, since a table takes them 9 logs per
// thread to fill.  (Four waves per SIMD: 55 us; eight, with registers spilled:
// 53; a grid of more workgroups than are resident: 10 us more for the solve.)
// Leaves, list entries and targets of any other kind take the general loop.
constexpr int kNodeReach = 31;  // offsets from -31 to 31 in either direction
constexpr int kNodeRows = 2 * kNodeReach + 1;
constexpr int kNodePitch = 72;  // (8 modulo 64 banks)
constexpr int kNodeWaves = 8;
constexpr int kNodeGroups = 3 * 256, kNodeGroups64 = 2 * 256;  // workgroups resident at once

// The weights of a list entry as its waves hold them: w[q] of lane r (modulo 16)
// is source 16 q + r's, so that any of the 16 reaches every lane as an operand
// of the multiply-add (row_newbcast), and w64 of lane l source l's in FP64.
// (Weights in scalar registers: their loads count with LDS reads, and a wave
// waits for both wherever it waits for one.)
struct EntryWeights {
  float w[4];
  double w64;
};
// sw and w64: the weights of the leaf's 64 sources (uniform: with the lane's
// part as the loads' offset, a load takes no address arithmetic).
__device__ inline void load_weights(EntryWeights& ew, const float* __restrict__ sw, const double* __restrict__ w64) {
  const unsigned lane = threadIdx.x % kWave;
#pragma unroll
  for (int q = 0; q < 4; ++q) ew.w[q] = sw[lane % 16 + 16 * q];
  ew.w64 = w64[lane];
}
// y + w_R l0 + ... + w_{R+7} l7, in order, w_i the value that lane i of the lane's
// row of 16 holds in w.  (A register that a vector instruction wrote may be read
// as such an operand two wait states later.)
template <int R>
__device__ inline float add_eight(float y, float w, const float (&l)[8]) {
  static_assert(R == 0 || R == 8, "half a row");
  if constexpr (R == 0)
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf"
        : "+v"(y)
        : "v"(w), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "v"(l[4]), "v"(l[5]), "v"(l[6]), "v"(l[7]));
  else
    asm("s_nop 1\n\t"
        "v_fmac_f32_dpp %0, %1, %2 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %3 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %4 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %5 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %6 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %7 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %8 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
        "v_fmac_f32_dpp %0, %1, %9 row_newbcast:15 row_mask:0xf bank_mask:0xf"
        : "+v"(y)
        : "v"(w), "v"(l[0]), "v"(l[1]), "v"(l[2]), "v"(l[3]), "v"(l[4]), "v"(l[5]), "v"(l[6]), "v"(l[7]));
  return y;
}

// 64 sources of a full leaf against the lane's target: eight groups, each as
// p2p32_group (neg carries its -comp).  T: three rows of the table from the
// lane's base, three from the fourth, and two from the seventh (a read of two
// words reaches 1 KB).
typedef const __attribute__((address_space(3))) float* TableRow;
constexpr int kTableRows = 3;
template <int S>
__device__ inline float node_log(const TableRow (&T)[3]) {
  constexpr int row = kNodeSide - 1 - morton_x(S >> 1);
  return T[row / kTableRows][(kNodeSide - 1 - morton_x(S)) + kNodePitch * (row % kTableRows)];
}
template <int G>
__device__ inline void node_group(const TableRow (&T)[3], const EntryWeights& ew, float& sum, float& neg) {
  constexpr int S = 8 * G;
  const float l[8] = {node_log<S>(T),     node_log<S + 1>(T), node_log<S + 2>(T), node_log<S + 3>(T),
                      node_log<S + 4>(T), node_log<S + 5>(T), node_log<S + 6>(T), node_log<S + 7>(T)};
  const float y = add_eight<S % 16>(neg, ew.w[S / 16], l);
  const float tt = sum + y;
  neg = y - (tt - sum);
  sum = tt;
}
__device__ inline void node_leaf(const float* base, const EntryWeights& ew, float& sum, float& comp) {
  TableRow T[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    T[r] = (TableRow)(base + r * kTableRows * kNodePitch);
    asm("" : "+v"(T[r]));  // (kept apart: as one base, every read forms its address again)
  }
  float neg = -comp;
  node_group<0>(T, ew, sum, neg);
  node_group<1>(T, ew, sum, neg);
  node_group<2>(T, ew, sum, neg);
  node_group<3>(T, ew, sum, neg);
  node_group<4>(T, ew, sum, neg);
  node_group<5>(T, ew, sum, neg);
  node_group<6>(T, ew, sum, neg);
  node_group<7>(T, ew, sum, neg);
  comp = -neg;
}

// The items of a resident workgroup.  An XCD's workgroups (every eighth) share a
// contiguous eighth of all items, each taking every so many: close leaves in one
// L2, and slow ones (split around other targets) spread over the workgroups.  A
// workgroup's waves take its items as they get free (taken: LDS, zero).
struct ItemQueue {
  int* taken;
  int first, end, step;
  __device__ ItemQueue(int* t, int count) : taken(t) {
    const int64_t items = count;
    const int xcd = blockIdx.x % kXcds;
    step = (gridDim.x - xcd + kXcds - 1) / kXcds;
    first = (int)(xcd * items / kXcds) + (int)(blockIdx.x / kXcds);
    end = (int)((xcd + 1) * items / kXcds);
  }
  __device__ int next() {  // the wave's next item; -1: none left
    const int turn = threadIdx.x % kWave == 0 ? atomicAdd(taken, 1) : 0;
    const int64_t i = first + (int64_t)__builtin_amdgcn_readfirstlane(turn) * step;
    return i < end ? __builtin_amdgcn_readfirstlane((int)i) : -1;
  }
};

__global__ __launch_bounds__(kNodeWaves* kWave) __attribute__((amdgpu_waves_per_eu(6, 8))) void k_p2p32_nodes(
    P2PArgs a, const float* __restrict__ sx, const float* __restrict__ sy, const float* __restrict__ sw) {
  __shared__ float tab[kNodeRows * kNodePitch];
  __shared__ Staged stage[kNodeWaves][kWave];
  __shared__ int taken;
  if (unasked(a)) return;
  if (threadIdx.x == 0) taken = 0;
  for (int i = threadIdx.x; i < kNodeRows * kNodePitch; i += kNodeWaves * kWave) {
    const int dy = i / kNodePitch - kNodeReach, dx = i % kNodePitch - kNodeReach;
    const int r2 = dx * dx + dy * dy;
    tab[i] = __builtin_amdgcn_logf((float)(r2 == 0 ? 1 : r2));
  }
  __syncthreads();
  const Planes q{sx, sy, sw};
  const TreeView& t = a.t;
  const int lane = threadIdx.x % kWave;
  ItemQueue queue(&taken, a.ntleaves * a.nparts);
  for (int wid = queue.next(); wid >= 0; wid = queue.next()) {
    const int part = wid % a.nparts;
    const int A = a.tleaves[wid / a.nparts];
    const int nb = a.list_cnt[A];
    const int* lst = a.list_src + a.list_off[A];
    const int e0 = (int)((int64_t)part * nb / a.nparts);
    const int e1 = (int)((int64_t)(part + 1) * nb / a.nparts);
    const int tb = t.tb[A], te = t.te[A];
    if (te - tb <= kSparseTargets) {  // wave-uniform
      near32_sparse<false>(a, stage[threadIdx.x / kWave], A, part, e0, e1, lst, wid);
      continue;
    }
    const int shA = t.D - t.lvl[A];
    const int cax = t.ix[A] << shA, cay = t.iy[A] << shA;
    const int reach = kNodeReach - (1 << min(shA, kNodeShift)) + 1;  // of the leaf's corner
    int64_t pairs = 0;
    bool bad = false;
    for (int chunk = tb; chunk < te; chunk += kWave) {
      const int k = chunk + lane;
      const bool active = k < te;
      const float2 r = active ? a.rel32[k] : make_float2(0.5f, 0.5f);
      const float fx = r.x - 0.5f, fy = r.y - 0.5f;
      const bool nodes = shA <= kNodeShift && __all(floorf(fx) == fx && floorf(fy) == fy && fx >= 0.0f && fy >= 0.0f &&
                                                    fx < (float)(1 << shA) && fy < (float)(1 << shA));
      const int own = (int)fx + kNodePitch * (int)fy;  // (used where nodes)
      float sum = 0.0f, comp = 0.0f;
      double wn = 0.0;
      int nsrc = 0;
      for (int e = e0; e < e1; e += kWave) {
        ListPart lp;
        const int n = load_part(a, lst, e, e1, cax, cay, lp, nsrc, bad);
        // the entries that the table serves, one bit each
        constexpr int kLast = kNodeSide - 1, low = kLast - kNodeReach;
        const uint64_t full =
            __ballot(nodes && lane < n && lp.s1 - lp.s0 == kNodeSide * kNodeSide && lp.sh == kNodeShift &&
                     lp.dx >= low && lp.dx <= reach && lp.dy >= low && lp.dy <= reach);
        // the weights of entry j + 1 travel while entry j is summed
        EntryWeights next = {};
        auto fetch = [&](int j) {
          const int s0 = __builtin_amdgcn_readlane(lp.s0, j);
          if ((full >> j) & 1) load_weights(next, sw + s0, a.w64 + s0);
        };
        if (n > 0) fetch(0);
        for (int j = 0; j < n; ++j) {
          const EntryWeights ew = next;
          if (j + 1 < n) fetch(j + 1);
          const int dx = __builtin_amdgcn_readlane(lp.dx, j), dy = __builtin_amdgcn_readlane(lp.dy, j);
          if ((full >> j) & 1) {
            wn += ew.w64;
            node_leaf(tab + own + (dx - low) + kNodePitch * (dy - low), ew, sum, comp);
            continue;
          }
          const int s0 = __builtin_amdgcn_readlane(lp.s0, j), s1 = __builtin_amdgcn_readlane(lp.s1, j);
          near_weight(a.w64, s0, s1, wn);
          const float tx = r.x + (float)dx, ty = r.y + (float)dy;
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

// FP64 near field of grid sources, full leaves by the table over node offsets:
// 109.5M pairs of a 301 x 243 node field in 49 us alone, 56 with a gather of ln n
// by r^2 per pair.  Taken as in FP32 (elsewhere its general loop loses to k_p2p64:
// 486 against 394 us for a 256^2 node field with leaf_max 256).  Two workgroups
// per compute unit (112 registers a thread; three with spilled registers: 67 us).
__global__ __launch_bounds__(kNodeWaves* kWave) void k_p2p64_nodes(P2PArgs a) {
  __shared__ double tab[kLogTable];
  __shared__ double nodes[kNodeRows64 * kNodePitch64];
  __shared__ int taken;
  if (unasked(a)) return;
  if (threadIdx.x == 0) taken = 0;
  load_log_table(tab, a.log_tab);  // (ends with a barrier)
  for (int i = threadIdx.x; i < kNodeRows64 * kNodePitch64; i += kNodeWaves * kWave) {
    const int dy = i / kNodePitch64 - kNodeReach64, dx = i % kNodePitch64 - kNodeReach64;
    nodes[i] = tab[dx * dx + dy * dy];
  }
  __syncthreads();
  ItemQueue queue(&taken, a.ntleaves * a.count);
  for (int wid = queue.next(); wid >= 0; wid = queue.next()) near64_wave<true>(a, tab, wid, nodes);
}

// FP64 near field with the table of ln n by r^2 in LDS (TABLE), for targets on
// nodes and leaves of any size.
//
// Without: nearly every pair calls log, and the table (32 KB a workgroup, read
// from L1 for the few that do not) only keeps workgroups off the compute unit: a
// 512^2 solve with 200,000 targets off the nodes 1,397 us against 1,420, 65,536
// scattered sources 256 against 264.  With leaf_max below 64 the waves are too
// short to load it for (256^2 nodes, leaf_max 8: 365 against 417 us).
template <bool TABLE>
__global__ __launch_bounds__(kP2PWaves* kWave) void k_p2p64(P2PArgs a) {
  __shared__ double tab[TABLE ? kLogTable : 1];
  if (unasked(a)) return;
  if constexpr (TABLE) load_log_table(tab, a.log_tab);
  const int b = TABLE ? xcd_contiguous(blockIdx.x, gridDim.x) : xcd_runs(blockIdx.x, gridDim.x);
  const int wid = __builtin_amdgcn_readfirstlane(b * kP2PWaves + threadIdx.x / kWave);
  if (wid < a.ntleaves * a.count) near64_wave(a, TABLE ? tab : a.log_tab, wid);
}

__global__ void k_p2p_fold(double* __restrict__ near_sum, int64_t m, int n) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  double v = near_sum[k];
  for (int q = 1; q < n; ++q) v += near_sum[(int64_t)q * m + k];
  near_sum[k] = v;
}

}  // namespace

void log_table(double* tab, hipStream_t s) { k_log_table<<<(kLogTable + 255) / 256, 256, 0, s>>>(tab); }

void p2p_fold(double* near_sum, int64_t m, int n, hipStream_t s) {
  if (m > 0) k_p2p_fold<<<(unsigned)((m + 255) / 256), 256, 0, s>>>(near_sum, m, n);
}

static void launch(const P2PArgs& a, int fp64, hipStream_t s) {
  const int64_t waves = (int64_t)a.ntleaves * a.count;
  if (waves <= 0) return;
  const unsigned g = (unsigned)((waves + kP2PWaves - 1) / kP2PWaves);
  const bool direct = a.list_cnt == nullptr;
  // (one workgroup for each XCD's share of the items at least)
  const unsigned resident = (unsigned)std::min<int64_t>(
      std::max<int64_t>((waves + kNodeWaves - 1) / kNodeWaves, kXcds), fp64 ? kNodeGroups64 : kNodeGroups);
  const bool table = a.nodes && !direct && a.leaf_max >= kNodeSide * kNodeSide && a.leaf_max < 4 * kNodeSide * kNodeSide;
  if (fp64 && table) {
    k_p2p64_nodes<<<resident, kNodeWaves * kWave, 0, s>>>(a);
  } else if (fp64) {
    if (direct || (a.nodes && a.leaf_max >= kNodeSide * kNodeSide))
      k_p2p64<true><<<g, kP2PWaves * kWave, 0, s>>>(a);
    else
      k_p2p64<false><<<g, kP2PWaves * kWave, 0, s>>>(a);
  } else if (a.staged && !direct) {
    if (a.ij)
      k_near32<true><<<g, kP2PWaves * kWave, 0, s>>>(a);
    else
      k_near32<false><<<g, kP2PWaves * kWave, 0, s>>>(a);
  } else {
    if (direct)
      k_p2p32<true><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
    else if (table)
      k_p2p32_nodes<<<resident, kNodeWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
    else
      k_p2p32<false><<<g, kP2PWaves * kWave, 0, s>>>(a, a.sx, a.sy, a.sw);
  }
}

// Targets of a resident solve may have moved off the nodes, or onto them, and the
// host does not see them before the near field goes out.  Once they have, for as long
// as the tree is kept, both kinds are launched, and the one that is not asked for ends
// at once: 512^2 in FP64, moved off 1,892 us as nodes, 1,310 so, moved on 453 and 226;
// in FP32 199 and 192, 186 and 149.  Trees whose targets stay as they are do not pay
// for it (149 against 143), nor do a few waves, which last less than the other launch
// (480 at 256^2 in FP64: 116 alone, 123 with it).
constexpr int64_t kBothWaves = 2048;
void p2p(const P2PArgs& a, int fp64, hipStream_t s) {
  if (a.votes && (fp64 || !a.staged) && (int64_t)a.ntleaves * a.count > kBothWaves) {
    P2PArgs other = a;
    other.nodes = !a.nodes;
    launch(a, fp64, s);
    launch(other, fp64, s);
  } else {
    P2PArgs only = a;
    only.votes = nullptr;
    launch(only, fp64, s);
  }
}

}  // namespace pp
