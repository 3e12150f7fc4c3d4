// Interaction-list traversal of one target cell by one wave: device code of the
// list launches (see lists.hip).
#pragma once

#include <climits>

#include "blockscan.h"
#include "internal.h"

namespace pp {

// Frontier capacity per wave (two level buffers, or one stack of twice the
// size at the target cell), in three tiers.  The frontier of a target cell holds
// the non-accepted source cells near its path, ~4 (2/theta + 1)^2 in a uniform
// tree (about 100 at theta = 0.5).  Tier 0 (256 entries, 8 KB of LDS per
// workgroup, so LDS no longer limits the waves per CU) serves theta >= 0.5;
// tier 1 (1024) theta >= 0.3; tier 2 (2048) smaller theta.  Overflow is flagged
// and the solve repeats at the next tier.
constexpr int kFrontierTiers[3] = {256, 1024, 2048};
inline int frontier_tier_for(int num, int den) {
  if (2 * num >= den) return 0;       // theta >= 0.5
  if (num * 10 >= 3 * den) return 1;  // theta >= 0.3
  return 2;
}

// Packed per-cell record for the traversal: {ix, iy, first child, meta} with
// meta = level | nchild << 5 | (children-with-sources mask) << 8 | has_src << 12.
__device__ inline int rec_level(int4 r) { return r.w & 31; }
__device__ inline int rec_nchild(int4 r) { return (r.w >> 5) & 7; }
__device__ inline int rec_kidmask(int4 r) { return (r.w >> 8) & 15; }
__device__ inline bool rec_has_src(int4 r) { return (r.w >> 12) & 1; }

// The traversal at the target cell A itself, from the source cells left on the
// stack st[0, top): accepted -> A's far list (M2L, or M2P for the tree-code);
// not accepted and a leaf -> A's near list when A is a leaf; not accepted and
// not a leaf -> its children with sources pushed when A is a leaf (for a
// non-leaf A the rest belongs to A's children).  Pops the top 64 entries at a
// time.  Returns true when the stack would exceed `cap` (the lists are then
// incomplete).
template <bool kTreecode>
__device__ bool lists_at_target(int* st, int top, int cap, int D, int4 rA, bool leafA, int num, int den,
                                const int4* __restrict__ rec, int emit, int* __restrict__ m_src, int64_t mbase,
                                int mlim, int* __restrict__ p_src, int64_t pbase, int plim, int& nm, int& np,
                                int lane, uint64_t lt_mask) {
  const int lA = rec_level(rA);
  while (top > 0) {
    const int n = min(kWave, top);
    const bool valid = lane < n;
    const int B = valid ? st[top - n + lane] : 0;
    top -= n;
    __syncwarp();  // the popped slots take this round's pushes
    bool acc = false, leafB = false;
    int kid0 = 0, kmask = 0;
    if (valid) {
      const int4 rB = rec[B];
      acc = kTreecode ? treecode_accept(D, lA, rA.x, rA.y, rec_level(rB), rB.x, rB.y, num, den)
                      : mac_accept(D, lA, rA.x, rA.y, rec_level(rB), rB.x, rB.y, num, den);
      kid0 = rB.z;
      leafB = kid0 < 0;
      kmask = rec_kidmask(rB);
    }
    const bool em = valid && acc;
    const bool ep = valid && !acc && leafB && leafA;
    const bool push = valid && !acc && !leafB && leafA;
    const uint64_t bm = __ballot(em);
    const uint64_t bp = __ballot(ep);
    if (emit) {
      const int im = nm + __popcll(bm & lt_mask), ip = np + __popcll(bp & lt_mask);
      if (em && im < mlim) m_src[mbase + im] = B;
      if (ep && ip < plim) p_src[pbase + ip] = B;
    }
    nm += __popcll(bm);
    np += __popcll(bp);
    const int npush = push ? __popc(kmask) : 0;
    const int incl = wave_incl_scan(npush);
    const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
    if (top + total > cap) return true;
    if (push) {
      int pos = top + incl - npush;
      for (int q = 0; q < 4; ++q)
        if ((kmask >> q) & 1) st[pos++] = kid0 + q;
    }
    top += total;
    __syncwarp();
  }
  return false;
}

// Where the lists of a launch go and what they are built from (lists_pass,
// lists_treecode_pass in internal.h).  cells: the target cells, or (tree-code)
// target leaves.  dense_off: cell numbers of the tree build's prefix table,
// needed when top > 0 (the request roots of a forest lie in it).
struct ListArgs {
  int D;
  const int4* rec;
  const int* cells;
  int n;
  int num, den, emit;
  int* cnt_m;
  int* cnt_p;
  const int* off_m;
  const int* off_p;
  int* m_src;
  int* p_src;
  int cap_m, cap_p;
  int* flags;
  int top;
  const int* dense_off;
};

// Lists of target cell cells[wid] of the dual traversal; buf: 2 kFrontierCap
// ints of LDS of the wave.
template <int kFrontierCap>
__device__ inline void walk_cell(const ListArgs& a, int wid, int* buf) {
  const int lane = threadIdx.x % kWave;
  const int D = a.D;
  const int A = a.cells[wid];
  const int4 rA = a.rec[A];
  const int lA = rec_level(rA);
  const bool leafA = rA.z < 0;
  const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (kWave - lane));
  int* cur = buf;
  int* nxt = buf + kFrontierCap;
  int ncur = 0;
  // top > 0 (a forest of requests): the walk starts at A's ancestor of level
  // top, its request's root, and cells above that level have no lists
  const int top = a.top;
  int R0 = top > 0 ? -1 : 0;
  if (top > 0 && lA >= top)
    R0 = a.dense_off[((((int64_t)1 << (2 * top)) - 1) / 3) +
                     (int64_t)morton((uint32_t)rA.x >> (lA - top), (uint32_t)rA.y >> (lA - top))];
  if (R0 >= 0 && rec_has_src(a.rec[R0])) {
    if (lane == 0) cur[0] = R0;
    ncur = 1;
  }
  __syncwarp();
  // emit 1: exact offsets from a count pass; emit 2: fixed capacity per cell
  const int64_t mbase = a.emit == 1 ? a.off_m[A] : (int64_t)A * a.cap_m;
  const int64_t pbase = a.emit == 1 ? a.off_p[A] : (int64_t)A * a.cap_p;
  const int mlim = a.emit == 2 ? a.cap_m : INT_MAX;
  const int plim = a.emit == 2 ? a.cap_p : INT_MAX;
  bool overflow = false;
  // Down the path: X (level xl) is a proper ancestor of A, so not a leaf, and a
  // pair accepted here belongs to X's lists.  A source leaf that is not
  // accepted stays for the next level, any other source cell is replaced by its
  // children with sources.  (X's place follows from A's: nothing is read for
  // it.  Following the parent links first took a dependent load per level.)
  for (int xl = top; xl < lA && ncur > 0; ++xl) {
    const int xx = rA.x >> (lA - xl), xy = rA.y >> (lA - xl);
    int nnext = 0;
    for (int base = 0; base < ncur; base += kWave) {
      const int i = base + lane;
      const bool valid = i < ncur;
      const int B = valid ? cur[i] : 0;
      bool keep = false, leafB = false;
      int kid0 = 0, kmask = 0;
      if (valid) {
        const int4 rB = a.rec[B];
        keep = !mac_accept(D, xl, xx, xy, rec_level(rB), rB.x, rB.y, a.num, a.den);
        kid0 = rB.z;
        leafB = kid0 < 0;
        kmask = rec_kidmask(rB);
      }
      const int npush = keep ? (leafB ? 1 : __popc(kmask)) : 0;
      const int incl = wave_incl_scan(npush);
      const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
      int pos = nnext + incl - npush;
      if (nnext + total > kFrontierCap) {
        overflow = true;
      } else {
        if (keep && leafB) nxt[pos] = B;
        if (keep && !leafB) {
          for (int q = 0; q < 4; ++q)
            if ((kmask >> q) & 1) nxt[pos++] = kid0 + q;
        }
        nnext += total;
      }
    }
    __syncwarp();
    if (overflow) break;
    int* tmp = cur;
    cur = nxt;
    nxt = tmp;
    ncur = nnext;
  }
  int nm = 0, np = 0;
  if (!overflow && ncur > 0) {
    if (cur != buf) {  // the stack starts at the bottom of the buffer (no overlap: ncur <= kFrontierCap)
      for (int i = lane; i < ncur; i += kWave) buf[i] = cur[i];
      __syncwarp();
    }
    overflow = lists_at_target<false>(buf, ncur, 2 * kFrontierCap, D, rA, leafA, a.num, a.den, a.rec, a.emit, a.m_src,
                                      mbase, mlim, a.p_src, pbase, plim, nm, np, lane, lt_mask);
  }
  if (overflow && lane == 0) atomicOr(a.flags, kFlagFrontierOverflow);
  if (a.emit == 2 && (nm > a.cap_m || np > a.cap_p) && lane == 0) atomicOr(a.flags, kFlagListOverflow);
  if (a.emit != 1 && lane == 0) {
    // in the capacity layout a list never reaches past its cell's slots: an
    // overflowing list is cut at the capacity (and flagged for an exact re-run),
    // so the kernels that read it stay inside the allocation
    a.cnt_m[A] = a.emit == 2 ? min(nm, a.cap_m) : nm;
    a.cnt_p[A] = a.emit == 2 ? min(np, a.cap_p) : np;
  }
}

// Lists of target leaf cells[wid] in the paper's tree-code: the wave walks the
// source tree from the root.  A source cell accepted for all of A's targets
// goes to A's M2P list; a leaf that is not accepted goes to its P2P list; any
// other cell is replaced by its children with sources.  The cells still to
// visit form a stack in LDS, popped and classified 64 at a time; ballots
// compact the output in a fixed order.  Same emit modes and layouts as above.
template <int kFrontierCap>
__device__ inline void walk_leaf_treecode(const ListArgs& a, int wid, int* buf) {
  const int lane = threadIdx.x % kWave;
  const int A = a.cells[wid];
  const int4 rA = a.rec[A];
  const uint64_t lt_mask = (lane == 0) ? 0ull : ((~0ull) >> (kWave - lane));
  int top = 0;
  if (rec_has_src(a.rec[0])) {
    if (lane == 0) buf[0] = 0;
    top = 1;
  }
  __syncwarp();
  int nm = 0, np = 0;
  const int64_t mbase = a.emit == 1 ? a.off_m[A] : (int64_t)A * a.cap_m;
  const int64_t pbase = a.emit == 1 ? a.off_p[A] : (int64_t)A * a.cap_p;
  const int mlim = a.emit == 2 ? a.cap_m : INT_MAX;
  const int plim = a.emit == 2 ? a.cap_p : INT_MAX;
  const bool overflow = lists_at_target<true>(buf, top, 2 * kFrontierCap, a.D, rA, true, a.num, a.den, a.rec, a.emit,
                                              a.m_src, mbase, mlim, a.p_src, pbase, plim, nm, np, lane, lt_mask);
  if (overflow && lane == 0) atomicOr(a.flags, kFlagFrontierOverflow);
  if (a.emit == 2 && (nm > a.cap_m || np > a.cap_p) && lane == 0) atomicOr(a.flags, kFlagListOverflow);
  if (a.emit != 1 && lane == 0) {
    a.cnt_m[A] = a.emit == 2 ? min(nm, a.cap_m) : nm;
    a.cnt_p[A] = a.emit == 2 ? min(np, a.cap_p) : np;
  }
}

}  // namespace pp
