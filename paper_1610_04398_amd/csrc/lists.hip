// Interaction lists of the dual-tree traversal.
//
// The paper sums group contributions, treating a group through its expansion
// once it is far enough away and the rest directly (Appendix A, the
// superposition equation after Fig. multipole).  The traversal read here pairs
// a target cell A with a source cell B starting from the roots: accepted by
// the exact integer test -> M2L; both leaves -> P2P; A leaf -> split B; B leaf
// -> split A; otherwise split both.  Only cells with sources are used as
// sources and only cells with targets as targets.
//
// GPU form: one wave per target cell A walks the traversal restricted to A's
// ancestor path.  The pairs (X, B) with X the current path cell form a
// frontier of source cells kept in LDS; the 64 lanes classify 64 candidates at
// a time and compact what they emit with ballots, so each cell's lists come out
// in a fixed order without atomics.  Down to A the frontier advances one level
// at a time; at A itself it becomes a stack popped 64 cells at a time, so that a
// target leaf much larger than the source cells beside it (whose breadth-first
// frontier would hold every source cell of a level near it) needs only about
// 3 x 64 entries per level below A.  A count pass sizes the lists, an emit pass
// writes them.
#include <algorithm>

#include "blockscan.h"
#include "internal.h"
#include "leafpass.h"
#include "listwalk.h"

namespace pp {

namespace {
constexpr int kListWaves = 4;
template <int kFrontierCap, bool kTreecode, bool kLeafPass>
__global__ __launch_bounds__(kListWaves * kWave) void k_lists(ListArgs a, LeafPass lp) {
  __shared__ int front[kListWaves][2 * kFrontierCap];
  if constexpr (kLeafPass) {  // the per-leaf passes riding on this launch
    const int list_blocks = (a.n + kListWaves - 1) / kListWaves;
    if ((int)blockIdx.x >= list_blocks) {
      run_leaf_pass(lp, (int)blockIdx.x - list_blocks);
      return;
    }
  }
  const int w = threadIdx.x / kWave;
  const int wid = __builtin_amdgcn_readfirstlane(blockIdx.x * kListWaves + w);
  if (wid >= a.n) return;
  if constexpr (kTreecode)
    walk_leaf_treecode<kFrontierCap>(a, wid, front[w]);
  else
    walk_cell<kFrontierCap>(a, wid, front[w]);
}

template <int kFrontierCap, bool kTreecode>
void launch(const ListArgs& a, const LeafPass* lp, hipStream_t s) {
  const int extra = lp ? lp->pack_blocks + lp->prep_blocks : 0;
  const unsigned g = (unsigned)((a.n + kListWaves - 1) / kListWaves + extra);
  if (g == 0) return;
  if (lp)
    k_lists<kFrontierCap, kTreecode, true><<<g, kListWaves * kWave, 0, s>>>(a, *lp);
  else
    k_lists<kFrontierCap, kTreecode, false><<<g, kListWaves * kWave, 0, s>>>(a, LeafPass{});
}

template <bool kTreecode>
void launch_tier(const ListArgs& a, int tier_boost, const LeafPass* lp, hipStream_t s) {
  switch (std::min(2, frontier_tier_for(a.num, a.den) + tier_boost)) {
    case 0: launch<kFrontierTiers[0], kTreecode>(a, lp, s); break;
    case 1: launch<kFrontierTiers[1], kTreecode>(a, lp, s); break;
    default: launch<kFrontierTiers[2], kTreecode>(a, lp, s);
  }
}

}  // namespace

void lists_pass(TreeView t, const int4* rec, const int* tcells, int ntcells, int num, int den, int emit, int* cnt_m2l,
                int* cnt_p2p, const int* off_m2l, const int* off_p2p, int* m2l_src, int* p2p_src, int cap_m, int cap_p,
                int* flags, int tier_boost, int top, const int* dense_off, const LeafPass* lp, hipStream_t s) {
  const ListArgs a{t.D,    rec,     tcells,  std::max(ntcells, 0), num,   den,   emit,  cnt_m2l, cnt_p2p,
                   off_m2l, off_p2p, m2l_src, p2p_src,              cap_m, cap_p, flags, top,     dense_off};
  launch_tier<false>(a, tier_boost, lp, s);
}

void lists_treecode_pass(TreeView t, const int4* rec, const int* tleaves, int ntleaves, int num, int den, int emit,
                         int* cnt_m, int* cnt_p, const int* off_m, const int* off_p, int* m_src, int* p_src, int cap_m,
                         int cap_p, int* flags, int tier_boost, const LeafPass* lp, hipStream_t s) {
  const ListArgs a{t.D,   rec,   tleaves, std::max(ntleaves, 0), num,   den,   emit,  cnt_m, cnt_p,
                   off_m, off_p, m_src,   p_src,                 cap_m, cap_p, flags, 0,     nullptr};
  launch_tier<true>(a, tier_boost, lp, s);
}

bool frontier_at_top(int num, int den, int tier_boost) { return frontier_tier_for(num, den) + tier_boost >= 2; }

}  // namespace pp
