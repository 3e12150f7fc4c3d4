// Downward pass of one cell by a group of lanes: device code of the downward
// launch (expand.hip) and of the launch that finishes small solves
// (finalize.hip).
#pragma once

#include "blockscan.h"
#include "internal.h"

namespace pp {

__device__ inline double cell_side(int D, int l) { return (double)(1 << (D - l)); }
// 1 / cell_side, exact (a power of two): x * inv_cell_side equals x / cell_side.
__device__ inline double inv_cell_side(int D, int l) { return ldexp(1.0, l - D); }

// L2L is exact for a degree-p polynomial, so the
// recursion "local(child) = own M2L + L2L(local(parent))" equals the sum, over
// the cell and each of its ancestors X, of X's own M2L local shifted from X's
// centre to the cell:  L'_m = sum_X 2^{-m (l_c - l_X)} sum_{k>=m} C(k, m) d_X^{k-m} L'_k(X),
// d_X = (z_c - z_X) / s_X.  Sixteen lanes per cell with targets (four cells per
// wave): lane j takes the ancestor at level j (and j + 16), loads its p + 1 own
// coefficients once, shifts them to the cell in place by synthetic division (a
// Taylor shift by d_X: p (p + 1) / 2 complex multiply-adds) and scales
// coefficient m by 2^{-m (l_c - l_X)}; the cell itself (j = l_c) contributes its
// own local unshifted.  The lanes' terms are then added through LDS, lane m of
// the cell summing coefficient m over the levels in ascending order (a fixed
// order, so the result is reproducible).  An ancestor at a level of the dense
// prefix table is found there directly from the cell's coordinates; deeper ones
// by following parent links.
constexpr int kDownLanes = 16;

// Lane sub of the group of cell c (c < 0: none): its ancestors' terms in acc.
template <int PM>
__device__ inline void down_terms(const TreeView& t, int c, int sub, int p, const double2* __restrict__ own,
                                  const int* __restrict__ dense_off, int dense_levels, int top, cplx (&acc)[PM + 1]) {
  const int P1 = p + 1;
  const int D = t.D;
  const int lc = c >= 0 ? t.lvl[c] : -1;
  const int icx = c >= 0 ? t.ix[c] : 0, icy = c >= 0 ? t.iy[c] : 0;
  const double sc = cell_side(D, c >= 0 ? lc : 0);
  const double cx = (icx + 0.5) * sc, cy = (icy + 0.5) * sc;
#pragma unroll
  for (int k = 0; k <= PM; ++k) acc[k] = {0.0, 0.0};
  // ancestors from level top (a forest's request roots; 0 otherwise): the
  // levels above it have no interactions, and starting there gives each
  // request's cells the lane assignment (and sums) of its lone solve
  for (int a = top + sub; a <= lc; a += kDownLanes) {
    if (a == lc) {
      // every coefficient requested before the first is added (index clamped
      // to p, terms past p dropped), so no load waits behind a branch
      double2 v[PM + 1];
#pragma unroll
      for (int k = 0; k <= PM; ++k) v[k] = own[(int64_t)c * P1 + (k <= p ? k : p)];
#pragma unroll
      for (int k = 0; k <= PM; ++k)
        if (k <= p) acc[k] = cadd(acc[k], {v[k].x, v[k].y});
      continue;
    }
    const int sh = lc - a;
    const int ax = icx >> sh, ay = icy >> sh;  // the ancestor's coordinates at level a
    int X;
    if (a <= dense_levels) {
      X = dense_off[((((int64_t)1 << (2 * a)) - 1) / 3) + (int64_t)morton((uint32_t)ax, (uint32_t)ay)];
    } else {
      X = c;
      for (int l = lc; l > a; --l) X = t.parent[X];
    }
    const double sX = cell_side(D, a), iX = inv_cell_side(D, a);
    const cplx d = {(cx - (ax + 0.5) * sX) * iX, (cy - (ay + 0.5) * sX) * iX};
    cplx L[PM + 1];
#pragma unroll
    for (int k = 0; k <= PM; ++k) {
      if (k <= p) {
        const double2 v = own[(int64_t)X * P1 + k];
        L[k] = {v.x, v.y};
      } else {
        L[k] = {0.0, 0.0};
      }
    }
    // Taylor shift by d: afterwards L[m] = sum_{k>=m} C(k, m) d^{k-m} L[k]
#pragma unroll
    for (int r = 0; r < PM; ++r)
#pragma unroll
      for (int k = PM - 1; k >= r; --k)
        if (k < p) L[k] = cadd(L[k], cmul(d, L[k + 1]));
    const double f = ldexp(1.0, -sh);  // s_c / s_X
    double g = 1.0;
#pragma unroll
    for (int k = 0; k <= PM; ++k) {
      acc[k] = cadd(acc[k], cscale(L[k], g));
      g *= f;  // exact: a power of two
    }
  }
}

// Coefficient m of the group's cell: its lanes' terms red[0 .. kDownLanes) in
// order of the levels.
template <int PM>
__device__ inline cplx down_sum(const double2 (*red)[PM + 1], int m) {
  cplx s = {0.0, 0.0};
  for (int q = 0; q < kDownLanes; ++q) {
    const double2 v = red[q][m];
    s = cadd(s, {v.x, v.y});
  }
  return s;
}

}  // namespace pp
