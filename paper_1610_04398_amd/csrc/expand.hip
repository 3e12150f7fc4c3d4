// Expansion passes in FP64: P2M by leaves, M2L, L2L, L2P, M2P (P2M by blocks of
// grid nodes and M2M: upward.hip).
//
// Notation: the sources of a cell with centre z_c and side s have the
// multipole expansion  Phi(z) = a_0 log(z - z_c) + sum_{k=1..p} a_k (z - z_c)^-k
// with a_0 = S = sum w and a_k = -alpha_k = -sum w (z_i - z_c)^k / k
// (Appendix A, eq. alphaK and eq. pressTruncated; P = Re Phi / 2pi).  Stored
// coefficients are scaled by the cell side, a'_k = a_k / s^k, and locals
// L'_l = L_l s^l, so every operator acts on O(1) numbers and depends only on
// offsets measured in cell sides.  Positions are in units of the finest cell
// (h), where every cell centre is exact in FP64.
//
// M2M is the re-centring of eq. expandedShift with the S term's sign derived
// from eq. logExpansion (+S z0^k / k in the paper's alpha convention; the
// printed minus sign does not reproduce the parent's expansion).  M2L, L2L and
// L2P are the local-expansion operators of the fast multipole method that the
// paper cites, derived from the same series:
//   M2L (z0 = z_B - z_A, t = s_A / z0, r = s_B / z0):
//     L'_0 = a_0 ln|z0| + sum_k a'_k (-r)^k
//     L'_l = t^l [ -a_0 / l + sum_k C(l+k-1, k-1) a'_k (-r)^k ],  l >= 1
//   L2L (d = (z_child - z_parent) / s_parent):
//     L'_m(child) = 2^-m sum_{k>=m} C(k, m) d^(k-m) L'_k(parent)
//   M2M (d as above):
//     a'_l(parent) += -a_0 d^l / l + sum_{k=1..l} C(l-1, k-1) 2^-k d^(l-k) a'_k(child)
//   L2P: far(z) = Re sum_l L'_l u^l,  u = (z - z_c) / s.
#include <algorithm>
#include <cstdlib>
#include <mutex>

#include "blockscan.h"
#include "downward.h"
#include "internal.h"

namespace pp {

namespace {

struct BinomTable {
  double v[2 * kMaxP + 1][2 * kMaxP + 1];
};
constexpr BinomTable make_binom() {
  BinomTable b{};
  for (int n = 0; n <= 2 * kMaxP; ++n) {
    b.v[n][0] = 1.0;
    for (int k = 1; k <= n; ++k) b.v[n][k] = b.v[n - 1][k - 1] + (k <= n - 1 ? b.v[n - 1][k] : 0.0);
  }
  return b;
}
__constant__ BinomTable c_binom = make_binom();

__device__ inline double binom(int n, int k) { return c_binom.v[n][k]; }

// Offset of child quadrant from its parent's centre, in parent sides.
__device__ inline cplx quadrant_offset(int ix, int iy) {
  return {(ix & 1) ? 0.25 : -0.25, (iy & 1) ? 0.25 : -0.25};
}

// P2M: LANES lanes per source leaf (8 by default: eight leaves per wave);
// lanes stride over the leaf's sources, four sources per lane per step with
// their loads issued together, and the per-lane powers are summed across the
// lane group by DPP moves (plain VALU, no LDS round trips): within quads
// (lane xor 1, xor 2), then half rows (mirror: lane i with 7 - i), then rows
// (rotate by 8).  After each step the lanes of a group hold bitwise equal
// sums (the partner's value is added in the same order).  The source offsets
// from the leaf corner (units of the finest cell) are formed here from the
// ordered sources, as the packing step forms them for the near field, so P2M
// does not wait for that step: grid nodes from their packed index (exact
// half-integers), scattered sources from their FP64 coordinates.
template <int CTRL>
__device__ inline double dpp_add(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return v + __hiloint2double(hi, lo);
}

template <int LANES>
__device__ inline double group_sum(double v) {
  v = dpp_add<0xB1>(v);                     // quad_perm [1, 0, 3, 2]
  v = dpp_add<0x4E>(v);                     // quad_perm [2, 3, 0, 1]
  if (LANES >= 8) v = dpp_add<0x141>(v);    // row_half_mirror
  if (LANES >= 16) v = dpp_add<0x128>(v);   // row_ror:8
  return v;
}

// One source leaf c, LANES lanes (sub = the lane's index in its group); only
// a group with store set writes the leaf's coefficients.
template <int PM, int LANES>
__device__ inline void p2m_leaf(const TreeView& t, int c, int sub, bool store, const uint32_t* __restrict__ ij,
                                const double* __restrict__ xs, const double* __restrict__ ys, double x0, double y0,
                                double u, const double* __restrict__ w64, int p, double2* __restrict__ mp) {
  const double side = cell_side(t.D, t.lvl[c]);
  const double inv = 1.0 / side;
  const int sh = t.D - t.lvl[c];
  const int cxi = t.ix[c] << sh, cyi = t.iy[c] << sh;
  cplx acc[PM + 1];
#pragma unroll
  for (int k = 0; k <= PM; ++k) acc[k] = {0.0, 0.0};
  const int sb = t.sb[c], se = t.se[c];
  // four sources per lane per step (a missing source gets weight 0 at the
  // leaf corner and adds nothing)
  constexpr int kR = 4;
  for (int s = sb + sub; s < se; s += kR * LANES) {
    double ox[kR], oy[kR], w[kR];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int sr = s + r * LANES;
      const bool ok = sr < se;
      if (ij) {
        const uint32_t v = ok ? ij[sr] : (uint32_t)cxi | ((uint32_t)cyi << 16);
        ox[r] = (double)((int)(v & 0xFFFFu) - cxi) + 0.5;
        oy[r] = (double)((int)(v >> 16) - cyi) + 0.5;
      } else {
        ox[r] = ok ? (xs[sr] - x0) / u - (double)cxi : 0.0;
        oy[r] = ok ? (ys[sr] - y0) / u - (double)cyi : 0.0;
      }
      w[r] = ok ? w64[sr] : 0.0;
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const cplx z = {ox[r] * inv - 0.5, oy[r] * inv - 0.5};
      acc[0].x += w[r];
      cplx zk = {w[r] * z.x, w[r] * z.y};
#pragma unroll
      for (int k = 1; k <= PM; ++k) {
        acc[k] = cadd(acc[k], zk);
        zk = cmul(zk, z);
      }
    }
  }
#pragma unroll
  for (int k = 0; k <= PM; ++k) {
    acc[k].x = group_sum<LANES>(acc[k].x);
    acc[k].y = group_sum<LANES>(acc[k].y);
  }
  if (!store) return;
  double2* out = mp + (int64_t)c * (p + 1);
#pragma unroll
  for (int k = 0; k <= PM; ++k)
    if (k <= p && (k % LANES) == sub)
      out[k] = (k == 0) ? make_double2(acc[0].x, 0.0) : make_double2(-acc[k].x / k, -acc[k].y / k);
}

template <int PM, int LANES>
__global__ __launch_bounds__(256) void k_p2m(TreeView t, const int* __restrict__ sleaves, int n,
                                             const uint32_t* __restrict__ ij, const double* __restrict__ xs,
                                             const double* __restrict__ ys, double x0, double y0, double u,
                                             const double* __restrict__ w64, int p, double2* __restrict__ mp) {
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int li = (int)(gtid / LANES);
  const int sub = (int)(gtid % LANES);
  // every lane of a group takes part in the group sums: lanes past the last
  // leaf work on a copy of it and store nothing
  const int c = sleaves[li < n ? li : n - 1];
  p2m_leaf<PM, LANES>(t, c, sub, li < n, ij, xs, ys, x0, y0, u, w64, p, mp);
}

// G lanes per target cell: lane j of the group takes list entries j, j+G, ...
// and accumulates their local contributions in registers.  The group then
// sums them through LDS: every lane stores its 2 (p + 1) partial values, and
// lane q of the group adds value q over the G lanes in lane order (a fixed
// order, so the result is reproducible).
constexpr int kM2LBlock = 128;
template <int PM, int G>
__global__ __launch_bounds__(kM2LBlock) void k_m2l(TreeView t, const int* __restrict__ tcells, int n,
                                             const int* __restrict__ off, const int* __restrict__ cnt,
                                             const int* __restrict__ src, int p, double lnh,
                                             const double2* __restrict__ mp, double2* __restrict__ loc,
                                             int* __restrict__ flags) {
  static_assert(2 * (PM + 1) <= 2 * G, "two partial values per coefficient and at most two per lane");
  __builtin_assume(p >= 1);  // the orders the library accepts
  __shared__ double red[kM2LBlock][2 * (PM + 1)];
  const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int gi = (int)(gtid / G);
  const int sub = (int)(gtid % G);
  const bool live = gi < n;  // whole groups agree; every lane reaches the barrier
  const int A = live ? tcells[gi] : 0;
  const int D = t.D;
  const int lA = t.lvl[A];
  const double sA = cell_side(D, lA);
  const double cax = (t.ix[A] + 0.5) * sA, cay = (t.iy[A] + 0.5) * sA;
  cplx L[PM + 1];
#pragma unroll
  for (int k = 0; k <= PM; ++k) L[k] = {0.0, 0.0};
  const int e0 = live ? off[A] : 0, ne = live ? cnt[A] : 0;
  for (int e = sub; e < ne; e += G) {
    const int B = src[e0 + e];
    if ((unsigned)B >= (unsigned)t.ncells) {
      atomicOr(flags, kFlagBadIndex);
      continue;
    }
    const int lB = t.lvl[B];
    const double sB = cell_side(D, lB);
    const cplx z0 = {(t.ix[B] + 0.5) * sB - cax, (t.iy[B] + 0.5) * sB - cay};
    const double r2 = z0.x * z0.x + z0.y * z0.y;
    const double ir2 = 1.0 / r2;
    const cplx inv = {z0.x * ir2, -z0.y * ir2};  // 1 / z0
    const cplx tt = cscale(inv, sA);
    const cplx mr = cscale(inv, -sB);           // -s_B / z0
    const double2* a = mp + (int64_t)B * (p + 1);
    // all p + 1 coefficients are requested before the first is used: the
    // index is clamped to p (inside the cell's own block; p >= 1) and the
    // terms past p are zeroed, so no load waits behind a branch
    double2 av[PM + 1];
#pragma unroll
    for (int k = 0; k <= PM; ++k) av[k] = a[k <= p ? k : p];
    const double a0 = av[0].x;
    cplx bk[PM + 1];
    cplx pw = mr;
    cplx sum0 = {a0 * (0.5 * log(r2) + lnh), 0.0};
#pragma unroll
    for (int k = 1; k <= PM; ++k) {
      bk[k] = k <= p ? cmul({av[k].x, av[k].y}, pw) : cplx{0.0, 0.0};
      pw = cmul(pw, mr);
      sum0 = cadd(sum0, bk[k]);
    }
    L[0] = cadd(L[0], sum0);
    cplx tl = tt;
#pragma unroll
    for (int l = 1; l <= PM; ++l) {
      cplx s = {-a0 * (1.0 / l), 0.0};  // 1 / l is a compile-time constant of the unrolled loop
#pragma unroll
      for (int k = 1; k <= PM; ++k) s = cadd(s, cscale(bk[k], binom(l + k - 1, k - 1)));
      L[l] = cadd(L[l], cmul(tl, s));
      tl = cmul(tl, tt);
    }
  }
#pragma unroll
  for (int k = 0; k <= PM; ++k) {
    red[threadIdx.x][2 * k] = L[k].x;
    red[threadIdx.x][2 * k + 1] = L[k].y;
  }
  __syncthreads();
  if (!live) return;
  const int g0 = (int)(threadIdx.x - sub);  // the group's first lane in the block
  double* out = (double*)(loc + (int64_t)A * (p + 1));
  for (int q = sub; q < 2 * (p + 1); q += G) {
    double v = 0.0;
    for (int j = 0; j < G; ++j) v += red[g0 + j][q];
    out[q] = v;
  }
}

template <int PM>
__global__ __launch_bounds__(kWave) void k_downward(TreeView t, const int* __restrict__ tcells, int n, int p,
                                                    const double2* __restrict__ own, double2* __restrict__ loc,
                                                    const int* __restrict__ dense_off, int dense_levels, int top) {
  __shared__ double2 red[kWave][PM + 1];
  const int lane = threadIdx.x;
  const int sub = lane % kDownLanes;
  const int grp = lane / kDownLanes;
  const int i = blockIdx.x * (kWave / kDownLanes) + grp;
  const bool live = i < n;
  const int c = live ? tcells[i] : -1;
  cplx acc[PM + 1];
  down_terms<PM>(t, c, sub, p, own, dense_off, dense_levels, top, acc);
#pragma unroll
  for (int k = 0; k <= PM; ++k) red[lane][k] = make_double2(acc[k].x, acc[k].y);
  __syncthreads();
  if (!live) return;
  for (int m = sub; m <= p; m += kDownLanes) {
    const cplx s = down_sum<PM>(red + grp * kDownLanes, m);
    loc[(int64_t)c * (p + 1) + m] = make_double2(s.x, s.y);
  }
}

__global__ void k_l2p(TreeView t, int64_t m, const int* __restrict__ tleaf, int p, const double2* __restrict__ loc,
                      const double2* __restrict__ rel64, int fp32, double* __restrict__ far) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= m) return;
  const int c = tleaf[k];
  far[k] = l2p_eval(loc + (int64_t)c * (p + 1), p, rel64[k], t.D, t.lvl[c], fp32 != 0);
}

// M2P of the paper's tree-code (eq. pressTruncated evaluated at the targets):
// one wave per target leaf A, lane j on target j of each 64-target chunk, and
// for every source cell B of A's list
//   far += a_0 (ln|w| + ln s_B) + Re sum_{k=1..p} a'_k w^-k,   w = (t - z_B) / s_B,
// by Horner in u = 1/w.  The list is consumed 64 cells at a time: lane i
// loads cell i's geometry (corner difference to A in units of h, 1/s_B, the
// ln s_B term) and its coefficients into the wave's LDS slice, so the
// evaluation loop reads only LDS broadcasts.  The slice holds PM + 1
// coefficients per cell, zero above p (Horner over zeros leaves the sum
// unchanged), so the loop is fully unrolled and its reads are issued ahead of
// the arithmetic.  T = float for mixed precision (coefficients rounded when
// staged, each cell's term added to an FP64 sum), double otherwise.
constexpr double kLn2d = 0.69314718055994530942;
constexpr int kM2PWaves = 4;

template <class T>
struct Cx2 {
  T x, y;
};

template <class T, int PM>
__global__ __launch_bounds__(kM2PWaves* kWave) void k_m2p(TreeView t, const int* __restrict__ tleaves, int n,
                                                          const int* __restrict__ off, const int* __restrict__ cnt,
                                                          const int* __restrict__ src, int p, double lnh,
                                                          const double2* __restrict__ mp,
                                                          const double2* __restrict__ rel64, int nparts,
                                                          int64_t m, double* __restrict__ far,
                                                          int* __restrict__ flags) {
  extern __shared__ double m2p_lds[];
  const int w = threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  const int P1 = p + 1;
  constexpr int kSlot = PM + 3;  // per cell: 2 geometry slots and PM + 1 coefficients
  Cx2<T>* coef = (Cx2<T>*)m2p_lds + (size_t)w * kWave * kSlot;
  const int wid = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * kM2PWaves + w));
  if (wid >= n * nparts) return;
  // wave (leaf, part): the part's share of the leaf's list, its partial far
  // field stored at far[part * m + k] (the finalize step adds the parts)
  const int part = wid % nparts;
  const int A = tleaves[wid / nparts];
  const int shA = t.D - t.lvl[A];
  const int64_t ax2 = (int64_t)(2 * t.ix[A]) << shA, ay2 = (int64_t)(2 * t.iy[A]) << shA;
  const int nall = cnt[A];
  const int e0 = off[A] + (int)((int64_t)nall * part / nparts);
  const int ne = (int)((int64_t)nall * (part + 1) / nparts) - (int)((int64_t)nall * part / nparts);
  double* far_part = far + (int64_t)part * m;
  const int tb = t.tb[A], te = t.te[A];
  bool bad = false;
  for (int chunk = tb; chunk < te; chunk += kWave) {
    const int k = chunk + lane;
    const bool active = k < te;
    const double2 r64 = active ? rel64[k] : make_double2(0.0, 0.0);
    const T rx = (T)r64.x, ry = (T)r64.y;
    double acc_far = 0.0;
    for (int base = 0; base < ne; base += kWave) {
      const int nb = min(kWave, ne - base);
      // stage: lane i takes list entry base + i
      if (lane < nb) {
        int B = src[e0 + base + lane];
        Cx2<T>* cb = coef + (size_t)lane * kSlot;
        for (int q = P1; q <= PM; ++q) cb[2 + q] = {(T)0, (T)0};
        if ((unsigned)B >= (unsigned)t.ncells) {
          bad = true;
          cb[0] = {(T)0, (T)0};
          cb[1] = {(T)1, (T)0};
          for (int q = 0; q < P1; ++q) cb[2 + q] = {(T)0, (T)0};
        } else {
          const int shB = t.D - t.lvl[B];
          const double dx = 0.5 * (double)(ax2 - ((int64_t)(2 * t.ix[B] + 1) << shB));
          const double dy = 0.5 * (double)(ay2 - ((int64_t)(2 * t.iy[B] + 1) << shB));
          cb[0] = {(T)dx, (T)dy};
          cb[1] = {(T)ldexp(1.0, -shB), (T)((double)shB * kLn2d + lnh)};
          const double2* a = mp + (int64_t)B * P1;
          for (int q = 0; q < P1; ++q) {
            const double2 v = a[q];
            cb[2 + q] = {(T)v.x, (T)v.y};
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      for (int j = 0; j < nb; ++j) {
        const Cx2<T>* cb = coef + (size_t)j * kSlot;
        const Cx2<T> g0 = cb[0], g1 = cb[1];
        const T wx = (rx + g0.x) * g1.x, wy = (ry + g0.y) * g1.x;
        const T r2 = wx * wx + wy * wy;
        T ir2;
        if constexpr (sizeof(T) == 4)
          ir2 = __builtin_amdgcn_rcpf(r2);  // v_rcp_f32 (1 ulp): the mixed-precision path rounds to FP32 anyway
        else
          ir2 = (T)1 / r2;
        const T ux = wx * ir2, uy = -wy * ir2;
        T hx = (T)0, hy = (T)0;
#pragma unroll
        for (int q = PM; q >= 1; --q) {
          const Cx2<T> c = cb[2 + q];
          const T nx = hx * ux - hy * uy + c.x;
          const T ny = hx * uy + hy * ux + c.y;
          hx = nx;
          hy = ny;
        }
        const T re = hx * ux - hy * uy;
        T lg;
        if constexpr (sizeof(T) == 4)
          lg = (T)(0.5 * kLn2d) * __builtin_amdgcn_logf(r2) + g1.y;
        else
          lg = (T)0.5 * log(r2) + g1.y;
        acc_far += (double)(re + cb[2].x * lg);
      }
      // the slice is rewritten by the next batch only after every lane is done with it
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    if (active) far_part[k] = acc_far;
  }
  if (bad && lane == 0) atomicOr(flags, kFlagBadIndex);
}

#define PP_DISPATCH(p, KERNEL, GRID, BLOCK, STREAM, ...)                      \
  do {                                                                        \
    if ((p) <= 4)                                                             \
      KERNEL<4><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);                     \
    else if ((p) <= 8)                                                        \
      KERNEL<8><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);                     \
    else if ((p) <= 12)                                                       \
      KERNEL<12><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);                    \
    else if ((p) <= 16)                                                       \
      KERNEL<16><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);                    \
    else                                                                      \
      KERNEL<20><<<GRID, BLOCK, 0, STREAM>>>(__VA_ARGS__);                    \
  } while (0)

}  // namespace

template <int LANES>
void p2m_lanes(TreeView t, const int* sleaves, int n, const uint32_t* ij, const double* xs, const double* ys,
               double x0, double y0, double u, const double* w64, int p, double2* mp, hipStream_t s) {
  const unsigned g = (unsigned)(((int64_t)n * LANES + 255) / 256);
  if (p <= 4)
    k_p2m<4, LANES><<<g, 256, 0, s>>>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp);
  else if (p <= 8)
    k_p2m<8, LANES><<<g, 256, 0, s>>>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp);
  else if (p <= 12)
    k_p2m<12, LANES><<<g, 256, 0, s>>>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp);
  else if (p <= 16)
    k_p2m<16, LANES><<<g, 256, 0, s>>>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp);
  else
    k_p2m<kMaxP, LANES><<<g, 256, 0, s>>>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp);
}

void p2m(TreeView t, const int* sleaves, int n, const uint32_t* ij, const double* xs, const double* ys, double x0,
         double y0, double u, const double* w64, int p, double2* mp, hipStream_t s) {
  if (n <= 0) return;
  // lanes per leaf: PP_P2M_LANES = 4, 8 (default) or 16
  static const int lanes = [] {
    const char* e = std::getenv("PP_P2M_LANES");
    const int v = e ? std::atoi(e) : 8;
    return (v == 4 || v == 16) ? v : 8;
  }();
  if (lanes == 4)
    p2m_lanes<4>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp, s);
  else if (lanes == 16)
    p2m_lanes<16>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp, s);
  else
    p2m_lanes<8>(t, sleaves, n, ij, xs, ys, x0, y0, u, w64, p, mp, s);
}

void m2l(TreeView t, const int* tcells, int n, const int* m2l_off, const int* m2l_cnt, const int* m2l_src, int p,
         double h, const double2* mp, double2* loc, int* flags, hipStream_t s) {
  if (n <= 0) return;
  constexpr int G = 32;
  const unsigned g = (unsigned)(((int64_t)n * G + kM2LBlock - 1) / kM2LBlock);
  const double lnh = log(h);
  if (p <= 4)
    k_m2l<4, G><<<g, kM2LBlock, 0, s>>>(t, tcells, n, m2l_off, m2l_cnt, m2l_src, p, lnh, mp, loc, flags);
  else if (p <= 8)
    k_m2l<8, G><<<g, kM2LBlock, 0, s>>>(t, tcells, n, m2l_off, m2l_cnt, m2l_src, p, lnh, mp, loc, flags);
  else if (p <= 12)
    k_m2l<12, G><<<g, kM2LBlock, 0, s>>>(t, tcells, n, m2l_off, m2l_cnt, m2l_src, p, lnh, mp, loc, flags);
  else if (p <= 16)
    k_m2l<16, G><<<g, kM2LBlock, 0, s>>>(t, tcells, n, m2l_off, m2l_cnt, m2l_src, p, lnh, mp, loc, flags);
  else
    k_m2l<20, G><<<g, kM2LBlock, 0, s>>>(t, tcells, n, m2l_off, m2l_cnt, m2l_src, p, lnh, mp, loc, flags);
}

void downward(TreeView t, const int* tcells, int n, int p, const double2* own, double2* loc, const int* dense_off,
              int dense_levels, int top, hipStream_t s) {
  if (n <= 0) return;
  const unsigned g = (unsigned)((n + kWave / kDownLanes - 1) / (kWave / kDownLanes));
  PP_DISPATCH(p, k_downward, g, kWave, s, t, tcells, n, p, own, loc, dense_off, dense_levels, top);
}

void l2p(TreeView t, int64_t m, const int* tleaf, int p, const double2* loc, const double2* rel64, int fp32,
         double* far, hipStream_t s) {
  if (m <= 0) return;
  k_l2p<<<(unsigned)((m + 255) / 256), 256, 0, s>>>(t, m, tleaf, p, loc, rel64, fp32, far);
}

template <class T, int PM>
void m2p_launch(unsigned g, TreeView t, const int* tleaves, int n, const int* off, const int* cnt, const int* src,
                int p, double h, const double2* mp, const double2* rel64, int nparts, int64_t m, double* far,
                int* flags, hipStream_t s) {
  // up to 94 KB of LDS at PM = 20 in FP64 (gfx950 allows 160 KB per workgroup)
  const size_t bytes = (size_t)kM2PWaves * kWave * (PM + 3) * sizeof(Cx2<T>);
  static std::once_flag lds_opt_in;
  std::call_once(lds_opt_in, [bytes] {
    (void)hipFuncSetAttribute((const void*)k_m2p<T, PM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  });
  k_m2p<T, PM><<<g, kM2PWaves * kWave, bytes, s>>>(t, tleaves, n, off, cnt, src, p, log(h), mp, rel64, nparts, m,
                                                   far, flags);
}

template <class T>
void m2p_dispatch(unsigned g, TreeView t, const int* tleaves, int n, const int* off, const int* cnt, const int* src,
                  int p, double h, const double2* mp, const double2* rel64, int nparts, int64_t m, double* far,
                  int* flags, hipStream_t s) {
  if (p <= 4)
    m2p_launch<T, 4>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
  else if (p <= 8)
    m2p_launch<T, 8>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
  else if (p <= 12)
    m2p_launch<T, 12>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
  else if (p <= 16)
    m2p_launch<T, 16>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
  else
    m2p_launch<T, 20>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
}

void m2p(TreeView t, const int* tleaves, int n, const int* off, const int* cnt, const int* src, int p, double h,
         const double2* mp, const double2* rel64, int fp32, int nparts, int64_t m, double* far, int* flags,
         hipStream_t s) {
  if (n <= 0) return;
  const unsigned g = (unsigned)(((int64_t)n * nparts + kM2PWaves - 1) / kM2PWaves);
  if (fp32)
    m2p_dispatch<float>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
  else
    m2p_dispatch<double>(g, t, tleaves, n, off, cnt, src, p, h, mp, rel64, nparts, m, far, flags, s);
}

}  // namespace pp
