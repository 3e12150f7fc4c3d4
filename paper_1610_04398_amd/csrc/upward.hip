// Upward pass on the FP64 matrix cores: multipoles of the leaves and of the
// three levels above them in one launch (grid sources), and three levels of
// M2M per launch above those (all levels otherwise).
//
// With coefficients scaled by the cell side (expand.hip), P2M of an 8 x 8 block
// of grid nodes is a product of its 64 weights by position with one fixed
// 64 x 2(p + 1) matrix, and M2M of four children is a product of their
// 4 x 2(p + 1) real coefficients with one fixed matrix: dense contractions
// whose right-hand sides never change.  Truncation does not interfere: a
// parent's coefficient l depends on its children's coefficients k <= l only.
//
// One workgroup takes a cell of level D - 6 (64 x 64 nodes): it lays the
// cell's weights out by position in LDS (at most 4,096 nodes, zero where a
// node was culled), forms the multipoles of the 64 blocks of level D - 3 and
// sums them up level by level.  Which of those cells the tree has does not
// matter for the arithmetic (a leaf 16, 32 or 64 nodes wide gets the sum over
// its blocks, a block split further by targets gets its own), only for what
// is stored.  Cells the blocks do not cover (leaves above level D - 6, cells
// below level D - 3) take one wave each in the same launch.
//
// What bounds it: at 4096^2 (5.9M sources, 1,564 workgroups) the weights and
// node indices are 71 MB and the products 11 us of the matrix cores; a
// workgroup's chain (cell record, sources, 16 products, three levels of 7 with
// two barriers each) takes 8 us alone, 13 beside others, and four of them fill a
// compute unit (at p = 12 its 32 wave slots as well as its LDS), so the launch
// takes 37 us there, 13 at 1024^2, 8 at 64^2.  P2M by leaves and M2M by subtrees staged in LDS took 28 + 27 us at
// 4096^2 and 10 + 13 at 1024^2, and the launches above them 13 + 9 us where
// these take 7 + 5.
//
// A workgroup finds its cells in the tree build's prefix table where that
// reaches its deepest level, and by the cells' child links below.  One P2M and
// one M2M kernel serve every depth, so a request's expansions are the same in a
// forest, whose extra top levels push its cells below the table.  A full 8192^2
// field (4.2M leaves; the blocks are one level below the table): 363 us for P2M
// and M2M, 690 with P2M by lane groups per leaf and a second M2M kernel there.
#include <algorithm>
#include <mutex>

#include "blockscan.h"
#include "internal.h"
#include "leafpass.h"
#include "listwalk.h"
#include "near.h"

namespace pp {

namespace {
typedef double v4d __attribute__((ext_vector_type(4)));

// A workgroup has four waves per tile of 16 matrix columns: wave = row tile (16
// of the 64 blocks; in M2M the child quadrant) + 4 x column tile.
constexpr int kUpQuads = 4;
template <int TILES>
constexpr int kUpBlock = kUpQuads * TILES * kWave;
constexpr int kUpCols = 48;                // columns of the matrices: 2 (kMaxP + 1) = 42, in tiles of 16
constexpr int kUpRows = 44;                // real coefficients of a child, padded to steps of 4
constexpr int kUpWidth = 64;               // nodes across a workgroup's cell
constexpr int kUpNodes = kUpWidth * kUpWidth;
constexpr int kUpSlots = 85;               // 1 + 4 + 16 + 64 cells
constexpr int kUpPitch = 68;               // doubles per row of 64 weights in LDS
__host__ __device__ constexpr int up_first(int d) { return ((1 << (2 * d)) - 1) / 3; }

// Z[pos][2k], Z[pos][2k + 1]: real and imaginary part of -zeta^k / k (1 and 0
// for k = 0), zeta = ((x + 1/2) / 8 - 1/2, (y + 1/2) / 8 - 1/2), pos the Morton
// index of (x, y).
struct P2MMatrix {
  double v[64][kUpCols];
};
constexpr P2MMatrix make_p2m_matrix() {
  P2MMatrix z{};
  for (int pos = 0; pos < 64; ++pos) {
    const int x = (pos & 1) | ((pos >> 1) & 2) | ((pos >> 2) & 4), y = ((pos >> 1) & 1) | ((pos >> 2) & 2) | ((pos >> 3) & 4);
    const double zx = (x + 0.5) * 0.125 - 0.5, zy = (y + 0.5) * 0.125 - 0.5;
    double ax = 1.0, ay = 0.0;
    z.v[pos][0] = 1.0;
    for (int k = 1; k < kUpCols / 2; ++k) {
      const double nx = ax * zx - ay * zy, ny = ax * zy + ay * zx;
      ax = nx;
      ay = ny;
      z.v[pos][2 * k] = -ax / k;
      z.v[pos][2 * k + 1] = -ay / k;
    }
  }
  return z;
}
__device__ const P2MMatrix c_p2m = make_p2m_matrix();

// With coefficients scaled by the cell side, the shift of a child's expansion to
// its parent's centre depends only on the child's quadrant q, through d_q =
// (+-1/4, +-1/4) (the child centre's offset in parent sides).  From eq.
// expandedShift with the corrected S term:
//   a'_l(parent) = sum_q sum_{k=0..l} T_q[l][k] a'_k(child q),
//   T_q[0][0] = 1,  T_q[l][0] = -d_q^l / l,  T_q[l][k] = C(l-1, k-1) 2^-k d_q^(l-k),
// here on real coefficients: row 2k + (0: real, 1: imaginary) of the child,
// column 2l + ... of the parent.  The table is built at compile time; every entry
// but the 1/l ones is exact.
struct M2MMatrix {
  double v[4][kUpRows][kUpCols];
};
constexpr M2MMatrix make_m2m_matrix() {
  M2MMatrix t{};
  for (int q = 0; q < 4; ++q) {
    const double dx = (q & 1) ? 0.25 : -0.25, dy = (q & 2) ? 0.25 : -0.25;
    double pw[kUpCols / 2 + 1][2] = {};
    pw[0][0] = 1.0;
    for (int n = 1; n <= kUpCols / 2; ++n) {
      pw[n][0] = pw[n - 1][0] * dx - pw[n - 1][1] * dy;
      pw[n][1] = pw[n - 1][0] * dy + pw[n - 1][1] * dx;
    }
    for (int l = 0; l < kUpCols / 2; ++l) {
      double c = 1.0, two = 0.5;  // C(l - 1, k - 1) and 2^-k
      for (int k = 0; k <= l && 2 * k + 1 < kUpRows; ++k) {
        double x = 0.0, y = 0.0;
        if (k == 0) {
          x = l == 0 ? 1.0 : -pw[l][0] / l;
          y = l == 0 ? 0.0 : -pw[l][1] / l;
        } else {
          x = c * two * pw[l - k][0];
          y = c * two * pw[l - k][1];
          c = c * (l - k) / k;
          two *= 0.5;
        }
        t.v[q][2 * k][2 * l] = x;
        t.v[q][2 * k][2 * l + 1] = y;
        t.v[q][2 * k + 1][2 * l] = -y;
        t.v[q][2 * k + 1][2 * l + 1] = x;
      }
    }
  }
  return t;
}
__device__ const M2MMatrix c_m2mr = make_m2m_matrix();

// Barrier between LDS writes and reads of a workgroup.  (__syncthreads also
// waits for the global stores in flight, here the finished expansions, which
// nothing in the workgroup reads: about a microsecond per level.)
__device__ inline void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A workgroup's cells: slots as in [0] = R, [1..4] its children in quadrant
// order, [5..20], [21..84]; id < 0: not a cell of the tree.
struct UpSlots {
  int id[kUpSlots];
  int own[kUpSlots];  // holds a final expansion that is not to be recomputed (a leaf), upper launches only
};

__device__ inline int up_steps(int p) { return (2 * (p + 1) + 3) / 4; }
__device__ inline int up_pitch(int p) { return 4 * up_steps(p) + 1; }

// The wave's fragment of the M2M matrix (child quadrant q, column tile tl),
// kept in registers for every level.  Tile tl (parent coefficients 8 tl .. 8 tl
// + 7) needs the child's first 4 (tl + 1) steps of four real coefficients only.
template <int TILES>
__device__ inline void load_frags(double (&f)[4 * TILES]) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, q = wave % kUpQuads, tl = wave / kUpQuads;
#pragma unroll
  for (int s = 0; s < 4 * TILES; ++s) {
    const int row = 4 * s + lane / 16;
    f[s] = s < 4 * (tl + 1) && row < kUpRows ? c_m2mr.v[q][row < kUpRows ? row : 0][16 * tl + lane % 16] : 0.0;
  }
}
// The fragments are in registers from here on.  (An empty statement that takes
// the values keeps the compiler from moving the loads down to their uses, each
// behind its own wait.)
template <int N>
__device__ inline void pin(double (&f)[N]) {
#pragma unroll
  for (int s = 0; s < N; ++s) asm volatile("" : "+v"(f[s]));
}

// Levels levels-1 .. 0 of the workgroup's subtree from the expansions E of its
// deepest slots (and of those marked own).  Wave (q, tl) multiplies the
// children of quadrant q with column tile tl; the four quadrants' products
// meet in LDS and are added in quadrant order.  E: kUpSlots rows of
// up_pitch(p); part: kUpQuads x 16 x 16 TILES.
template <int TILES>
__device__ inline void up_levels(double* E, double* part, const UpSlots& sl, const double (&f)[4 * TILES], int levels,
                                 int p, double2* __restrict__ mp) {
  constexpr int kCols = 16 * TILES;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave, q = wave % kUpQuads, tl = wave / kUpQuads;
  const int r16 = lane % 16, kq = lane / 16;
  const int ks = up_steps(p), pitch = up_pitch(p), cols = 2 * (p + 1);
  const int steps = min(ks, 4 * (tl + 1));
  const int pi = tid / kCols, pc = tid % kCols;  // parent and column that this thread adds up
  for (int d = levels - 1; d >= 0; --d) {
    const int lo = up_first(d), n = 1 << (2 * d);
    const double* row = E + (up_first(d + 1) + 4 * min(r16, n - 1) + q) * pitch + kq;
    double a[4 * TILES];
#pragma unroll
    for (int s = 0; s < 4 * TILES; ++s) a[s] = s < steps ? row[4 * s] : 0.0;
    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4 * TILES; ++s)
      if (s < steps) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], f[s], acc, 0, 0, 0);
    // lane (r16, kq), element e: parent 4 e + kq, column 16 tl + r16
#pragma unroll
    for (int e = 0; e < 4; ++e) part[(q * 16 + 4 * e + kq) * kCols + 16 * tl + r16] = acc[e];
    lds_barrier();
    if (pi < n && !sl.own[lo + pi]) {
      double v = 0.0;
#pragma unroll
      for (int c = 0; c < kUpQuads; ++c) v += part[(c * 16 + pi) * kCols + pc];
      const int id = sl.id[lo + pi];
      if (pc < 4 * ks) E[(lo + pi) * pitch + pc] = v;
      if (id >= 0 && pc < cols) reinterpret_cast<double*>(mp + (int64_t)id * (p + 1))[pc] = v;
    }
    lds_barrier();
  }
}

// Slot i of the subtree of R (level L, Morton index PR in its level): its cell.
__device__ inline int up_cell(int i, int R, int L, int64_t PR, const int* __restrict__ dense_off) {
  int d = 0;
  while (up_first(d + 1) <= i) ++d;
  if (d == 0) return R;
  const int64_t idx = ((((int64_t)1 << (2 * (L + d))) - 1) / 3) + (PR << (2 * d)) + (i - up_first(d));
  return dense_off[idx];
}

// The same by the child links of the cells' records (rR: R's), for levels below
// the prefix table: four threads per parent slot, a load for each level.  A child's quadrant
// follows from its coordinates.  Cells without sources are left out (id -1).  own
// is < 0 for a leaf.  (The whole workgroup calls it; the slots are complete after
// the caller's next barrier.)
__device__ inline void up_linked_cells(UpSlots& sl, const int4* __restrict__ rec, int R, int4 rR, int levels) {
  const int tid = threadIdx.x;
  auto links = [](int4 r) { return r.z < 0 ? -1 : (r.z << 3) | rec_nchild(r); };  // (cell numbers are below 2^28)
  if (tid < kUpSlots) {
    sl.id[tid] = tid == 0 ? R : -1;
    sl.own[tid] = tid == 0 ? links(rR) : -1;
  }
  for (int d = 0; d < levels; ++d) {
    lds_barrier();
    const int par = up_first(d) + tid / 4, j = tid % 4;
    if (tid >= 4 << (2 * d) || sl.id[par] < 0) continue;
    const int kids = sl.own[par];
    if (kids < 0 || j >= (kids & 7)) continue;
    const int c = (kids >> 3) + j;
    const int4 r = rec[c];
    if (!rec_has_src(r)) continue;
    const int slot = up_first(d + 1) + 4 * (tid / 4) + ((r.x & 1) | ((r.y & 1) << 1));
    sl.id[slot] = c;
    sl.own[slot] = links(r);
  }
}

// P2M of one cell by one wave, a source per lane and pass.
__device__ inline double wave_total(double v) {
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ inline void p2m_wave(const TreeView& t, int c, const uint32_t* __restrict__ ij,
                                const double* __restrict__ w64, int p, double2* __restrict__ mp) {
  const int lane = threadIdx.x % kWave;
  const int sh = t.D - t.lvl[c];
  const int cx = t.ix[c] << sh, cy = t.iy[c] << sh;
  const int sb = t.sb[c], se = t.se[c];
  const double inv = ldexp(1.0, -sh);
  double2* out = mp + (int64_t)c * (p + 1);
  for (int s0 = sb; s0 < se; s0 += kWave) {
    const int s = s0 + lane;
    const bool ok = s < se;
    const uint32_t v = ok ? ij[s] : 0u;
    const double zx = ok ? ((double)((int)(v & 0xFFFFu) - cx) + 0.5) * inv - 0.5 : 0.0;
    const double zy = ok ? ((double)((int)(v >> 16) - cy) + 0.5) * inv - 0.5 : 0.0;
    double ax = ok ? w64[s] : 0.0, ay = 0.0;
    for (int k = 0; k <= p; ++k) {
      const double x = wave_total(ax), y = wave_total(ay);
      if (lane == 0) {
        const double g = k == 0 ? 1.0 : -1.0 / k;
        const double2 before = s0 == sb ? make_double2(0.0, 0.0) : out[k];
        out[k] = make_double2(before.x + g * x, before.y + g * y);
      }
      const double nx = ax * zx - ay * zy;
      ay = ax * zy + ay * zx;
      ax = nx;
    }
  }
}

// Workgroups [0, c1 - c0): the cells [c0, c1) of level L = D - 6.  The next
// ones: a wave per cell of [0, c0) that is a leaf (wider than a workgroup's
// cell) and of [f0, f1) (narrower than a block of 8 x 8 nodes).
struct UpP2M {
  TreeView t;
  int c0, c1, f0, f1, L;
  const uint32_t* ij;
  const double* w64;
  int p;
  double2* mp;
  UpCells cells;
};
int up_p2m_blocks(const UpP2M& a, int tiles) {
  const int waves = a.c0 + std::max(a.f1 - a.f0, 0), per = kUpQuads * tiles;
  return (a.c1 - a.c0) + (waves + per - 1) / per;
}

template <int TILES>
__device__ inline void up_p2m_block(const UpP2M& a, int blk, double* up_lds, UpSlots& sl) {
  const TreeView& t = a.t;
  const int c0 = a.c0, p = a.p;
  double2* __restrict__ mp = a.mp;
  constexpr int kBlock = kUpBlock<TILES>;
  constexpr int kSources = (kUpNodes + kBlock - 1) / kBlock;  // per thread
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  if (blk >= a.c1 - c0) {  // uniform per workgroup
    const int i = (blk - (a.c1 - c0)) * (kBlock / kWave) + wave;
    const int c = i < c0 ? i : a.f0 + (i - c0);
    if (c >= (i < c0 ? c0 : a.f1) || t.se[c] <= t.sb[c] || (i < c0 && t.child[c] >= 0)) return;
    p2m_wave(t, c, a.ij, a.w64, p, mp);
    return;
  }
  const int R = c0 + blk;
  const int sb = t.sb[R], n = t.se[R] - sb;
  const int ix = t.ix[R], iy = t.iy[R];
  const int4 rR = a.cells.rec ? a.cells.rec[R] : int4{};
  const int r16 = lane % 16, kq = lane / 16, rt = wave % kUpQuads, tl = wave / kUpQuads;
  if (n <= 0) return;  // uniform
  // the cell's sources, all requested at once
  uint32_t v[kSources];
  double w[kSources];
#pragma unroll
  for (int i = 0; i < kSources; ++i) {
    const int s = tid + i * kBlock;
    v[i] = s < n ? a.ij[sb + s] : 0u;
    w[i] = s < n ? a.w64[sb + s] : 0.0;
  }
  if (a.cells.rec) {  // uniform
    up_linked_cells(sl, a.cells.rec, R, rR, 3);
    lds_barrier();
    if (tid < kUpSlots) sl.own[tid] = 0;
  } else if (tid < kUpSlots) {
    sl.id[tid] = up_cell(tid, R, a.L, (int64_t)morton((uint32_t)ix, (uint32_t)iy), a.cells.off);
    sl.own[tid] = 0;
  }
  double* W = up_lds;
  for (int i = 2 * tid; i < 64 * kUpPitch; i += 2 * kBlock) *reinterpret_cast<double2*>(W + i) = make_double2(0.0, 0.0);
  lds_barrier();
  // weight of node (x, y) of the cell at its Morton index: row of its 8 x 8
  // block, column of its place in the block.  x and y sit in the halves of one
  // word and are spread together.
  const uint32_t base = ((uint32_t)ix << 6) | ((uint32_t)iy << 22);
#pragma unroll
  for (int i = 0; i < kSources; ++i) {
    uint32_t m = v[i] - base;
    const bool ok = tid + i * kBlock < n && (m & 0xFFC0FFC0u) == 0;
    m = (m | (m << 4)) & 0x030F030Fu;
    m = (m | (m << 2)) & 0x33333333u;
    m = (m | (m << 1)) & 0x55555555u;
    m = (m | (m >> 15)) & 0xFFFu;
    if (ok) W[m + (kUpPitch - 64) * (m >> 6)] = w[i];
  }
  // the wave's fragments of both matrices (requested here, not earlier: the
  // sources' registers are free now, and with at most 64 registers four
  // workgroups share a compute unit, which hides these loads)
  double z[16], f[4 * TILES];
#pragma unroll
  for (int s = 0; s < 16; ++s) z[s] = c_p2m.v[4 * s + kq][16 * tl + r16];
  lds_barrier();
  const int ks = up_steps(p), pitch = up_pitch(p), cols = 2 * (p + 1);
  v4d acc = {0.0, 0.0, 0.0, 0.0};
  const double* wrow = W + (16 * rt + r16) * kUpPitch + kq;
#pragma unroll
  for (int h = 0; h < 16; h += 4) {
    double x[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) x[s] = wrow[4 * (h + s)];
#pragma unroll
    for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[s], z[h + s], acc, 0, 0, 0);
  }
  load_frags<TILES>(f);
  lds_barrier();  // the weights are read: their place takes the expansions
  double* E = up_lds;
  double* part = E + kUpSlots * pitch;
  const int col = 16 * tl + r16;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int slot = up_first(3) + 16 * rt + 4 * e + kq;
    const int id = sl.id[slot];
    if (col < 4 * ks) E[slot * pitch + col] = acc[e];
    if (col < cols && id >= 0) reinterpret_cast<double*>(mp + (int64_t)id * (p + 1))[col] = acc[e];
  }
  lds_barrier();
  up_levels<TILES>(E, part, sl, f, 3, p, mp);
}

template <int TILES>
__global__ __launch_bounds__(kUpBlock<TILES>, TILES == 1 ? 4 : TILES == 2 ? 8 : 6) void k_up_p2m(UpP2M a) {
  extern __shared__ __align__(16) double up_lds[];  // (16-byte accesses: aligned past the static LDS)
  __shared__ UpSlots sl;
  up_p2m_block<TILES>(a, (int)blockIdx.x, up_lds, sl);
}

// M2M from the cells of level L + levels up to the cells [c0, c1) of level L,
// a workgroup per cell.  Slots of the deepest level, and leaves above it, hold
// final expansions.
struct UpM2M {
  TreeView t;
  int c0, c1, L, levels, p;
  double2* mp;
  UpCells cells;
};
template <int TILES>
__device__ inline void up_m2m_block(const UpM2M& a, int blk, double* up_lds, UpSlots& sl) {
  const TreeView& t = a.t;
  const int levels = a.levels, p = a.p;
  double2* __restrict__ mp = a.mp;
  const int tid = threadIdx.x;
  const int R = a.c0 + blk;
  double f[4 * TILES];
  load_frags<TILES>(f);
  const int4 rR = a.cells.rec ? a.cells.rec[R] : int4{};
  if (a.cells.rec ? !rec_has_src(rR) || rR.z < 0 : t.se[R] <= t.sb[R] || t.child[R] < 0) return;  // uniform: nothing to form
  const int ks = up_steps(p), pitch = up_pitch(p), cols = 2 * (p + 1);
  const int nslots = up_first(levels + 1), deepest = up_first(levels);
  if (a.cells.rec) {  // uniform
    up_linked_cells(sl, a.cells.rec, R, rR, levels);
    lds_barrier();
    if (tid < nslots) sl.own[tid] = sl.id[tid] >= 0 && (tid >= deepest || sl.own[tid] < 0);
  } else if (tid < nslots) {
    int c = up_cell(tid, R, a.L, (int64_t)morton((uint32_t)t.ix[R], (uint32_t)t.iy[R]), a.cells.off);
    const int at = c >= 0 ? c : R;
    if (t.se[at] <= t.sb[at]) c = -1;  // targets only: no expansion
    sl.id[tid] = c;
    sl.own[tid] = c >= 0 && (tid >= deepest || t.child[at] < 0);
  }
  __syncthreads();
  double* E = up_lds;
  double* part = E + kUpSlots * pitch;
  // 16 slots at a time, a lane per column, every load requested before the first is stored
  constexpr int kCols = 16 * TILES, kGroups = (kUpSlots + 15) / 16;
  const int row = tid / kCols, col = tid % kCols;
  double x[kGroups];
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int i = 16 * g + row;
    const int id = i < nslots && sl.own[i] ? sl.id[i] : -1;
    x[g] = id >= 0 && col < cols ? reinterpret_cast<const double*>(mp + (int64_t)id * (p + 1))[col] : 0.0;
  }
#pragma unroll
  for (int g = 0; g < kGroups; ++g) {
    const int i = 16 * g + row;
    if (i < nslots && col < 4 * ks) E[i * pitch + col] = x[g];
  }
  pin(f);
  __syncthreads();
  up_levels<TILES>(E, part, sl, f, levels, p, mp);
}

template <int TILES>
__global__ __launch_bounds__(kUpBlock<TILES>) void k_up_m2m(UpM2M a) {
  extern __shared__ __align__(16) double up_lds[];  // (16-byte accesses: aligned past the static LDS)
  __shared__ UpSlots sl;
  up_m2m_block<TILES>(a, (int)blockIdx.x, up_lds, sl);
}

// ---- two launches of a small solve -------------------------------------------------
// Launches of independent passes joined into one, for solves whose kernels are
// all too small to fill the chip (compact_setup, compact_near in internal.h).

// Interaction lists (a wave per target cell), then P2M by blocks, then the
// target preparation (a wave per target leaf).
template <int TILES, int CAP, bool TREECODE>
__global__ __launch_bounds__(kUpBlock<TILES>) void k_compact_setup(ListArgs la, UpP2M ua, int up_blocks, LeafPass lp) {
  extern __shared__ __align__(16) double up_lds[];  // (16-byte accesses: aligned past the static LDS)
  __shared__ UpSlots sl;
  constexpr int kWaves = kUpQuads * TILES;
  const int list_blocks = (la.n + kWaves - 1) / kWaves;
  const int blk = (int)blockIdx.x;
  if (blk < list_blocks) {  // uniform per workgroup, as below
    const int w = threadIdx.x / kWave;
    const int wid = __builtin_amdgcn_readfirstlane(blk * kWaves + w);
    int* buf = reinterpret_cast<int*>(up_lds) + w * 2 * CAP;
    if (wid >= la.n) return;
    if constexpr (TREECODE)
      walk_leaf_treecode<CAP>(la, wid, buf);
    else
      walk_cell<CAP>(la, wid, buf);
  } else if (blk < list_blocks + up_blocks) {
    up_p2m_block<TILES>(ua, blk - list_blocks, up_lds, sl);
  } else {
    run_leaf_pass(lp, blk - list_blocks - up_blocks);
  }
}

// The first M2M launch's workgroups, then the near field (a wave per target
// leaf and list part) in FP32 from the unpacked sources, or in FP64.
template <int TILES, bool FP64>
__global__ __launch_bounds__(kUpBlock<TILES>) void k_compact_near(UpM2M ua, int m2m_blocks, P2PArgs na) {
  extern __shared__ __align__(16) double up_lds[];  // (16-byte accesses: aligned past the static LDS)
  __shared__ UpSlots sl;
  constexpr int kWaves = kUpQuads * TILES;
  const int blk = (int)blockIdx.x;
  if (blk < m2m_blocks) {  // uniform per workgroup
    up_m2m_block<TILES>(ua, blk, up_lds, sl);
    return;
  }
  const int w = threadIdx.x / kWave;
  const int wid = __builtin_amdgcn_readfirstlane(
      xcd_contiguous(blk - m2m_blocks, (int)gridDim.x - m2m_blocks) * kWaves + w);
  if constexpr (FP64) load_log_table(up_lds, na.log_tab);  // (a barrier)
  if (wid >= na.ntleaves * na.count) return;
  if constexpr (FP64)
    near64_wave(na, up_lds, wid);
  else
    near32_wave<true>(na, reinterpret_cast<Staged*>(up_lds) + w * kWave, wid);
}

int host_pitch(int p) { return 4 * ((2 * (p + 1) + 3) / 4) + 1; }
int tiles_for(int p) { return (2 * (p + 1) + 15) / 16; }
size_t up_lds_bytes(int p) {
  const size_t e = ((size_t)kUpSlots * host_pitch(p) + (size_t)kUpQuads * 16 * 16 * tiles_for(p)) * sizeof(double);
  return std::max(e, (size_t)64 * kUpPitch * sizeof(double));
}

// dynamic LDS above the default limit
template <class K>
void allow_lds(K kernel, size_t bytes, std::once_flag& once) {
  std::call_once(once, [&] {
    (void)hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  });
}
size_t list_lds_bytes(int tiles, int cap) { return (size_t)kUpQuads * tiles * 2 * cap * sizeof(int); }

template <int TILES>
void launch_p2m(const UpP2M& a, hipStream_t s) {
  const unsigned g = (unsigned)up_p2m_blocks(a, TILES);
  if (g == 0) return;
  static std::once_flag once;
  allow_lds(k_up_p2m<TILES>, up_lds_bytes(kMaxP), once);
  k_up_p2m<TILES><<<g, kUpBlock<TILES>, up_lds_bytes(a.p), s>>>(a);
}

template <int TILES>
void launch_m2m(const UpM2M& a, hipStream_t s) {
  static std::once_flag once;
  allow_lds(k_up_m2m<TILES>, up_lds_bytes(kMaxP), once);
  k_up_m2m<TILES><<<(unsigned)(a.c1 - a.c0), kUpBlock<TILES>, up_lds_bytes(a.p), s>>>(a);
}

template <int TILES, int CAP, bool TREECODE>
void launch_setup(const ListArgs& la, const UpP2M& ua, LeafPass lp, hipStream_t s) {
  constexpr int kWaves = kUpQuads * TILES;
  lp.pack_blocks = 0;
  lp.prep_blocks = (lp.gb.nt + kWaves - 1) / kWaves;
  const int up = up_p2m_blocks(ua, TILES);
  const size_t lds = std::max(up_lds_bytes(ua.p), list_lds_bytes(TILES, CAP));
  static std::once_flag once;
  allow_lds(k_compact_setup<TILES, CAP, TREECODE>, std::max(up_lds_bytes(kMaxP), list_lds_bytes(TILES, CAP)), once);
  const unsigned g = (unsigned)((la.n + kWaves - 1) / kWaves + up + lp.prep_blocks);
  if (g > 0) k_compact_setup<TILES, CAP, TREECODE><<<g, kUpBlock<TILES>, lds, s>>>(la, ua, up, lp);
}

template <int TILES>
void setup_for(const ListArgs& la, bool treecode, int tier, const UpP2M& ua, const LeafPass& lp, hipStream_t s) {
  if (tier <= 0 && treecode)
    launch_setup<TILES, kFrontierTiers[0], true>(la, ua, lp, s);
  else if (tier <= 0)
    launch_setup<TILES, kFrontierTiers[0], false>(la, ua, lp, s);
  else if (treecode)
    launch_setup<TILES, kFrontierTiers[1], true>(la, ua, lp, s);
  else
    launch_setup<TILES, kFrontierTiers[1], false>(la, ua, lp, s);
}

template <int TILES, bool FP64>
void launch_near(const UpM2M& ua, const P2PArgs& na, hipStream_t s) {
  constexpr int kWaves = kUpQuads * TILES;
  const int m2m = std::max(ua.c1 - ua.c0, 0);
  const unsigned g = (unsigned)(m2m + (na.ntleaves * na.count + kWaves - 1) / kWaves);
  const size_t own = FP64 ? kLogTable * sizeof(double) : (size_t)kWaves * kWave * sizeof(Staged);
  const size_t lds = std::max(m2m > 0 ? up_lds_bytes(ua.p) : 0, own);
  static std::once_flag once;
  allow_lds(k_compact_near<TILES, FP64>, std::max(up_lds_bytes(kMaxP), own), once);
  if (g > 0) k_compact_near<TILES, FP64><<<g, kUpBlock<TILES>, lds, s>>>(ua, m2m, na);
}
}  // namespace

bool compact_tier_ok(int num, int den, int tier_boost) { return frontier_tier_for(num, den) + tier_boost <= 1; }

void compact_setup(const ListArgs& la, bool treecode, int tier_boost, TreeView t, int c0, int c1, int f0, int f1, int L,
                   const uint32_t* ij, const double* w64, int p, double2* mp, const UpCells& cells,
                   const LeafPass& lp, hipStream_t s) {
  const UpP2M ua{t, c0, c1, f0, f1, L, ij, w64, p, mp, cells};
  const int tier = frontier_tier_for(la.num, la.den) + tier_boost;
  switch (tiles_for(p)) {
    case 1: setup_for<1>(la, treecode, tier, ua, lp, s); break;
    case 2: setup_for<2>(la, treecode, tier, ua, lp, s); break;
    default: setup_for<3>(la, treecode, tier, ua, lp, s);
  }
}

void compact_near(const P2PArgs& na, bool fp64, TreeView t, int c0, int c1, int L, int levels, int p, double2* mp,
                  const UpCells& cells, hipStream_t s) {
  const UpM2M ua{t, c0, c1, L, levels, p, mp, cells};
  switch (tiles_for(p)) {
    case 1: fp64 ? launch_near<1, true>(ua, na, s) : launch_near<1, false>(ua, na, s); break;
    case 2: fp64 ? launch_near<2, true>(ua, na, s) : launch_near<2, false>(ua, na, s); break;
    default: fp64 ? launch_near<3, true>(ua, na, s) : launch_near<3, false>(ua, na, s);
  }
}

void up_p2m(TreeView t, int c0, int c1, int f0, int f1, int L, const uint32_t* ij, const double* w64, int p,
            double2* mp, const UpCells& cells, hipStream_t s) {
  const UpP2M a{t, c0, c1, f0, f1, L, ij, w64, p, mp, cells};
  switch (tiles_for(p)) {
    case 1: launch_p2m<1>(a, s); break;
    case 2: launch_p2m<2>(a, s); break;
    default: launch_p2m<3>(a, s);
  }
}

void up_m2m(TreeView t, int c0, int c1, int L, int levels, int p, double2* mp, const UpCells& cells, hipStream_t s) {
  if (c1 <= c0) return;
  const UpM2M a{t, c0, c1, L, levels, p, mp, cells};
  switch (tiles_for(p)) {
    case 1: launch_m2m<1>(a, s); break;
    case 2: launch_m2m<2>(a, s); break;
    default: launch_m2m<3>(a, s);
  }
}

}  // namespace pp
