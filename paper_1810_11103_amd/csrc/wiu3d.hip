// Three-dimensional Euler equations on curvilinear grids (gfx950, fp64): the
// paper's method in its general form (Sec. 2.1, Eq. 2.2) -- metrics in the
// symmetric conservative form (Eq. 2.4) with each scheme's central operator,
// Jacobian by Eq. 2.5, the characteristic projection of Sec. 3.4 with five
// eigenvectors, the WENOIU midpoint fluxes and upwind-biased difference of
// every scheme, TVD-RK3; the scheme options in kernels of their own.
//
// A direction pass is one LDS-tiled sweep (states staged once, one item per
// lane, item records in LDS, the flux difference and the stage update in the
// same kernel), with lanes along i wherever global memory is touched so
// loads and stores coalesce whatever the line direction.  The passes run
// zeta, eta, xi: the xi pass, whose lines are contiguous in memory, writes
// dU/dt or the RK stage (and the next state's maxima).  On grids that do not fill
// the chip zeta and eta are one launch.
#include "wenoiu.h"

#include "wiu_kernels.hpp"

namespace wiu {

constexpr double TAG_MAGIC3 = 1810.111033;
constexpr int NP3 = 19;   // metric planes (see wenoiu.h)

struct Dims3 {
  int n[3], bc[3];
  double L[3];
  long long np;        // nodes
  int mp[2];           // metric box pitches nx+2G, ny+2G
  long long mplane;    // metric plane size
};

WIU_DEV long long m3idx(const Dims3& d, int i, int j, int k) {
  return ((long long)(k + GHOST) * d.mp[1] + (j + GHOST)) * d.mp[0] + (i + GHOST);
}
WIU_DEV long long u3idx(const Dims3& d, int i, int j, int k) {
  return ((long long)k * d.n[1] + j) * d.n[0] + i;
}

// ===========================================================================
// Coordinates at any position: a node coordinate (base) plus an offset --
// shifts across periodic seams, and beyond transmissive ends the linear
// extension direction by direction (trilinear at edges and corners, as
// sum over the out-of-range set T of prod_{d in T} e_d times the mixed
// backward difference at the clamped node) -- so differences of nearby
// positions take the base difference error-free.
// ===========================================================================
// The index part, the same for the three coordinates: the clamped node, the
// distance beyond it and the step inward per direction, and the periods
// crossed.
struct Pos3 {
  int cc[3], in[3], e[3], turns[3];
};
WIU_DEV Pos3 c3_pos(const Dims3& d, const int p_in[3]) {
  Pos3 r;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    int p = p_in[a];
    r.turns[a] = 0;
    if (d.bc[a] == WIU_BC_PERIODIC) {
      const int w = bc_index(p, d.n[a], 0), by = p - w;
      r.turns[a] = by == 0 ? 0 : (by == d.n[a] ? 1 : (by == -d.n[a] ? -1 : by / d.n[a]));
      p = w;
    }
    r.cc[a] = min(max(p, 0), d.n[a] - 1);
    r.e[a] = abs(p - r.cc[a]);
    r.in[a] = r.e[a] ? (p < 0 ? 1 : -1) : 0;
  }
  return r;
}

WIU_DEV void c3_at(const Dims3& d, const double* __restrict__ X, int c, const Pos3& r, double& base, double& off) {
  off = (c == 0 ? r.turns[0] * d.L[0] : (c == 1 ? r.turns[1] * d.L[1] : r.turns[2] * d.L[2]));
  const int* e = r.e;
  auto at = [&](int da, int db, int dc) {
    return X[((long long)(r.cc[2] + dc) * d.n[1] + (r.cc[1] + db)) * d.n[0] + (r.cc[0] + da)];
  };
  base = at(0, 0, 0);
  if (e[0] | e[1] | e[2]) {
    // mixed differences over the out-of-range directions
    double ext = 0.0;
    for (int t = 1; t < 8; ++t) {
      const int t0 = t & 1, t1 = (t >> 1) & 1, t2 = (t >> 2) & 1;
      if ((t0 && !e[0]) || (t1 && !e[1]) || (t2 && !e[2])) continue;
      double md = 0.0;
      for (int s = 0; s < 8; ++s) {
        if ((s & ~t) != 0) continue;  // s a subset of t
        const int s0 = s & 1, s1 = (s >> 1) & 1, s2 = (s >> 2) & 1;
        const double v = at(s0 * r.in[0], s1 * r.in[1], s2 * r.in[2]);
        md += ((s0 + s1 + s2) & 1) ? -v : v;
      }
      ext += (double)((t0 ? e[0] : 1) * (t1 ? e[1] : 1) * (t2 ? e[2] : 1)) * md;
    }
    off += ext;
  }
}

WIU_DEV double c3_diff(const Dims3& d, const double* X, int c, const int p1[3], const int p0[3]) {
  double b1, o1, b0, o0, s, e;
  c3_at(d, X, c, c3_pos(d, p1), b1, o1);
  c3_at(d, X, c, c3_pos(d, p0), b0, o0);
  two_sum(b1, -b0, s, e);
  return s + ((o1 - o0) + e);
}

struct Coord3 {
  const double* x[3];
};

// ===========================================================================
// Metrics: four kernels over boxes of nodes around the grid.
//   m3_ext_kernel    the extended coordinates, each once, as hi + lo
//   m3_inner_kernel  the nine inner derivatives D_a x_c
//   m3_nodal_kernel  the nine nodal metrics (Eq. 2.4) and J^{-1} (Eq. 2.5)
//   m3_band_kernel   the stored planes and their midpoint interpolation
// K is the reach of the scheme's central operator (3 .. 7).  Along a bounded
// direction the nodal box is the band B the interpolation needs, along a
// periodic one the grid alone (the band kernel wraps its reads, so band
// copies are the nodal values); the inner box is K wider, the coordinates K
// wider again.  The boundary rule is thus applied once per position, and the
// stencils behind it are plain accesses at constant strides.  150 x 131 x 117
// periodic, WENOIU5-2MP: 641 us (traced: ext 42, inner 176, nodal 241, band 199),
// bound by the L2 traffic of the stencils and, in the nodal kernel, by LDS
// reads and issue alike; 4818 us (inner 643, nodal 3961, band 214) when every
// tap applied the rule to both of its ends.  The same nodes with bounded ends, whose
// boxes hold as many positions beyond the grid as in it: 1011 us (76, 300, 467, 191).
// Coordinates relative to a tile's first node, one word each, took 895 there and 640
// on the periodic grid, but left metrics off by up to 1.6e-14 of their value where
// the spacing is small against the tile's extent (now 8e-16).
// Scratch arrays are stored row by row, the components of a row next to each
// other ([k][j][component][i]): a stencil tap then touches one stretch of
// memory for all its components instead of one page for each.
// ===========================================================================
struct Box3 {
  int h[3];         // halo beyond the grid, per direction
  int w[3];         // widths n + 2 h
  int off, pitch;   // slot of i = 0 in a row and slots of a row, multiples of 16 (whole cache lines)
  long long P;      // slots: pitch w[1] w[2]
};

// Offset of node (i, j, k) in an array of nc components, and its strides
// along i, j and k (components are one pitch apart).
WIU_DEV long long b3idx(const Box3& b, int nc, int i, int j, int k) {
  return ((long long)(k + b.h[2]) * b.w[1] + (j + b.h[1])) * nc * b.pitch + (i + b.off);
}
WIU_DEV void b3strides(const Box3& b, int nc, long long st[3]) {
  st[0] = 1;
  st[1] = (long long)nc * b.pitch;
  st[2] = st[1] * b.w[1];
}

// The node of a thread.  A block is 256 consecutive nodes of a plane (i, then
// j); `grp` consecutive blocks (about B3_ROWS rows) form a slab whose planes
// follow each other, in XCD-aware order.  The blocks an XCD works on at a time
// then span a few rows of many planes, so that the stencils along j and k
// find their operands in its L2.
constexpr int B3_ROWS = 16;
WIU_DEV bool b3_node(const Box3& b, int& i, int& j, int& k) {
  const int plane = b.w[0] * b.w[1], per = (plane + 255) >> 8;
  const int grp = min(per, max(1, (B3_ROWS * b.w[0]) >> 8));
  const int lid = xcd_remap(blockIdx.x, gridDim.x);
  const int slab = lid / (grp * b.w[2]);
  const int rest = lid - slab * grp * b.w[2];
  const int g = min(grp, per - slab * grp);  // the last slab may hold fewer blocks
  const int z = rest / g;
  const int r = (slab * grp + rest - z * g) * 256 + threadIdx.x;
  if (r >= plane) return false;
  const int y = r / b.w[0];
  i = r - y * b.w[0] - b.h[0]; j = y - b.h[1]; k = z - b.h[2];
  return true;
}

// Tile of the derivative kernels: 16 x 8 x 4 nodes.
constexpr int T3_X = 16, T3_Y = 8, T3_Z = 4;

// Whether (i, j, k) is a node of the grid.
WIU_DEV bool inside3(const Dims3& d, int i, int j, int k) {
  return i >= 0 && i < d.n[0] && j >= 0 && j < d.n[1] && k >= 0 && k < d.n[2];
}

// Coordinates on the box, as the unevaluated sum hi + lo of node coordinate
// and offset (exact): components 0..2 hi, 3..5 lo.  A difference of two
// positions is (hi1 - hi0) + (lo1 - lo0), which keeps its digits across a
// seam and where the spacing is small against the coordinates of the nodes
// around.  The lo part of a node of the grid is zero, neither written nor read.
__global__ void __launch_bounds__(256) m3_ext_kernel(Dims3 d, Box3 bx, Coord3 X, double* __restrict__ XE) {
  int p[3];
  if (!b3_node(bx, p[0], p[1], p[2])) return;
  double* xe = XE + b3idx(bx, 6, p[0], p[1], p[2]);
  if (inside3(d, p[0], p[1], p[2])) {
    const long long o = u3idx(d, p[0], p[1], p[2]);
#pragma unroll
    for (int c = 0; c < 3; ++c) xe[c * bx.pitch] = X.x[c][o];
    return;
  }
  const Pos3 r = c3_pos(d, p);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    double b, f, hi, lo;
    c3_at(d, X.x[c], c, r, b, f);
    two_sum(b, f, hi, lo);
    xe[c * bx.pitch] = hi;
    xe[(3 + c) * bx.pitch] = lo;
  }
}

// Both derivative kernels work on tiles of 16 x 8 x 4 nodes, one per lane, and
// take one outer direction o at a time: the tile and K nodes beyond both of
// its faces across o (n_o + 2 K positions along o by the nodes across) are
// staged in LDS, each value once where the lanes' taps read it 2 K times.
// Sixteen nodes along i are one cache line of the aligned rows.
// 150 x 131 x 117, WENOIU5-2MP: taps read from global memory (216 loads a node
// in the nodal kernel, every one an L1 miss) took 550 + 210 us (nodal, inner),
// tiles of 8 x 8 x 8 on unaligned rows 349 + 248 us.
template <int O, int K> struct Stage3 {
  static constexpr int A = (O == 0 ? T3_X : (O == 1 ? T3_Y : T3_Z)) + 2 * K;  // positions along o
  static constexpr int C = O == 0 ? T3_Y * T3_Z : (O == 1 ? T3_X * T3_Z : T3_X * T3_Y);
  // slots from one position along o to the next: the 32 lanes of an LDS
  // access (sixteen along x by two along y) fall into different banks
  static constexpr int S = O == 0 ? C + 2 : (O == 1 ? C + 16 : C);
};
template <int K> constexpr int stage3_slots() {
  constexpr int a = Stage3<0, K>::A * Stage3<0, K>::S, b = Stage3<1, K>::A * Stage3<1, K>::S;
  constexpr int c = Stage3<2, K>::A * Stage3<2, K>::S;
  return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

struct Tile3 {
  int q[3];   // first node of the tile
  int e[3];   // end of the box
  int x, y, z;  // this lane's node in the tile
  bool in;    // every position the tile reads is a node of the grid
};

WIU_DEV Tile3 tile3(const Dims3& d, const Box3& b, int K) {
  const int n[3] = {T3_X, T3_Y, T3_Z};
  Tile3 t;
  int lid = xcd_remap(blockIdx.x, gridDim.x);
  t.in = true;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int nt = (b.w[a] + n[a] - 1) / n[a];
    t.q[a] = (lid % nt) * n[a] - b.h[a];
    lid /= nt;
    t.e[a] = d.n[a] + b.h[a];
    t.in = t.in && t.q[a] >= K && t.q[a] + n[a] + K <= d.n[a];
  }
  t.x = threadIdx.x & 15; t.y = (threadIdx.x >> 4) & 7; t.z = threadIdx.x >> 7;
  return t;
}

// Staged position e of direction O: its slot and node (positions beyond the
// box's reach are clamped into it).
template <int O, int K> WIU_DEV int tile3_pos(const Tile3& t, int e, int p[3]) {
  using G = Stage3<O, K>;
  const int cross = O == 0 ? e / G::A : e % G::C, a = O == 0 ? e % G::A : e / G::C;
  p[0] = O == 0 ? a - K : cross & 15;
  p[1] = O == 0 ? cross & 7 : (O == 1 ? a - K : cross >> 4);
  p[2] = O == 0 ? cross >> 3 : (O == 1 ? cross >> 4 : a - K);
#pragma unroll
  for (int q = 0; q < 3; ++q) p[q] = min(t.q[q] + p[q], t.e[q] - 1 + (q == O ? K : 0));
  return a * G::S + cross;
}

// This lane's slot (its node) in direction O.
template <int O, int K> WIU_DEV int tile3_slot(const Tile3& t) {
  constexpr int S = Stage3<O, K>::S;
  return O == 0 ? (t.x + K) * S + t.y + 8 * t.z : (O == 1 ? (t.y + K) * S + t.x + 16 * t.z : (t.z + K) * S + t.x + 16 * t.y);
}

// What a lane stages for one direction, held in registers between its loads
// (all issued together, before the work on the direction before) and its
// LDS stores: the hi parts of the coordinates and, with G, three of the inner
// derivatives.
template <int O, int K, bool X, bool G> struct Lane3 {
  static constexpr int N = (Stage3<O, K>::A * Stage3<O, K>::C + 511) / 512;
  double x[N][3], g[N][3];
  WIU_DEV void load(const Tile3& t, const Box3& bx, const double* __restrict__ XE, const Box3& bi,
                    const double* __restrict__ Dx, int inner) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      int p[3];
      tile3_pos<O, K>(t, min((int)threadIdx.x + 512 * n, Stage3<O, K>::A * Stage3<O, K>::C - 1), p);
      if constexpr (X) {
        const double* v = XE + b3idx(bx, 6, p[0], p[1], p[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) x[n][c] = v[c * bx.pitch];
      }
      if constexpr (G) {
        const double* v = Dx + b3idx(bi, 9, p[0], p[1], p[2]);
#pragma unroll
        for (int c = 0; c < 3; ++c) g[n][c] = v[(3 * inner + c) * bi.pitch];
      }
    }
  }
  WIU_DEV void store(const Tile3& t, double* L) const {
    constexpr int NP = stage3_slots<K>();
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int e = threadIdx.x + 512 * n;
      if (e >= Stage3<O, K>::A * Stage3<O, K>::C) break;
      int p[3];
      const int slot = tile3_pos<O, K>(t, e, p);
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if constexpr (X) L[c * NP + slot] = x[n][c];
        if constexpr (G) L[(3 + c) * NP + slot] = g[n][c];
      }
    }
  }
};

// The lo parts of the positions m along O from this lane's node (a lane beyond the
// box takes the box's last).  They are zero but beyond the grid, where they are
// read from memory: few waves of the tiles at its ends do, and staging them too
// would take half as much LDS again.
template <int O> struct Lo3 {
  int a, n, pitch;
  bool out;  // the whole line lies beyond the grid
  long long st;
  const double* p;
  WIU_DEV Lo3(const Dims3& d, const Tile3& t, const Box3& bx, const double* __restrict__ XE) : out(false) {
    const int q[3] = {min(t.q[0] + t.x, t.e[0] - 1), min(t.q[1] + t.y, t.e[1] - 1), min(t.q[2] + t.z, t.e[2] - 1)};
    long long s3[3];
    b3strides(bx, 6, s3);
    a = q[O]; n = d.n[O]; pitch = bx.pitch; st = s3[O];
    p = XE + b3idx(bx, 6, q[0], q[1], q[2]) + 3 * pitch;
#pragma unroll
    for (int c = 0; c < 3; ++c) out = out || (c != O && (q[c] < 0 || q[c] >= d.n[c]));
  }
  // whether any of the positions 0 .. K (sd 0) or -K .. 0 (sd 1) lies beyond the grid
  WIU_DEV bool beyond(int sd, int K) const { return out || a < (sd ? K : 0) || a + (sd ? 0 : K) >= n; }
  WIU_DEV void at(int m, double v[3]) const {
    const bool o = out || a + m < 0 || a + m >= n;
#pragma unroll
    for (int c = 0; c < 3; ++c) v[c] = o ? p[m * st + c * pitch] : 0.0;
  }
};

// Derivatives along O of the three coordinates, whose hi parts are staged, added to s.
template <int O, int K> WIU_DEV void inner3_dir(const Tile3& t, const MetricStencil& ms, const double* L, double s[3]) {
  constexpr int NP = stage3_slots<K>(), S = Stage3<O, K>::S;
  const double* v = L + tile3_slot<O, K>(t);
#pragma unroll 1
  for (int m = 1; m <= K; ++m)
#pragma unroll
    for (int c = 0; c < 3; ++c) s[c] += ms.d[m - 1] * (v[c * NP + m * S] - v[c * NP - m * S]);
}
// Those of the lo parts, in s (as differences from the node's: zero on a line where
// they are all the same).
template <int O, int K>
WIU_DEV void inner3_lo(const Dims3& d, const Tile3& t, const Box3& bx, const double* __restrict__ XE,
                       const MetricStencil& ms, double s[3]) {
#pragma unroll
  for (int c = 0; c < 3; ++c) s[c] = 0.0;
  if (t.in) return;
  const Lo3<O> lo(d, t, bx, XE);
  if (!lo.beyond(0, K) && !lo.beyond(1, K)) return;
  double own[3];
  lo.at(0, own);
#pragma unroll
  for (int sd = 0; sd < 2; ++sd) {
    if (!lo.beyond(sd, K)) continue;
    double v[K][3];
#pragma unroll
    for (int m = 1; m <= K; ++m) lo.at(sd ? -m : m, v[m - 1]);
#pragma unroll
    for (int m = 1; m <= K; ++m)
#pragma unroll
      for (int c = 0; c < 3; ++c) s[c] = fma(sd ? -ms.d[m - 1] : ms.d[m - 1], v[m - 1][c] - own[c], s[c]);
  }
}

// Inner derivatives D_a x_c (a, c = 0..2) on their box: component 3a + c.
template <int K>
__global__ void __launch_bounds__(512) m3_inner_kernel(Dims3 d, MetricStencil ms, Box3 bi, Box3 bx,
                                                       const double* __restrict__ XE, double* __restrict__ Dx) {
  __shared__ double L[3 * stage3_slots<K>()];
  const Tile3 t = tile3(d, bi, K);
  double s[9];
  Lane3<0, K, true, false> l0;
  Lane3<1, K, true, false> l1;
  Lane3<2, K, true, false> l2;
  inner3_lo<0, K>(d, t, bx, XE, ms, s);
  inner3_lo<1, K>(d, t, bx, XE, ms, s + 3);
  inner3_lo<2, K>(d, t, bx, XE, ms, s + 6);
  l0.load(t, bx, XE, bi, Dx, 0);
  l0.store(t, L);
  __syncthreads();
  l1.load(t, bx, XE, bi, Dx, 0);
  inner3_dir<0, K>(t, ms, L, s);
  __syncthreads();
  l1.store(t, L);
  __syncthreads();
  l2.load(t, bx, XE, bi, Dx, 0);
  inner3_dir<1, K>(t, ms, L, s + 3);
  __syncthreads();
  l2.store(t, L);
  __syncthreads();
  inner3_dir<2, K>(t, ms, L, s + 6);
  const int i = t.q[0] + t.x, j = t.q[1] + t.y, k = t.q[2] + t.z;
  if (i >= t.e[0] || j >= t.e[1] || k >= t.e[2]) return;
  double* g = Dx + b3idx(bi, 9, i, j, k);
#pragma unroll
  for (int q = 0; q < 9; ++q) g[q * bi.pitch] = s[q];
}

// Outer direction O of the nodal metrics: D_O(r x g_i) of the staged inner
// direction i, added to n^_{O+2} (i = O+1) or taken from n^_{O+1} (i = O+2).
template <int O, int K, int H> WIU_DEV void nodal3_add(const double r[3], const double* u, double nh[9]) {
  constexpr int NP = stage3_slots<K>(), to = (O + 2 - H) % 3;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const int p = (l + 1) % 3, q = (l + 2) % 3;
    nh[3 * to + l] = fma(r[p], u[(3 + q) * NP], nh[3 * to + l]);
    nh[3 * to + l] = fma(-r[q], u[(3 + p) * NP], nh[3 * to + l]);
  }
}
template <int O, int K, int H>
WIU_DEV void nodal3_dir(const Tile3& t, const MetricStencil& ms, const double* L, double nh[9]) {
  constexpr int NP = stage3_slots<K>(), S = Stage3<O, K>::S;
  const double* v = L + tile3_slot<O, K>(t);
  const double x0[3] = {v[0], v[NP], v[2 * NP]};
#pragma unroll 1
  for (int m = 1; m <= K; ++m)
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      const double w = (sd != H) ? -ms.d[m - 1] : ms.d[m - 1];
      const double* u = v + (sd ? -m : m) * S;
      double r[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) r[c] = w * (u[c * NP] - x0[c]);
      nodal3_add<O, K, H>(r, u, nh);
    }
}
// What the lo parts of the coordinates add to it: those of a lane's taps in
// registers, where both inner directions of O use them.
template <int O, int K> struct Taps3 {
  double own[3], lo[2][K][3];  // of the node; of the positions m (0) and -m (1)
  bool far[2];
  WIU_DEV Taps3(const Dims3& d, const Tile3& t, const Box3& bx, const double* __restrict__ XE) {
    far[0] = far[1] = false;
    if (t.in) return;
    const Lo3<O> l(d, t, bx, XE);
    far[0] = l.beyond(0, K);
    far[1] = l.beyond(1, K);
    if (far[0] || far[1]) l.at(0, own);
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      if (!far[sd]) continue;
#pragma unroll
      for (int m = 1; m <= K; ++m) l.at(sd ? -m : m, lo[sd][m - 1]);
    }
  }
};
template <int O, int K, int H>
WIU_DEV void nodal3_lo(const Tile3& t, const MetricStencil& ms, const double* L, const Taps3<O, K>& x, double nh[9]) {
  const double* v = L + tile3_slot<O, K>(t);
#pragma unroll
  for (int sd = 0; sd < 2; ++sd) {
    if (!x.far[sd]) continue;
#pragma unroll
    for (int m = 1; m <= K; ++m) {
      const double w = (sd != H) ? -ms.d[m - 1] : ms.d[m - 1];
      double r[3];
#pragma unroll
      for (int c = 0; c < 3; ++c) r[c] = w * (x.lo[sd][m - 1][c] - x.own[c]);
      nodal3_add<O, K, H>(r, v + (sd ? -m : m) * Stage3<O, K>::S, nh);
    }
  }
}

// Nodal metrics (Eq. 2.4) and J^{-1} (Eq. 2.5) on their box, ten components.
// With r = x - x(node) and g_i = D_i x, Eq. 2.4 is for direction m and the next
// two directions a, b cyclically
//   n^_m = 1/2 [D_a(r x g_b) - D_b(r x g_a)].
template <int K>
__global__ void __launch_bounds__(512) m3_nodal_kernel(Dims3 d, MetricStencil ms, Box3 bt, Box3 bi, Box3 bx,
                                                       const double* __restrict__ XE, const double* __restrict__ Dx,
                                                       double* __restrict__ T) {
  __shared__ double L[6 * stage3_slots<K>()];
  const Tile3 t = tile3(d, bt, K);
  double nh[9];
#pragma unroll
  for (int q = 0; q < 9; ++q) nh[q] = 0.0;
  // per outer direction the coordinates and g_{O+1}, then g_{O+2} in the
  // place of g_{O+1}
  Lane3<0, K, true, true> a0;
  Lane3<0, K, false, true> b0;
  Lane3<1, K, true, true> a1;
  Lane3<1, K, false, true> b1;
  Lane3<2, K, true, true> a2;
  Lane3<2, K, false, true> b2;
  a0.load(t, bx, XE, bi, Dx, 1);
  a0.store(t, L);
  __syncthreads();
  {
    b0.load(t, bx, XE, bi, Dx, 2);
    nodal3_dir<0, K, 0>(t, ms, L, nh);
    const Taps3<0, K> lo(d, t, bx, XE);
    nodal3_lo<0, K, 0>(t, ms, L, lo, nh);
    __syncthreads();
    b0.store(t, L);
    __syncthreads();
    nodal3_lo<0, K, 1>(t, ms, L, lo, nh);
  }
  a1.load(t, bx, XE, bi, Dx, 2);
  nodal3_dir<0, K, 1>(t, ms, L, nh);
  __syncthreads();
  a1.store(t, L);
  __syncthreads();
  {
    b1.load(t, bx, XE, bi, Dx, 0);
    nodal3_dir<1, K, 0>(t, ms, L, nh);
    const Taps3<1, K> lo(d, t, bx, XE);
    nodal3_lo<1, K, 0>(t, ms, L, lo, nh);
    __syncthreads();
    b1.store(t, L);
    __syncthreads();
    nodal3_lo<1, K, 1>(t, ms, L, lo, nh);
  }
  a2.load(t, bx, XE, bi, Dx, 0);
  nodal3_dir<1, K, 1>(t, ms, L, nh);
  __syncthreads();
  a2.store(t, L);
  __syncthreads();
  {
    b2.load(t, bx, XE, bi, Dx, 1);
    nodal3_dir<2, K, 0>(t, ms, L, nh);
    const Taps3<2, K> lo(d, t, bx, XE);
    nodal3_lo<2, K, 0>(t, ms, L, lo, nh);
    __syncthreads();
    b2.store(t, L);
    __syncthreads();
    nodal3_lo<2, K, 1>(t, ms, L, lo, nh);
  }
  nodal3_dir<2, K, 1>(t, ms, L, nh);
  const int i = t.q[0] + t.x, j = t.q[1] + t.y, k = t.q[2] + t.z;
  if (i >= t.e[0] || j >= t.e[1] || k >= t.e[2]) return;
  const double* g = Dx + b3idx(bi, 9, i, j, k);
  double* tv = T + b3idx(bt, 10, i, j, k);
  double J = 0.0;
#pragma unroll
  for (int q = 0; q < 9; ++q) {
    nh[q] *= 0.5;
    J += nh[q] * g[q * bi.pitch];
    tv[q * bt.pitch] = nh[q];
  }
  tv[9 * bt.pitch] = J * (1.0 / 3.0);
}

// Stored metrics: nodal planes and midpoint interpolation in each metric's
// own direction, ghost band included, plus the tag.  jform 6 replaces
// J^{-1} by Eq. 2.6, 1/3 sum_{m,l} D_m(n^_{m,l} x_l) with x_l relative to
// the (wrapped) node, which needs the nodal band B >= GHOST + METRIC_REACH.
template <bool J6>
__global__ void __launch_bounds__(256) m3_band_kernel(Dims3 d, int scheme, Box3 bt, const double* __restrict__ T,
                                                      double* __restrict__ M, int* __restrict__ status,
                                                      MetricStencil ms, Coord3 X, double ah) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    double* tag = M + NP3 * d.mplane;
    tag[0] = TAG_MAGIC3; tag[1] = (double)scheme; tag[2] = (double)d.n[0]; tag[3] = (double)d.n[1];
    tag[4] = (double)d.n[2]; tag[5] = (double)(d.bc[0] + 2 * d.bc[1] + 4 * d.bc[2]); tag[6] = ah;
    tag[7] = J6 ? 6.0 : 5.0;
  }
  Box3 bm;
  for (int a = 0; a < 3; ++a) { bm.h[a] = GHOST; bm.w[a] = d.n[a] + 2 * GHOST; }
  int p[3];
  if (!b3_node(bm, p[0], p[1], p[2])) return;
  const long long t = m3idx(d, p[0], p[1], p[2]);
  // offset of position q along direction a in the nodal box
  const int W = bt.pitch;
  long long st[3];
  b3strides(bt, 10, st);
  auto at = [&](int a, int q) {
    return st[a] * (d.bc[a] == WIU_BC_PERIODIC ? bc_index(q, d.n[a], 0) : q + (a == 0 ? bt.off : bt.h[a]));
  };
  const long long o3[3] = {at(0, p[0]), at(1, p[1]), at(2, p[2])};
  const double* v0 = T + (o3[0] + o3[1] + o3[2]);
#pragma unroll
  for (int q = 0; q < 10; ++q) M[q * d.mplane + t] = v0[q * W];
  if constexpr (J6) {
    int w[3] = {p[0], p[1], p[2]};
    for (int a = 0; a < 3; ++a)
      if (d.bc[a] == WIU_BC_PERIODIC) w[a] = bc_index(w[a], d.n[a], 0);
    double J = 0.0;
    for (int m = 0; m < 3; ++m)
      for (int l = 0; l < 3; ++l)
        for (int k = 1; k <= METRIC_REACH; ++k) {
          const double ck = ms.d[k - 1];
          if (ck == 0.0) continue;
          int p1[3] = {w[0], w[1], w[2]}, p0[3] = {w[0], w[1], w[2]};
          p1[m] += k;
          p0[m] -= k;
          const double* v = v0 + ((3 * m + l) * W - o3[m]);
          J += ck * (v[at(m, p1[m])] * c3_diff(d, X.x[l], l, p1, w) - v[at(m, p0[m])] * c3_diff(d, X.x[l], l, p0, w));
        }
    M[9 * d.mplane + t] = J * (1.0 / 3.0);
  }
  const bool eight = scheme >= 4;
#pragma unroll
  for (int m = 0; m < 3; ++m) {
    long long q[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) q[s] = at(m, p[m] + (eight || (s > 0 && s < 7) ? s - 3 : 0)) - o3[m];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const double* v = v0 + (3 * m + l) * W;
      M[(10 + 3 * m + l) * d.mplane + t] =
          eight ? (-5.0 * (v[q[0]] + v[q[7]]) + 49.0 * (v[q[1]] + v[q[6]]) - 245.0 * (v[q[2]] + v[q[5]]) +
                   1225.0 * (v[q[3]] + v[q[4]])) * (1.0 / 2048.0)
                : (3.0 * v[q[1]] - 25.0 * v[q[2]] + 150.0 * v[q[3]] + 150.0 * v[q[4]] - 25.0 * v[q[5]] +
                   3.0 * v[q[6]]) * (1.0 / 256.0);
    }
  }
  if (inside3(d, p[0], p[1], p[2])) {
    const double j = J6 ? M[9 * d.mplane + t] : v0[9 * W];
    if (!(j > 0.0) || !(j < 1.0e300)) atomicOr(status, ST_JACOBIAN);
  }
}

// ===========================================================================
// Physics in three dimensions (Sec. 2.1; Sec. 3.4 eigenvectors).
// ===========================================================================
WIU_DEV void flux3(const double Q[5], const double k[3], double gam, double E[5]) {
  const double ri = rcp(Q[0]);
  const double u = Q[1] * ri, v = Q[2] * ri, w = Q[3] * ri;
  const double p = (gam - 1.0) * (Q[4] - 0.5 * (Q[1] * u + Q[2] * v + Q[3] * w));
  const double U = k[0] * u + k[1] * v + k[2] * w;
  E[0] = Q[0] * U;
  E[1] = Q[1] * U + k[0] * p;
  E[2] = Q[2] * U + k[1] * p;
  E[3] = Q[3] * U + k[2] * p;
  E[4] = (Q[4] + p) * U;
}

// Lax-Friedrichs half flux (E^ + sl Q)/2, as half_flux in two dimensions.
WIU_DEV void half_flux3(const double Q[5], const double k[3], double sl, double gam, double F[5]) {
  const double h[3] = {0.5 * k[0], 0.5 * k[1], 0.5 * k[2]}, hs = 0.5 * sl;
  const double ri = rcp(Q[0]);
  const double u = Q[1] * ri, v = Q[2] * ri, w = Q[3] * ri;
  const double p = (gam - 1.0) * (Q[4] - 0.5 * (Q[1] * u + Q[2] * v + Q[3] * w));
  const double U = h[0] * u + h[1] * v + h[2] * w;
  F[0] = Q[0] * U + hs * Q[0];
  for (int a = 0; a < 3; ++a) F[1 + a] = Q[1 + a] * U + h[a] * p + hs * Q[1 + a];
  F[4] = (Q[4] + p) * U + hs * Q[4];
}

// |k . u| + c |k| without contraction (every kernel rounds it alike).
WIU_DEV double speed3(const double Q[5], const double k[3], double gam, bool& bad) {
#pragma clang fp contract(off)
  const double ri = rcp(Q[0]);
  const double u = Q[1] * ri, v = Q[2] * ri, w = Q[3] * ri;
  const double p = (gam - 1.0) * (Q[4] - 0.5 * (Q[1] * u + Q[2] * v + Q[3] * w));
  const double c2 = gam * p * ri;
  bad = !(Q[0] > 0.0) || !(p > 0.0);
  const double s = fabs(k[0] * u + k[1] * v + k[2] * w) + sqrt(c2 * (k[0] * k[0] + k[1] * k[1] + k[2] * k[2]));
  bad = bad || !(s < 1.0e300);
  return s;
}

// Tangent basis of the unit direction n: t1 the axis of the smallest
// component of n (ties to the later axis) made orthogonal to n, t2 = t1 x n.
// SEL: that component by selects, where the compiler leaves n[e] in scratch memory
// (the options' kernels: 3-1MP with WENO-Z weights on 130 x 131 x 132 nodes 1933 us a
// step with the scratch, 1789 so; in the others they cost a spill).
template <bool SEL> WIU_DEV void tangents3(const double n[3], double t1[3], double t2[3]) {
  int e = 2;
  if (fabs(n[1]) < fabs(n[e])) e = 1;
  if (fabs(n[0]) < fabs(n[e])) e = 0;
  const double an = !SEL ? n[e] : (e == 0 ? n[0] : (e == 1 ? n[1] : n[2]));
  for (int c = 0; c < 3; ++c) t1[c] = (c == e ? 1.0 : 0.0) - an * n[c];
  const double r = rsqrt_(t1[0] * t1[0] + t1[1] * t1[1] + t1[2] * t1[2]);
  for (int c = 0; c < 3; ++c) t1[c] *= r;
  t2[0] = t1[1] * n[2] - t1[2] * n[1];
  t2[1] = t1[2] * n[0] - t1[0] * n[2];
  t2[2] = t1[0] * n[1] - t1[1] * n[0];
}

// Another split of the midpoint flux at the interpolated state Q with the
// midpoint metric k (Sec. 7; the 3-D forms of the 2-D ones).
//   split 1, Steger-Warming: F+- = R diag(l+-) L Q along n = k/|k| at Q, with
//     l = |k| (q_n - c, q_n, q_n, q_n, q_n + c), l+- = (l +- |l|)/2; the
//     shear rows of L annihilate Q, so only the acoustic and entropy fields
//     contribute;
//   split 2, van Leer: the Mach-number split along n.
WIU_DEV void mid_split_alt3(int split, const double Q[5], const double k[3], int side, double gam, double G[5]) {
  const double kn = sqrt(k[0] * k[0] + k[1] * k[1] + k[2] * k[2]);
  const double rkn = rcp(kn);
  const double n[3] = {k[0] * rkn, k[1] * rkn, k[2] * rkn};
  const double ri = rcp(Q[0]);
  const double V[3] = {Q[1] * ri, Q[2] * ri, Q[3] * ri};
  const double q2 = V[0] * V[0] + V[1] * V[1] + V[2] * V[2];
  const double p = (gam - 1.0) * (Q[4] - 0.5 * Q[0] * q2);
  const double c2 = gam * p * ri;
  const double rc = rsqrt_(c2);
  const double c = c2 * rc;
  const double qn = V[0] * n[0] + V[1] * n[1] + V[2] * n[2];
  if (split == 1) {
    const double H = (Q[4] + p) * ri;
    const double b1 = (gam - 1.0) * (rc * rc);
    const double b2 = 0.5 * b1 * q2;
    const double A = b2 * Q[0] - b1 * (V[0] * Q[1] + V[1] * Q[2] + V[2] * Q[3] - Q[4]);
    const double Bn = rc * (qn * Q[0] - (n[0] * Q[1] + n[1] * Q[2] + n[2] * Q[3]));
    const double l0 = kn * (qn - c), l1 = kn * qn, l4 = kn * (qn + c);
    auto part = [&](double l) { return side == 0 ? 0.5 * (l + fabs(l)) : 0.5 * (l - fabs(l)); };
    const double w0 = part(l0) * 0.5 * (A + Bn), w1 = part(l1) * (Q[0] - A), w4 = part(l4) * 0.5 * (A - Bn);
    G[0] = w0 + w1 + w4;
    for (int a = 0; a < 3; ++a) G[1 + a] = (w0 + w1 + w4) * V[a] + c * n[a] * (w4 - w0);
    G[4] = H * (w0 + w4) + c * qn * (w4 - w0) + 0.5 * q2 * w1;
    return;
  }
  const double M = qn * rc;
  if ((side == 0 && 1.0 <= M) || (side == 1 && M <= -1.0)) {
    flux3(Q, k, gam, G);
    return;
  }
  if ((side == 0 && M <= -1.0) || (side == 1 && 1.0 <= M)) {
    for (int a = 0; a < 5; ++a) G[a] = 0.0;
    return;
  }
  const double sg = side == 0 ? 1.0 : -1.0;
  const double fm = sg * kn * Q[0] * c * (M + sg) * (M + sg) * 0.25;
  const double vt = -qn + sg * 2.0 * c;
  const double e2 = (gam - 1.0) * qn + sg * 2.0 * c;
  G[0] = fm;
  for (int a = 0; a < 3; ++a) G[1 + a] = fm * (V[a] + n[a] * vt / gam);
  G[4] = fm * (e2 * e2 / (2.0 * (gam * gam - 1.0)) + 0.5 * (q2 - qn * qn));
}

// One side of the midpoint k+1/2 (side 0: F+, reference Q_k; side 1: F-,
// reference Q_{k+1}): project the stencil's deviations from the reference
// on the characteristic fields (rows of L for q_n - c, q_n, shear t2, shear
// t1, q_n + c), interpolate each with WENO, map back with R, add the
// reference, then the Lax-Friedrichs half flux with the midpoint metric.
// q(s, c): state at window slot s = 0..7 (nodes k-3 .. k+4).
// With split != 0, Dacc accumulates the other split's difference G - F.
template <int R, bool ZOK = false, class QF>
WIU_DEV void side_flux3(QF q, int side, const double n[3], const double mk[3], double lam, double gam, double eps,
                        int ppm, double F[5], int split = 0, double* Dacc = nullptr) {
  double Qr[5];
  for (int c = 0; c < 5; ++c) Qr[c] = q(3 + side, c);
  double t1[3], t2[3];
  tangents3<ZOK>(n, t1, t2);
  const double gm1 = gam - 1.0;
  const double rr = rcp(Qr[0]);
  const double V[3] = {Qr[1] * rr, Qr[2] * rr, Qr[3] * rr};
  const double hq = 0.5 * (V[0] * V[0] + V[1] * V[1] + V[2] * V[2]);
  const double p = gm1 * (Qr[4] - Qr[0] * hq);
  const double c2 = gam * p * rr;
  const double rc = rsqrt_(c2);
  const double c = c2 * rc;
  const double H = (Qr[4] + p) * rr;
  const double qn = V[0] * n[0] + V[1] * n[1] + V[2] * n[2];
  const double qa = V[0] * t2[0] + V[1] * t2[1] + V[2] * t2[2];
  const double qb = V[0] * t1[0] + V[1] * t1[1] + V[2] * t1[2];
  // halves, as in the 2-D side flux: A and B below are halved too
  const double b1 = 0.5 * gm1 * (rc * rc), b2 = b1 * hq, hrc = 0.5 * rc;
  // window slots of the stencil in interpolation order (left-biased for side
  // 0, mirrored for side 1); the reference slot has zero deviation
  // r = 2: k-2 .. k+1, r = 3: k-2 .. k+2, r = 4: k-3 .. k+3 (for side 0)
  constexpr int NS = R == 2 ? 4 : (R == 3 ? 5 : 7);
  constexpr int C0 = R == 4 ? 3 : 2;     // index of the reference in that order
  double w[5][NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    if (s == C0) {
      for (int f = 0; f < 5; ++f) w[f][s] = 0.0;
      continue;
    }
    const int slot = side == 0 ? 3 - C0 + s : 4 + C0 - s;
    double dq[5];
    for (int cc = 0; cc < 5; ++cc) dq[cc] = q(slot, cc) - Qr[cc];
    const double dmV = V[0] * dq[1] + V[1] * dq[2] + V[2] * dq[3];
    const double A = b2 * dq[0] - b1 * (dmV - dq[4]);
    const double Bn = hrc * (qn * dq[0] - (n[0] * dq[1] + n[1] * dq[2] + n[2] * dq[3]));
    w[0][s] = A + Bn;
    w[1][s] = fma(-2.0, A, dq[0]);
    w[2][s] = t2[0] * dq[1] + t2[1] * dq[2] + t2[2] * dq[3] - qa * dq[0];
    w[3][s] = t1[0] * dq[1] + t1[1] * dq[2] + t1[2] * dq[3] - qb * dq[0];
    w[4][s] = A - Bn;
  }
  double Wf[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    if constexpr (R == 2) Wf[f] = weno3<ZOK>(w[f][0], w[f][1], w[f][3], eps, ppm);
    else if constexpr (R == 3) Wf[f] = weno5<ZOK>(w[f][0], w[f][1], w[f][3], w[f][4], eps, ppm);
    else Wf[f] = weno7<ZOK>(w[f][0], w[f][1], w[f][2], w[f][4], w[f][5], w[f][6], eps, ppm);
  }
  // Q = Q_ref + R W (W undoing its scale)
  constexpr double ws = 1.0 / WSCALE<R>;
  const double s04 = Wf[0] + Wf[4], cd = c * (Wf[4] - Wf[0]);
  const double sum = s04 + Wf[1];
  double r[5];
  r[0] = fma(ws, sum, Qr[0]);
  for (int a = 0; a < 3; ++a) r[1 + a] = fma(ws, V[a] * sum + n[a] * cd + t2[a] * Wf[2] + t1[a] * Wf[3], Qr[1 + a]);
  r[4] = fma(ws, H * s04 + qn * cd + hq * Wf[1] + qa * Wf[2] + qb * Wf[3], Qr[4]);
  half_flux3(r, mk, side == 0 ? lam : -lam, gam, F);
  if (split != 0) {
    double G[5];
    mid_split_alt3(split, r, mk, side, gam, G);
    for (int a = 0; a < 5; ++a) Dacc[a] += G[a] - F[a];
  }
}

// The same side flux with the interpolation component by component
// (Sec. 2.4): vars 1 conservative, vars 2 primitive (rho, u, v, w, p), on
// deviations from the reference node's values.
template <int R, bool ZOK, class QF>
WIU_DEV void side_flux3_comp(QF q, int side, int vars, const double mk[3], double lam, double gam, double eps,
                             int ppm, double F[5], int split = 0, double* Dacc = nullptr) {
  constexpr int NS = R == 2 ? 4 : (R == 3 ? 5 : 7);
  constexpr int C0 = R == 4 ? 3 : 2;
  auto val = [&](int slot, double V[5]) {
    for (int c = 0; c < 5; ++c) V[c] = q(slot, c);
    if (vars == 2) {
      const double ri = rcp(V[0]);
      const double u = V[1] * ri, v = V[2] * ri, w = V[3] * ri;
      V[4] = (gam - 1.0) * (V[4] - 0.5 * (V[1] * u + V[2] * v + V[3] * w));
      V[1] = u; V[2] = v; V[3] = w;
    }
  };
  double Vr[5];
  val(3 + side, Vr);
  double w[5][NS];
#pragma unroll
  for (int s_ = 0; s_ < NS; ++s_) {
    if (s_ == C0) {
      for (int f = 0; f < 5; ++f) w[f][s_] = 0.0;
      continue;
    }
    const int slot = side == 0 ? 3 - C0 + s_ : 4 + C0 - s_;
    double V[5];
    val(slot, V);
    for (int f = 0; f < 5; ++f) w[f][s_] = V[f] - Vr[f];
  }
  double Vm[5];
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    double W;
    if constexpr (R == 2) W = weno3<ZOK>(w[f][0], w[f][1], w[f][3], eps, ppm);
    else if constexpr (R == 3) W = weno5<ZOK>(w[f][0], w[f][1], w[f][3], w[f][4], eps, ppm);
    else W = weno7<ZOK>(w[f][0], w[f][1], w[f][2], w[f][4], w[f][5], w[f][6], eps, ppm);
    Vm[f] = fma(1.0 / WSCALE<R>, W, Vr[f]);
  }
  double r[5];
  if (vars == 2) {
    r[0] = Vm[0];
    for (int a = 0; a < 3; ++a) r[1 + a] = Vm[0] * Vm[1 + a];
    r[4] = Vm[4] / (gam - 1.0) + 0.5 * Vm[0] * (Vm[1] * Vm[1] + Vm[2] * Vm[2] + Vm[3] * Vm[3]);
  } else {
    for (int a = 0; a < 5; ++a) r[a] = Vm[a];
  }
  half_flux3(r, mk, side == 0 ? lam : -lam, gam, F);
  if (split != 0) {
    double G[5];
    mid_split_alt3(split, r, mk, side, gam, G);
    for (int a = 0; a < 5; ++a) Dacc[a] += G[a] - F[a];
  }
}

// ===========================================================================
// Direction passes.
// ===========================================================================
struct S3Args {
  Dims3 d;
  const double* U;                 // state the fluxes are built from
  const double* M;
  const unsigned long long* lam;   // line maxima: xi lines [ny nz], eta [nx nz], zeta [nx ny]
  unsigned long long* nlam;        // xi pass of an RK stage: the next stage's maxima (or null)
  unsigned long long* ncfl;        // with nlam, when set: the next state's CFL maximum per j [ny]
  double gamma, alpha, eps;
  int ppm;
  int vars;                        // WIU_VARS_* (interpolation variables)
  double ah;                       // free parameter of the one-midpoint schemes
  int weights;                     // WIU_WEIGHTS_*
  int split;                       // WIU_SPLIT_* of the leading midpoint flux
  double* Racc;                    // accumulated flux differences [5][np]
  double* Reta;                    // those of the eta pass when it runs beside the zeta pass (or null)
  double* out;                     // dU/dt (mode 2) or the new stage state (mode 3)
  const double* U0;                // RK base state
  const double* dt;                // device time step
  double ca, cb;
  int* status;
  // rules beyond the sides of non-periodic directions (x lo .. z hi):
  // WIU_SIDE_TRANSMISSIVE, _WALL or _FIXED with the state `fixed`
  int side[6];
  double fixed[6][5];
};

WIU_DEV long long lam_off(const Dims3& d, int D) {
  return D == 0 ? 0 : (D == 1 ? (long long)d.n[1] * d.n[2] : (long long)d.n[1] * d.n[2] + (long long)d.n[0] * d.n[2]);
}
WIU_DEV long long line3(const Dims3& d, int D, const int p[3]) {
  return D == 0 ? (long long)p[2] * d.n[1] + p[1] : (D == 1 ? (long long)p[2] * d.n[0] + p[0]
                                                             : (long long)p[1] * d.n[0] + p[0]);
}

WIU_DEV bool tag3_ok(const Dims3& d, const double* M, int scheme, double ah) {
  const double* tag = M + NP3 * d.mplane;
  return tag[0] == TAG_MAGIC3 && tag[1] == (double)scheme && tag[2] == (double)d.n[0] &&
         tag[3] == (double)d.n[1] && tag[4] == (double)d.n[2] &&
         tag[5] == (double)(d.bc[0] + 2 * d.bc[1] + 4 * d.bc[2]) && tag[6] == ah;
}

// LDS of a 3-D sweep tile: NA items along the line by NB lines.  Per item
// the nodal flux E^ and both midpoint side fluxes (15 values; f+- are rebuilt
// from E^ and the staged state); the states of items k - QL .. k + QL + 1.
// Lanes of a wave touch consecutive words: line-major for xi tiles (lanes
// along the line), position-major otherwise (lanes across lines along i).
template <int SC, int DIR, int NA, int NB, bool OPT = false> struct Sweep3Lds {
  static constexpr int QL = Range<SC>::QL;
  static constexpr int NQ = NA + 2 * QL + 1;
  // with the options, 5 more per item: D, the difference another midpoint
  // split makes to H at the item's midpoint
  static constexpr int NREC = OPT ? 20 : 15;
  double sh[NREC][NA * NB];
  double sq[5][NB * NQ];
  double red[DIR == 0 ? NA * NB : 1];  // xi tiles: the next stage's eta speeds, reduced over the lines
  static WIU_DEV int si(int tb, int ta) { return DIR == 0 ? tb * NA + ta : ta * NB + tb; }
  static WIU_DEV int qi(int tb, int pos) { return DIR == 0 ? tb * NQ + pos : pos * NB + tb; }
};

// One direction pass.  A workgroup owns NB lines (consecutive j for xi,
// consecutive i otherwise, at one value of the remaining index) and a
// segment of OUT = NA - EXTRA output nodes along them: it stages the states
// of the segment (boundary rule applied) in LDS, computes one item per lane
// (nodal flux at k and both side fluxes at k + 1/2), then the first OUT
// lanes of each line form H_{i+1/2} - H_{i-1/2} and, by `mode`: 0 Racc = R;
// 1 Racc += R; 2 dU/dt = -(Racc + R)/J^{-1}; 3 the RK stage
// U_out = ca U0 + cb (U + dt dU/dt); the xi pass adds Reta to Racc when that is set.
// Four block-wide barriers on every path (five in an xi pass that accumulates the next
// stage's maxima).
// OPT: compiled with the scheme options (a.vars, a.ah, a.weights); without
// it the sweep runs the paper's configuration and carries no code for them, and
// PPM says whether the weights are mapped.
template <int SC, int DIR, int NA, int NB, bool OPT, bool PPM>
WIU_DEV void s3_sweep(const S3Args& a, int mode, long long tile, Sweep3Lds<SC, DIR, NA, NB, OPT>& L) {
  using R_ = Range<SC>;
  using LT = Sweep3Lds<SC, DIR, NA, NB, OPT>;
  constexpr int OUT = NA - R_::EXTRA, QL = R_::QL, NQ = LT::NQ, NT = NA * NB;
  const Dims3& d = a.d;
  const double ah = OPT ? a.ah : 1.0;
  const int ppm = OPT ? (a.weights != 0 ? 2 : a.ppm) : PPM;  // 2: WENO-Z weights
  const int split = OPT ? a.split : 0;                 // another split of the leading midpoint flux
  if (!tag3_ok(d, a.M, SC, ah)) {  // block-uniform
    if (threadIdx.x == 0 && threadIdx.y == 0) atomicOr(a.status, ST_SCHEME);
    return;
  }
  const int n = d.n[DIR];
  const int nac = DIR == 0 ? d.n[1] : d.n[0];   // grouped index across the lines
  const int nseg = (n + OUT - 1) / OUT, ngrp = (nac + NB - 1) / NB;
  // XCD-aware order: consecutive logical tiles share an XCD's L2; for eta
  // and zeta the line group (along i) varies fastest, so neighbouring tiles
  // read the same rows and pages of the k-planes
  int seg, grp, cb;
  if (DIR == 0) {
    seg = (int)(tile % nseg);
    const long long rest = tile / nseg;
    grp = (int)(rest % ngrp); cb = (int)(rest / ngrp);
  } else {
    grp = (int)(tile % ngrp);
    const long long rest = tile / ngrp;
    seg = (int)(rest % nseg); cb = (int)(rest / nseg);
  }
  const int ta = DIR == 0 ? threadIdx.x : threadIdx.y;           // along
  const int tb = DIR == 0 ? threadIdx.y : threadIdx.x;           // across
  const int la = grp * NB + tb;
  const bool live = la < nac;
  const int o0 = seg * OUT;
  const int out = min(OUT, n - o0);
  const int k = o0 + R_::LO + ta;
  auto node = [&](int kk, int line, int p[3]) {
    if (DIR == 0) { p[0] = kk; p[1] = line; p[2] = cb; }
    else if (DIR == 1) { p[0] = line; p[1] = kk; p[2] = cb; }
    else { p[0] = line; p[1] = cb; p[2] = kk; }
  };
  // stage the states of the segment: each thread's elements (NIT at most)
  // are all loaded before any is stored, so their latencies overlap; a
  // segment whose window lies inside the line needs no index mapping
  {
    const int tid = threadIdx.x + blockDim.x * threadIdx.y;
    const int k0 = o0 + R_::LO - QL;
    const bool inside = k0 >= 0 && k0 + NQ <= n;  // uniform over the block
    constexpr int NIT = (NQ * NB + NT - 1) / NT;
    double Qs[NIT][5];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = tid + it * NT;
      if (e >= NQ * NB) break;
      const int pos = DIR == 0 ? e % NQ : e / NB;
      const int lb = DIR == 0 ? e / NQ : e % NB;
      const int ln = grp * NB + lb;
      double* Qv = Qs[it];
      if (ln >= nac) continue;
      if (inside) {
        int p[3];
        node(k0 + pos, ln, p);
        const long long o = u3idx(d, p[0], p[1], p[2]);
#pragma unroll
        for (int c = 0; c < 5; ++c) Qv[c] = a.U[c * d.np + o];
      } else {
        // beyond a non-periodic end the side's rule: transmissive (boundary
        // node), reflecting wall (mirror node, momentum along the boundary
        // node's unit metric direction reversed) or a fixed state
        const int kr = k0 + pos;
        const bool out_of = d.bc[DIR] != WIU_BC_PERIODIC && (kr < 0 || kr >= n);
        const int sd = 2 * DIR + (kr < 0 ? 0 : 1);
        const int rule = out_of ? a.side[sd] : WIU_SIDE_TRANSMISSIVE;
        if (rule == WIU_SIDE_FIXED) {
#pragma unroll
          for (int c = 0; c < 5; ++c) Qv[c] = a.fixed[sd][c];
        } else {
          const int kb = kr < 0 ? 0 : n - 1;
          const int kk = rule == WIU_SIDE_WALL ? min(max(2 * kb - kr, 0), n - 1) : bc_index(kr, n, d.bc[DIR]);
          int p[3];
          node(kk, ln, p);
          const long long o = u3idx(d, p[0], p[1], p[2]);
#pragma unroll
          for (int c = 0; c < 5; ++c) Qv[c] = a.U[c * d.np + o];
          if (rule == WIU_SIDE_WALL) {
            node(kb, ln, p);
            const long long mo = m3idx(d, p[0], p[1], p[2]);
            double nv[3];
            for (int c = 0; c < 3; ++c) nv[c] = a.M[(3 * DIR + c) * d.mplane + mo];
            const double rn = rsqrt_(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
            const double mn = (Qv[1] * nv[0] + Qv[2] * nv[1] + Qv[3] * nv[2]) * rn;
            for (int c = 0; c < 3; ++c) Qv[1 + c] -= 2.0 * mn * (nv[c] * rn);
          }
        }
      }
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int e = tid + it * NT;
      if (e >= NQ * NB) break;
      const int pos = DIR == 0 ? e % NQ : e / NB;
      const int lb = DIR == 0 ? e / NQ : e % NB;
      if (grp * NB + lb >= nac) continue;
#pragma unroll
      for (int c = 0; c < 5; ++c) L.sq[c][LT::qi(lb, pos)] = Qs[it][c];
    }
  }
  __syncthreads();
  double lam = 0.0;
  if (live) {
    int p[3];
    node(0, la, p);
    lam = a.alpha * __longlong_as_double((long long)a.lam[lam_off(d, DIR) + line3(d, DIR, p)]);
  }
  const double gam = a.gamma;
  const int slot = LT::si(tb, ta);
  const bool need_node = live && k >= o0 + Traits<SC>::NLO && k < o0 + out + Traits<SC>::NHI;
  const bool need_mid = live && k >= o0 + Traits<SC>::MLO && k < o0 + out + Traits<SC>::MHI;
  auto kn = [&](int kk, double v[3]) {
    int p[3];
    node(kk, la, p);
    const long long o = m3idx(d, p[0], p[1], p[2]);
    for (int c = 0; c < 3; ++c) v[c] = a.M[(3 * DIR + c) * d.mplane + o];
  };
  if (need_node) {
    double Q[5], k0v[3], E[5];
    for (int c = 0; c < 5; ++c) Q[c] = L.sq[c][LT::qi(tb, ta + QL)];
    kn(k, k0v);
    flux3(Q, k0v, gam, E);
    for (int c = 0; c < 5; ++c) L.sh[c][slot] = E[c];
  }
  if (need_mid) {
    double k0v[3], k1v[3], mk[3], nv[3];
    kn(k, k0v);
    kn(k + 1, k1v);
    int p[3];
    node(k, la, p);
    const long long o = m3idx(d, p[0], p[1], p[2]);
    for (int c = 0; c < 3; ++c) {
      mk[c] = a.M[(10 + 3 * DIR + c) * d.mplane + o];
      nv[c] = 0.5 * (k0v[c] + k1v[c]);
    }
    const double rn = rsqrt_(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
    for (int c = 0; c < 3; ++c) nv[c] *= rn;
    // window slot s = 0..7 is node k - 3 + s
    auto q = [&](int s_, int c) { return L.sq[c][LT::qi(tb, ta + QL - 3 + s_)]; };
    double D[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      asm volatile("" ::: "memory");  // one side at a time (register pressure)
      double F[5];
      if (OPT && a.vars != 0)
        side_flux3_comp<Traits<SC>::R, OPT>(q, side, a.vars, mk, lam, gam, a.eps, ppm, F, split, D);
      else
        side_flux3<Traits<SC>::R, OPT>(q, side, nv, mk, lam, gam, a.eps, ppm, F, split, D);
      for (int c = 0; c < 5; ++c) L.sh[5 + 5 * side + c][slot] = F[c];
    }
    if constexpr (OPT) {
      for (int c = 0; c < 5; ++c) L.sh[LT::NREC - 5 + c][slot] = D[c];
    }
  }
  // epilogue operands of this lane's output node, issued before the
  // barriers so that their latency overlaps them and the flux difference
  const bool act = live && ta < out;
  const int i = o0 + ta;
  double xr[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, x0[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, jv = 1.0;
  long long t = 0;
  if (act) {
    int p[3];
    node(i, la, p);
    t = u3idx(d, p[0], p[1], p[2]);
    if (mode != 0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) xr[c] = a.Racc[c * d.np + t];
      if (DIR == 0 && a.Reta) {
#pragma unroll
        for (int c = 0; c < 5; ++c) xr[c] += a.Reta[c * d.np + t];
      }
    }
    if (mode >= 2) jv = a.M[9 * d.mplane + m3idx(d, p[0], p[1], p[2])];
    if (mode == 3 && a.ca != 0.0) {
#pragma unroll
      for (int c = 0; c < 5; ++c) x0[c] = a.U0[c * d.np + t];
    }
  }
  // nodal metrics of all three directions, for the next stage's maxima
  double km[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) km[c] = 0.0;
  const bool fused = DIR == 0 && mode == 3 && a.nlam != nullptr;  // uniform over the grid
  if (fused && act) {
    int p[3];
    node(i, la, p);
    const long long mo = m3idx(d, p[0], p[1], p[2]);
#pragma unroll
    for (int c = 0; c < 9; ++c) km[c] = a.M[c * d.mplane + mo];
  }
  __syncthreads();
  constexpr int S = DIR == 0 ? 1 : NB;
  // H_{k+1/2} once per item, for the midpoints k + 1/2 of k in [o0 - 1,
  // o0 + out), into the item's nodal-flux slots once every record is read;
  // each midpoint's H is then read by both of its nodes (exact telescoping)
  {
    const bool hact = live && k >= o0 - 1 && k < o0 + out;
    double Hk[5];
    if (hact) {
      const int qs = LT::qi(tb, ta + QL);
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        const double* e = &L.sh[c][slot];
        const double* qv = &L.sq[c][qs];
        const double* gp = &L.sh[5 + c][slot];
        const double* gm = &L.sh[10 + c][slot];
        if constexpr (SC == 3) {
          Hk[c] = hsum52(lam, [&](int m) { return e[m * S]; }, [&](int m) { return qv[m * S]; },
                         [&](int m) { return gp[m * S]; }, [&](int m) { return gm[m * S]; });
        } else {
          auto fp = [&](int kk) { return 0.5 * (e[(kk - k) * S] + lam * qv[(kk - k) * S]); };
          auto fm = [&](int kk) { return 0.5 * (e[(kk - k) * S] - lam * qv[(kk - k) * S]); };
          auto Fp = [&](int kk) { return gp[(kk - k) * S]; };
          auto Fm = [&](int kk) { return gm[(kk - k) * S]; };
          Hk[c] = hflux<SC>(k, ah, fp, fm, Fp, Fm);
        }
        if constexpr (OPT) {
          if (split != 0) Hk[c] += L.sh[LT::NREC - 5 + c][slot];
        }
      }
    }
    __syncthreads();
    if (hact) {
#pragma unroll
      for (int c = 0; c < 5; ++c) L.sh[c][slot] = Hk[c];
    }
    __syncthreads();
  }
  if constexpr (DIR == 0) {
    if (fused) {
      // RK stage with the next stage's line maxima (Sec. 2.3), every lane
      // taking part in the reductions: a wave is one line (j, k) along i, the
      // tile's NB lines are consecutive j at one k.  Wave speeds as in the
      // separate maxima pass (same routine, clamped at zero), so the maxima
      // are bit-identical to it.
      static_assert(NA == 64, "xi tile: one line per wave");
      double sx = 0.0, se = 0.0, sz = 0.0;
      bool bad = false;
      if (act) {
        const int hs = LT::si(tb, i - (o0 + R_::LO));
        const double rj = -rcp(jv);
        const double dt = a.dt[0];
        const int pq = LT::qi(tb, ta - R_::LO + QL);
        double Qn[5];
#pragma unroll
        for (int c = 0; c < 5; ++c) {
          const double Lv = (xr[c] + (L.sh[c][hs] - L.sh[c][hs - S])) * rj;
          const double us = L.sq[c][pq] + dt * Lv;
          Qn[c] = a.ca == 0.0 ? a.cb * us : a.ca * x0[c] + a.cb * us;
          a.out[c * d.np + t] = Qn[c];
        }
        double sp[3];
#pragma unroll
        for (int D = 0; D < 3; ++D) {
          const double kk[3] = {km[3 * D], km[3 * D + 1], km[3 * D + 2]};
          bool b;
          sp[D] = speed3(Qn, kk, a.gamma, b);
          bad |= b;
        }
        sx = fmax(0.0, sp[0]);
        se = fmax(0.0, sp[1]);
        sz = fmax(0.0, sp[2]);
      }
      if (bad) atomicOr(a.status, ST_NONPHYS);
      unsigned long long* lx = a.nlam;
      unsigned long long* le = lx + (long long)d.n[1] * d.n[2];
      unsigned long long* lz = le + (long long)d.n[0] * d.n[2];
      if (a.ncfl) {
        // CFL maximum, formed as the separate maxima pass forms it, in
        // partial maxima per j: the tiles of one k plane run together, so
        // their atomics spread over ny addresses
        double cf = act ? (sx + se + sz) / jv : 0.0;
        for (int off = 32; off > 0; off >>= 1) cf = fmax(cf, __shfl_xor(cf, off, 64));
        if (ta == 0 && live) atomicMax(&a.ncfl[la], (unsigned long long)__double_as_longlong(cf));
      }
      // xi lines (j, k): reduce over the wave (along i)
      for (int off = 32; off > 0; off >>= 1) sx = fmax(sx, __shfl_xor(sx, off, 64));
      if (ta == 0 && live) atomicMax(&lx[(long long)cb * d.n[1] + la], (unsigned long long)__double_as_longlong(sx));
      // zeta lines (i, j): one node of the tile each
      if (act) atomicMax(&lz[(long long)la * d.n[0] + i], (unsigned long long)__double_as_longlong(sz));
      // eta lines (i, k): reduce over the tile's lines
      L.red[LT::si(tb, ta)] = se;
      __syncthreads();
      if (tb == 0 && ta < out) {
        double m = L.red[LT::si(0, ta)];
#pragma unroll
        for (int l = 1; l < NB; ++l) m = fmax(m, L.red[LT::si(l, ta)]);
        atomicMax(&le[(long long)cb * d.n[0] + i], (unsigned long long)__double_as_longlong(m));
      }
      return;
    }
  }
  if (!act) return;
  const int hs = LT::si(tb, i - (o0 + R_::LO));
  double Rv[5];
#pragma unroll
  for (int c = 0; c < 5; ++c) Rv[c] = L.sh[c][hs] - L.sh[c][hs - S];
  if (mode == 0) {
    for (int c = 0; c < 5; ++c) a.Racc[c * d.np + t] = Rv[c];
    return;
  }
  if (mode == 1) {
    for (int c = 0; c < 5; ++c) a.Racc[c * d.np + t] = xr[c] + Rv[c];
    return;
  }
  const double rj = -rcp(jv);
  if (mode == 2) {
    for (int c = 0; c < 5; ++c) a.out[c * d.np + t] = (xr[c] + Rv[c]) * rj;
    return;
  }
  // the stage state at the output node is the staged tile entry (an interior
  // node, untouched by the side rules); U0 is not read when its coefficient
  // is zero (first stage)
  const double dt = a.dt[0];
  const int pq = LT::qi(tb, ta - R_::LO + QL);
  for (int c = 0; c < 5; ++c) {
    const double Lv = (xr[c] + Rv[c]) * rj;
    const double us = L.sq[c][pq] + dt * Lv;
    a.out[c * d.np + t] = a.ca == 0.0 ? a.cb * us : a.ca * x0[c] + a.cb * us;
  }
}

template <int SC, int DIR, int NA, int NB, bool OPT, bool PPM>
__global__ void __launch_bounds__(NA * NB, NA == 30 ? 4 : 1) s3_sweep_kernel(S3Args a, int mode) {
  __shared__ Sweep3Lds<SC, DIR, NA, NB, OPT> L;
  s3_sweep<SC, DIR, NA, NB, OPT, PPM>(a, mode, xcd_remap(blockIdx.x, gridDim.x), L);
}

// The zeta pass (the first tz tiles, into Racc) and the eta pass (into Reta) side by
// side, both with mode 0.
template <int SC, bool OPT, bool PPM>
__global__ void __launch_bounds__(256) s3_pair_kernel(S3Args a, int tz) {
  union Lds {
    Sweep3Lds<SC, 1, 32, 8, OPT> e;
    Sweep3Lds<SC, 2, 32, 8, OPT> z;
  };
  __shared__ Lds L;
  const int b = blockIdx.x;
  if (b < tz) {
    s3_sweep<SC, 2, 32, 8, OPT, PPM>(a, 0, xcd_remap(b, tz), L.z);
  } else {
    a.Racc = a.Reta;
    s3_sweep<SC, 1, 32, 8, OPT, PPM>(a, 0, xcd_remap(b - tz, gridDim.x - tz), L.e);
  }
}

// Line maxima of the wave speeds in all three directions and the CFL
// maximum.  One thread per (i, j) column walks a chunk of kc <= KC3 nodes along k
// (the third grid dimension covers the chunks): zeta lines reduce in
// registers over the chunk, xi lines across the wave (threads along i), eta
// lines by atomics.
constexpr int KC3 = 16;
__global__ void __launch_bounds__(256) w3_max_kernel(Dims3 d, int kc, const double* __restrict__ U,
                                                     const double* __restrict__ M, double gam,
                                                     unsigned long long* __restrict__ lam, int* __restrict__ status) {
  const int i = blockIdx.x * 64 + (threadIdx.x & 63);
  const int j = blockIdx.y * 4 + (threadIdx.x >> 6);
  const bool act = i < d.n[0] && j < d.n[1];
  unsigned long long* lx = lam;
  unsigned long long* le = lam + (long long)d.n[1] * d.n[2];
  unsigned long long* lz = le + (long long)d.n[0] * d.n[2];
  unsigned long long* cflm = lz + (long long)d.n[0] * d.n[1];
  double smz = 0.0, cm = 0.0;
  bool bad = false;
  const int k0 = blockIdx.z * kc, k1 = min(k0 + kc, d.n[2]);  // uniform over the block
  for (int k = k0; k < k1; ++k) {
    double sx = 0.0;
    if (act) {
      const long long o = u3idx(d, i, j, k), mo = m3idx(d, i, j, k);
      double Q[5];
      for (int c = 0; c < 5; ++c) Q[c] = U[c * d.np + o];
      double s[3];
      for (int D = 0; D < 3; ++D) {
        const double kk[3] = {M[(3 * D) * d.mplane + mo], M[(3 * D + 1) * d.mplane + mo],
                              M[(3 * D + 2) * d.mplane + mo]};
        bool b;
        s[D] = speed3(Q, kk, gam, b);
        bad |= b;
      }
      sx = fmax(0.0, s[0]);
      atomicMax(&le[(long long)k * d.n[0] + i], (unsigned long long)__double_as_longlong(fmax(0.0, s[1])));
      smz = fmax(smz, s[2]);
      cm = fmax(cm, (sx + fmax(0.0, s[1]) + fmax(0.0, s[2])) / M[9 * d.mplane + mo]);
    }
    double v = sx;
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    if ((threadIdx.x & 63) == 0 && j < d.n[1])
      atomicMax(&lx[(long long)k * d.n[1] + j], (unsigned long long)__double_as_longlong(v));
  }
  if (act) atomicMax(&lz[(long long)j * d.n[0] + i], (unsigned long long)__double_as_longlong(smz));
  for (int off = 32; off > 0; off >>= 1) cm = fmax(cm, __shfl_xor(cm, off, 64));
  if ((threadIdx.x & 63) == 0) atomicMax(cflm, (unsigned long long)__double_as_longlong(cm));
  if (bad) atomicOr(status, ST_NONPHYS);
}

}  // namespace wiu

using namespace wiu;

namespace {

constexpr size_t A3 = 256;
size_t al3(size_t v) { return (v + A3 - 1) / A3 * A3; }

bool grid3_ok(const wiu_grid3* g) {
  if (!g) return false;
  const int n[3] = {g->nx, g->ny, g->nz};
  for (int a = 0; a < 3; ++a) {
    if (n[a] < 1 || g->bc[a] < 0 || g->bc[a] > 1) return false;
    if (g->bc[a] == WIU_BC_TRANSMISSIVE && n[a] < 2) return false;
    if (g->bc[a] == WIU_BC_PERIODIC && !(g->period[a] > 0.0 && g->period[a] < 1.0e300)) return false;
    if (n[a] > 4096) return false;
    if (g->bc[a] == WIU_BC_PERIODIC) continue;
    for (int e = 2 * a; e < 2 * a + 2; ++e) {
      if (g->side[e] < WIU_SIDE_TRANSMISSIVE || g->side[e] > WIU_SIDE_FIXED) return false;
      if (g->side[e] == WIU_SIDE_FIXED) {
        const double* q = g->fixed[e];
        if (!(q[0] > 0.0) || !(q[0] < 1.0e300)) return false;
        const double p = q[4] - 0.5 * (q[1] * q[1] + q[2] * q[2] + q[3] * q[3]) / q[0];  // (gamma - 1) p
        if (!(p > 0.0) || !(p < 1.0e300)) return false;
      }
    }
  }
  return (long long)n[0] * n[1] * n[2] <= (1LL << 31);
}

Dims3 dims3(const wiu_grid3* g) {
  Dims3 d;
  d.n[0] = g->nx; d.n[1] = g->ny; d.n[2] = g->nz;
  for (int a = 0; a < 3; ++a) { d.bc[a] = g->bc[a]; d.L[a] = g->period[a]; }
  d.np = (long long)g->nx * g->ny * g->nz;
  d.mp[0] = g->nx + 2 * GHOST; d.mp[1] = g->ny + 2 * GHOST;
  d.mplane = (long long)d.mp[0] * d.mp[1] * (g->nz + 2 * GHOST);
  return d;
}

// Workspace: [status | line maxima, a ring of four sets (one per state) | dt | big
// area], the big area holding either the metric scratch (inner derivatives, nodal band
// and, on small grids, the extended coordinates) or the stepping buffers (Racc, U1, U2
// and, below PAIR3_NODES, Reta).
struct Ws3 {
  size_t lam, dt, big, metric_dx, metric_t, metric_x, racc, u1, u2, reta, total;
  long long nlam, set;  // words of a maxima set in use, and from one set to the next
};

// A metric box: `band` beyond the grid along bounded directions, plus
// `reach` along every direction.
Box3 box3(const Dims3& d, int band, int reach) {
  Box3 b;
  for (int a = 0; a < 3; ++a) {
    b.h[a] = (d.bc[a] == WIU_BC_PERIODIC ? 0 : band) + reach;
    b.w[a] = d.n[a] + 2 * b.h[a];
  }
  b.off = (b.h[0] + 15) / 16 * 16;
  b.pitch = (b.off + d.n[0] + b.h[0] + 15) / 16 * 16;
  b.P = (long long)b.pitch * b.w[1] * b.w[2];
  return b;
}

// The extended coordinates (six planes) stay in the metric array M, which
// only the last metric kernel writes, unless the grid is so small that their
// halo exceeds it.
bool ext_in_metrics(const Dims3& d, const Box3& bx) { return 6 * bx.P <= NP3 * d.mplane; }

// Grids whose zeta and eta passes run side by side, the eta differences in an array of
// their own.  A pass of a small grid is as long as one wave's work, so one launch for
// two saves its whole time: steps of 5-2MP on 40 x 36 x 33 nodes 122.2 -> 97.2 us,
// 64^3 306.8 -> 289.9, 112^3 965 -> 945.  From 128^3 on (1543 and 1541, 160^3 2712 and
// 2704) the passes fill the chip by themselves, and the array would be the
// workspace's largest growth.
constexpr long long PAIR3_NODES = 1LL << 21;
bool pair3(const Dims3& d) { return d.np < PAIR3_NODES; }

Ws3 ws3(const wiu_grid3* g) {
  const Dims3 d = dims3(g);
  Ws3 w;
  w.nlam = (long long)g->ny * g->nz + (long long)g->nx * g->nz + (long long)g->nx * g->ny + 1;
  w.lam = A3;
  // a maxima set: the line maxima and the CFL maximum (nlam entries), then
  // the partial CFL maxima per j [ny] that several steps per call carry
  const size_t set = al3((w.nlam + g->ny) * 8);
  w.set = (long long)(set / 8);
  w.dt = w.lam + 4 * set;
  w.big = w.dt + A3;
  const int B = GHOST + METRIC_REACH;  // the widest band (Eq. 2.6) and operator
  const Box3 bx = box3(d, B, 2 * METRIC_REACH);
  w.metric_dx = w.big;
  w.metric_t = w.metric_dx + al3(9 * (size_t)box3(d, B, METRIC_REACH).P * 8);
  w.metric_x = w.metric_t + al3(10 * (size_t)box3(d, B, 0).P * 8);
  w.racc = w.big;
  w.u1 = w.racc + al3(5 * (size_t)d.np * 8);
  w.u2 = w.u1 + al3(5 * (size_t)d.np * 8);
  w.reta = w.u2 + al3(5 * (size_t)d.np * 8);
  const size_t step_end = w.reta + (pair3(d) ? al3(5 * (size_t)d.np * 8) : 0);
  const size_t met_end = w.metric_x + (ext_in_metrics(d, bx) ? 0 : al3(6 * (size_t)bx.P * 8));
  w.total = step_end > met_end ? step_end : met_end;
  return w;
}

bool alpha3_ok(int scheme, double a) {
  return a > 0.0 && a < 1.0e300 && (a == 1.0 || scheme == WIU_3_1MP || scheme == WIU_5_1MP || scheme == WIU_7_1MP);
}

bool params3_ok(const wiu_params* p, int scheme) {
  return p && p->gamma > 1.0 && p->alpha_lf > 0.0 && p->eps >= 0.0 && (p->ppm == 0 || p->ppm == 1) &&
         p->vars >= WIU_VARS_CHARACTERISTIC && p->vars <= WIU_VARS_PRIMITIVE && alpha3_ok(scheme, p->alpha_h) &&
         (p->weights == WIU_WEIGHTS_JS || p->weights == WIU_WEIGHTS_Z) && p->split >= WIU_SPLIT_LF &&
         p->split <= WIU_SPLIT_VL;
}

void options3(const wiu_params* p, S3Args& a) {
  a.vars = p->vars; a.ah = p->alpha_h; a.weights = p->weights; a.split = p->split;
}

void sides3(const wiu_grid3* g, S3Args& a) {
  for (int e = 0; e < 6; ++e) {
    a.side[e] = g->bc[e / 2] == WIU_BC_PERIODIC ? WIU_SIDE_TRANSMISSIVE : g->side[e];
    for (int c = 0; c < 5; ++c) a.fixed[e][c] = g->fixed[e][c];
  }
}

dim3 tile_grid(const Box3& b) {
  return dim3((unsigned)((b.w[0] + T3_X - 1) / T3_X) * ((b.w[1] + T3_Y - 1) / T3_Y) * ((b.w[2] + T3_Z - 1) / T3_Z));
}
dim3 box_grid(const Box3& b) { return dim3((unsigned)(((b.w[0] * b.w[1] + 255) / 256) * b.w[2])); }

// Tile shapes: xi 64 items x 4 lines (lanes along the line, one line per
// wave), eta and zeta 32 items x 8 lines (lanes across the lines, along i).
template <int SC, int DIR, int NA, int NB> unsigned tiles3(const Dims3& d) {
  constexpr int OUT = NA - Range<SC>::EXTRA;
  const int nac = DIR == 0 ? d.n[1] : d.n[0];
  const int nb = DIR == 2 ? d.n[1] : d.n[2];
  return (unsigned)((long long)((d.n[DIR] + OUT - 1) / OUT) * ((nac + NB - 1) / NB) * nb);
}

template <int SC, int DIR, int NA, int NB, bool OPT, bool PPM>
hipError_t launch_sweep3_t(const S3Args& a, int mode, hipStream_t st) {
  const unsigned tiles = tiles3<SC, DIR, NA, NB>(a.d);
  const dim3 block = DIR == 0 ? dim3(NA, NB) : dim3(NB, NA);
  void* h = prof_open(WIU_K_SWEEP3, st);
  hipLaunchKernelGGL((s3_sweep_kernel<SC, DIR, NA, NB, OPT, PPM>), dim3(tiles), block, 0, st, a, mode);
  prof_close(h);
  return hipGetLastError();
}

// An eta or zeta pass of its own.  Tiles of 30 x 8 items need 40.0 KB of LDS, so four
// workgroups share a CU where of 32 x 8 (42.6 KB) three do; they are taken where a line
// has no more segments for it.  Steps with 32 x 8 against 30 x 8: 5-2MP on 256^3 (10
// segments with either) 11.31 and 11.00-11.10 ms, 3-1MP on 200 x 200 x 180 4.39 and
// 4.15-4.17; with more segments 5-2MP on 160^3 (6 against 7) 2.77 and 2.82-2.87.  The
// seventh-order and options kernels hold more LDS or registers than that.
template <int SC, int DIR, bool OPT, bool PPM>
hipError_t launch_across3(const S3Args& a, int mode, hipStream_t st) {
  if constexpr (!OPT && Range<SC>::QL == 2) {
    auto segments = [&](int na) { const int out = na - Range<SC>::EXTRA; return (a.d.n[DIR] + out - 1) / out; };
    if (segments(30) == segments(32)) return launch_sweep3_t<SC, DIR, 30, 8, OPT, PPM>(a, mode, st);
  }
  return launch_sweep3_t<SC, DIR, 32, 8, OPT, PPM>(a, mode, st);
}

// The three passes: zeta, eta, then xi with mode `last`, which reads what they left.
template <int SC, bool OPT, bool PPM>
hipError_t launch_passes3_o(const S3Args& a, int last, hipStream_t st) {
  hipError_t e;
  if (a.Reta) {
    const unsigned tz = tiles3<SC, 2, 32, 8>(a.d), te = tiles3<SC, 1, 32, 8>(a.d);
    void* h = prof_open(WIU_K_SWEEP3, st);
    hipLaunchKernelGGL((s3_pair_kernel<SC, OPT, PPM>), dim3(tz + te), dim3(8, 32), 0, st, a, (int)tz);
    prof_close(h);
    e = hipGetLastError();
  } else {
    e = launch_across3<SC, 2, OPT, PPM>(a, 0, st);
    if (e == hipSuccess) e = launch_across3<SC, 1, OPT, PPM>(a, 1, st);
  }
  return e == hipSuccess ? launch_sweep3_t<SC, 0, 64, 4, OPT, PPM>(a, last, st) : e;
}

// the options kernels only when an option is in use
template <int SC>
hipError_t launch_passes3(const S3Args& a, int last, hipStream_t st) {
  if (a.vars != 0 || a.ah != 1.0 || a.weights != 0 || a.split != 0) return launch_passes3_o<SC, true, true>(a, last, st);
  return a.ppm ? launch_passes3_o<SC, false, true>(a, last, st) : launch_passes3_o<SC, false, false>(a, last, st);
}

hipError_t passes3(int scheme, const S3Args& a, int last, hipStream_t st) {
  switch (scheme) {
    case 0: return launch_passes3<0>(a, last, st);
    case 1: return launch_passes3<1>(a, last, st);
    case 2: return launch_passes3<2>(a, last, st);
    case 3: return launch_passes3<3>(a, last, st);
    case 4: return launch_passes3<4>(a, last, st);
    case 5: return launch_passes3<5>(a, last, st);
    case 6: return launch_passes3<6>(a, last, st);
    case 7: return launch_passes3<7>(a, last, st);
    default: return hipErrorInvalidValue;
  }
}

// Line maxima and the CFL maximum of U into a cleared set.  Each thread walks
// KC3 nodes along k, fewer while that leaves the chip without blocks; more blocks
// are more atomics on the same lines.  Steps with at least 64, 128, 256 and 1024
// blocks: 40 x 36 x 33 nodes 88.8, 90.5, 97.5 and 97.4 us, 64^3 259, 254, 257 and 290,
// 47 x 180 x 98 612, 614, 613 and 642.  On 40 x 36 x 33 nodes 27 blocks took 34 us for
// this pass alone.
hipError_t maxima3(const Dims3& d, const double* U, const double* M, double gam, unsigned long long* lam, int* status,
                   hipStream_t st) {
  const long long cols = (long long)((d.n[0] + 63) / 64) * ((d.n[1] + 3) / 4);
  int kc = KC3;
  while (kc > 1 && cols * ((d.n[2] + kc - 1) / kc) < 128) kc >>= 1;
  hipLaunchKernelGGL(w3_max_kernel, dim3((d.n[0] + 63) / 64, (d.n[1] + 3) / 4, (d.n[2] + kc - 1) / kc), dim3(256), 0,
                     st, d, kc, U, M, gam, lam, status);
  return hipGetLastError();
}

int rc3(hipError_t e) { return e == hipSuccess ? WIU_OK : WIU_EHIP; }

}  // namespace

// nsteps TVD-RK3 steps with cfl > 0, each at the CFL time step of its state,
// written to dt[step] before the stages read it, or one step of the device
// scalar *dt, only read.  Only the first step has a separate maxima pass: the
// xi pass of each stage accumulates the next stage's maxima (that of the last
// stage, for the next step, also the partial CFL maxima per j).
static int rk3_3d(const wiu_grid3* g, int scheme, const wiu_params* p, double* U, const double* M, double cfl, double* dt,
           void* ws, wiu_stream_t stream, int nsteps = 1) {
  if (!grid3_ok(g) || scheme < 0 || scheme > 7 || !params3_ok(p, scheme) || !U || !M || !dt || !ws || nsteps < 1 ||
      (nsteps > 1 && !(cfl > 0.0)))
    return WIU_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const Dims3 d = dims3(g);
  const Ws3 w = ws3(g);
  char* base = (char*)ws;
  double* U1 = (double*)(base + w.u1);
  double* U2 = (double*)(base + w.u2);
  S3Args a;
  a.nlam = nullptr;
  a.ncfl = nullptr;
  a.d = d; a.M = M; a.lam = (unsigned long long*)(base + w.lam);
  a.gamma = p->gamma; a.alpha = p->alpha_lf; a.eps = p->eps; a.ppm = p->ppm;
  a.Racc = (double*)(base + w.racc);
  a.Reta = pair3(d) ? (double*)(base + w.reta) : nullptr;
  a.U0 = U; a.status = (int*)base;
  sides3(g, a);
  options3(p, a);
  // U1 = U + dt L(U); U2 = 3/4 U + 1/4 (U1 + dt L(U1)); U = 1/3 U + 2/3 (U2 + dt L(U2))
  const double* src[3] = {U, U1, U2};
  double* dst[3] = {U1, U2, U};
  const double ca[3] = {0.0, 0.75, 1.0 / 3.0}, cb[3] = {1.0, 0.25, 2.0 / 3.0};
  // maxima sets in a ring of four, one per state: all cleared at first, the
  // three that a later step accumulates by the launch that forms its step
  // size; the first step's maxima come from a separate pass
  unsigned long long* sets = (unsigned long long*)(base + w.lam);
  int c = 0;
  auto set = [&](int k) { return sets + ((c + k) & 3) * w.set; };
  if (launch_fill_u64(sets, 4 * w.set, st) != hipSuccess) return WIU_EHIP;
  if (maxima3(d, U, M, p->gamma, sets, a.status, st) != hipSuccess) return WIU_EHIP;
  for (int step = 0; step < nsteps; ++step) {
    double* dts = cfl > 0.0 ? dt + step : dt;
    if (cfl > 0.0) {
      const hipError_t e = step == 0 ? launch_step_begin(set(0) + w.nlam - 1, 1, cfl, dts, nullptr, 0, 0, 0, st)
                                     : launch_step_begin(set(0) + w.nlam, d.n[1], cfl, dts, sets, w.set, 4, c, st);
      if (e != hipSuccess) return WIU_EHIP;
    }
    a.dt = dts;
    for (int s = 0; s < 3; ++s, c = (c + 1) & 3) {
      a.U = src[s]; a.out = dst[s]; a.ca = ca[s]; a.cb = cb[s];
      a.lam = set(0);  // the maxima of U, U1, U2
      unsigned long long* next = s < 2 || step + 1 < nsteps ? set(1) : nullptr;
      a.nlam = next;
      a.ncfl = s == 2 && next ? next + w.nlam : nullptr;
      if (passes3(scheme, a, 3, st) != hipSuccess) return WIU_EHIP;
    }
  }
  return WIU_OK;
}

extern "C" {

size_t wiu3_metrics_size(const wiu_grid3* g) {
  if (!grid3_ok(g)) return 0;
  return ((size_t)NP3 * dims3(g).mplane + 8) * sizeof(double);
}

size_t wiu3_workspace_bytes(const wiu_grid3* g) { return grid3_ok(g) ? ws3(g).total : 0; }

int wiu3_metrics(const wiu_grid3* g, int scheme, int jform, const wiu_params* p, const double* x, const double* y,
                 const double* z, double* M, void* ws, wiu_stream_t stream) {
  const double ah = p ? p->alpha_h : 1.0;
  if (!grid3_ok(g) || scheme < 0 || scheme > 7 || (jform != 5 && jform != 6) || !alpha3_ok(scheme, ah) || !x ||
      !y || !z || !M || !ws)
    return WIU_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const Dims3 d = dims3(g);
  const Ws3 w = ws3(g);
  char* base = (char*)ws;
  double* Dx = (double*)(base + w.metric_dx);
  double* T = (double*)(base + w.metric_t);
  int* status = (int*)base;
  const MetricStencil ms = metric_stencil(scheme, ah);
  int K = METRIC_REACH;
  while (K > 3 && ms.d[K - 1] == 0.0) --K;
  const int B = jform == 6 ? GHOST + METRIC_REACH : metric_band(scheme);
  const Box3 bt = box3(d, B, 0), bi = box3(d, B, K), bx = box3(d, B, 2 * K);
  double* XE = ext_in_metrics(d, bx) ? M : (double*)(base + w.metric_x);
  const Coord3 X{{x, y, z}};
  Box3 bm;
  for (int q = 0; q < 3; ++q) bm.w[q] = d.n[q] + 2 * GHOST;
  hipLaunchKernelGGL(m3_ext_kernel, box_grid(bx), dim3(256), 0, st, d, bx, X, XE);
#define WIU_M3(k)                                                                                      \
  case k:                                                                                              \
    hipLaunchKernelGGL(m3_inner_kernel<k>, tile_grid(bi), dim3(512), 0, st, d, ms, bi, bx, XE, Dx);    \
    hipLaunchKernelGGL(m3_nodal_kernel<k>, tile_grid(bt), dim3(512), 0, st, d, ms, bt, bi, bx, XE, Dx, T); \
    break;
  switch (K) { WIU_M3(3) WIU_M3(4) WIU_M3(5) WIU_M3(6) WIU_M3(7) }
#undef WIU_M3
  if (jform == 6)
    hipLaunchKernelGGL(m3_band_kernel<true>, box_grid(bm), dim3(256), 0, st, d, scheme, bt, T, M, status, ms, X, ah);
  else
    hipLaunchKernelGGL(m3_band_kernel<false>, box_grid(bm), dim3(256), 0, st, d, scheme, bt, T, M, status, ms, X, ah);
  return rc3(hipGetLastError());
}

int wiu3_rhs(const wiu_grid3* g, int scheme, const wiu_params* p, const double* U, const double* M, double* dUdt,
             void* ws, wiu_stream_t stream) {
  if (!grid3_ok(g) || scheme < 0 || scheme > 7 || !params3_ok(p, scheme) || !U || !M || !dUdt || !ws) return WIU_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const Dims3 d = dims3(g);
  const Ws3 w = ws3(g);
  char* base = (char*)ws;
  S3Args a;
  a.nlam = nullptr;
  a.ncfl = nullptr;
  a.d = d; a.U = U; a.M = M; a.lam = (unsigned long long*)(base + w.lam);
  a.gamma = p->gamma; a.alpha = p->alpha_lf; a.eps = p->eps; a.ppm = p->ppm;
  a.Racc = (double*)(base + w.racc);
  a.Reta = pair3(d) ? (double*)(base + w.reta) : nullptr; a.out = dUdt;
  sides3(g, a);
  options3(p, a);
  a.U0 = nullptr; a.dt = nullptr; a.ca = 0.0; a.cb = 1.0; a.status = (int*)base;
  if (launch_fill_u64((unsigned long long*)a.lam, w.nlam, st) != hipSuccess) return WIU_EHIP;
  if (maxima3(d, U, M, p->gamma, (unsigned long long*)a.lam, a.status, st) != hipSuccess) return WIU_EHIP;
  return rc3(passes3(scheme, a, 2, st));
}

int wiu3_cfl_dt(const wiu_grid3* g, const wiu_params* p, const double* U, const double* M, double cfl, double* dt,
                void* ws, wiu_stream_t stream) {
  if (!grid3_ok(g) || !p || !(p->gamma > 1.0) || !U || !M || !dt || !ws || !(cfl > 0.0)) return WIU_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  const Dims3 d = dims3(g);
  const Ws3 w = ws3(g);
  char* base = (char*)ws;
  unsigned long long* lam = (unsigned long long*)(base + w.lam);
  if (launch_fill_u64(lam, w.nlam, st) != hipSuccess) return WIU_EHIP;
  if (maxima3(d, U, M, p->gamma, lam, (int*)base, st) != hipSuccess) return WIU_EHIP;
  return rc3(launch_cfl_dt(lam + w.nlam - 1, cfl, dt, st));
}

int wiu3_rk3_step(const wiu_grid3* g, int scheme, const wiu_params* p, double* U, const double* M, const double* dt,
                  void* ws, wiu_stream_t stream) {
  return rk3_3d(g, scheme, p, U, M, 0.0, const_cast<double*>(dt), ws, stream);
}

int wiu3_rk3_step_cfl(const wiu_grid3* g, int scheme, const wiu_params* p, double* U, const double* M, double cfl,
                      double* dt, void* ws, wiu_stream_t stream) {
  if (!(cfl > 0.0)) return WIU_EINVAL;
  return rk3_3d(g, scheme, p, U, M, cfl, dt, ws, stream);
}

int wiu3_rk3_steps_cfl(const wiu_grid3* g, int scheme, const wiu_params* p, double* U, const double* M, double cfl,
                       int nsteps, double* dt, void* ws, wiu_stream_t stream) {
  if (!(cfl > 0.0) || nsteps < 1) return WIU_EINVAL;
  return rk3_3d(g, scheme, p, U, M, cfl, dt, ws, stream, nsteps);
}

}  // extern "C"
