// gfx950 kernels of the V-cycle on the split-colour layout (flat.hpp).
//
// Operator and rounding: c phi is accumulated with explicit fused multiply-adds
// in the order own pair, pair beside, ylo, yhi, zlo, zhi, a cell's update is (f +
// sum) times 1 / diag, and the compiler fuses nothing by itself (contract off),
// so every kernel that updates a cell - a half-sweep of its own, blocks of
// sweeps, the one-work-group tail - rounds the same way.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device.hpp"
#include "flat.hpp"

namespace amrmg {

namespace {

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

template <typename T, int V, bool NT>
__device__ __forceinline__ void ldv(T (&d)[V], const T* p) {
  if constexpr (V == 1) {
    d[0] = NT ? __builtin_nontemporal_load(p) : *p;
  } else {
    using X = T __attribute__((ext_vector_type(V)));
    const X* q = reinterpret_cast<const X*>(p);
    const X x = NT ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
    for (int v = 0; v < V; ++v) d[v] = x[v];
  }
}

// Stores the first `n` of V values (p aligned to V elements).
template <typename T, int V>
__device__ __forceinline__ void stv(T* p, const T (&s)[V], int n) {
  if constexpr (V > 1) {
    if (n >= V) {
      using X = T __attribute__((ext_vector_type(V)));
      X x;
#pragma unroll
      for (int v = 0; v < V; ++v) x[v] = s[v];
      *reinterpret_cast<X*>(p) = x;
      return;
    }
  }
#pragma unroll
  for (int v = 0; v < V; ++v)
    if (v < n) p[v] = s[v];
}

// Coefficients of V consecutive cells of a colour (pairs p0 .. p0 + V - 1 of
// row (j, k); sh = (j + k + colour) & 1, the cells' offset in their pairs).
// Along x a cell has a neighbour in its own pair (face 2p + 1, o) and one in the
// pair beside it (the pair before for sh = 0, after for sh = 1; s).
template <typename T, int V>
struct Coef {
  T o[V], s[V], yl[V], yh[V], zl[V], zh[V], a[V];
};

template <typename T, int V, bool NT>
__device__ __forceinline__ void load_coef(Coef<T, V>& c, const FlatOp<T>& op, int colour, int sh,
                                          int p0, int j, int k) {
  const FlatDims& d = op.d;
  const int r = p0 + d.sp * (j + d.ny * k);
  ldv<T, V, NT>(c.o, op.x + d.half + r);
  if (V == 1) {
    c.s[0] = op.x[r + sh];
  } else {
    T ev[V];
    ldv<T, V, NT>(ev, op.x + r);
    // the face past the last pair of the group, for cells on odd columns
    const T en = sh ? op.x[r + V] : ev[V - 1];
#pragma unroll
    for (int v = 0; v < V; ++v) c.s[v] = sh ? (v + 1 < V ? ev[v + 1 < V ? v + 1 : v] : en) : ev[v];
  }
  const int ry = p0 + d.sp * (j + (d.ny + 1) * k);
  ldv<T, V, NT>(c.yl, op.y + colour * d.yh + ry);
  ldv<T, V, NT>(c.yh, op.y + (1 - colour) * d.yh + ry + d.sp);
  ldv<T, V, NT>(c.zl, op.z + colour * d.zh + r);
  ldv<T, V, NT>(c.zh, op.z + (1 - colour) * d.zh + r + d.sp * d.ny);
  if (op.a) ldv<T, V, NT>(c.a, op.a + colour * d.half + r);
}

// The cells' neighbours, all of the other colour (O: its half).  Past a wall
// an in-range element is read and not used.
template <typename T, int V>
struct Nb {
  T o[V], s[V], yl[V], yh[V], zl[V], zh[V];
};

struct RowIx {
  int jm, jp, km, kp;  // neighbour rows and planes, wrapped or clamped
};

__device__ __forceinline__ RowIx row_ix(const FlatDims& d, int j, int k) {
  RowIx x;
  x.jm = j > 0 ? j - 1 : ((d.wall & 4) ? 0 : d.ny - 1);
  x.jp = j < d.ny - 1 ? j + 1 : ((d.wall & 8) ? j : 0);
  x.km = k > 0 ? k - 1 : ((d.wall & 16) ? 0 : d.nz - 1);
  x.kp = k < d.nz - 1 ? k + 1 : ((d.wall & 32) ? k : 0);
  return x;
}

template <typename T, int V>
__device__ __forceinline__ void load_nb(Nb<T, V>& n, const FlatDims& d, const T* O, int sh, int p0,
                                        int j, int k, const RowIx& x) {
  const int row = d.sp * (j + d.ny * k);
  ldv<T, V, false>(n.o, O + row + p0);
  const int pl = p0 > 0 ? p0 - 1 : ((d.wall & 1) ? 0 : d.np - 1);
  const int ph = p0 + V < d.np ? p0 + V : ((d.wall & 2) ? p0 : 0);
  const T ex = O[row + (sh ? ph : pl)];
#pragma unroll
  for (int v = 0; v < V; ++v)
    n.s[v] = sh ? (v + 1 < V ? n.o[v + 1 < V ? v + 1 : v] : ex) : (v > 0 ? n.o[v > 0 ? v - 1 : 0] : ex);
  ldv<T, V, false>(n.yl, O + p0 + d.sp * (x.jm + d.ny * k));
  ldv<T, V, false>(n.yh, O + p0 + d.sp * (x.jp + d.ny * k));
  ldv<T, V, false>(n.zl, O + p0 + d.sp * (j + d.ny * x.km));
  ldv<T, V, false>(n.zh, O + p0 + d.sp * (j + d.ny * x.kp));
}

// Coarse parents' corrections of the other-colour neighbours of the cells:
// own[v] the parent of pair p0 + v, x[v] that of the pair beside the cell, y and
// z those of the neighbour rows in the next coarse row and plane.
template <typename T, int V>
struct Par {
  T own[V], x[V], y[V], z[V];
};

template <typename T>
__device__ __forceinline__ T coarse_at(const FlatDims& c, const T* e, int I, int J, int K) {
  return e[((I + J + K) & 1) * c.half + (I >> 1) + c.sp * (J + c.ny * K)];
}

template <typename T, int V>
__device__ __forceinline__ void load_par(Par<T, V>& q, const FlatDims& d, const FlatDims& c,
                                         const T* e, int sh, int p0, int j, int k) {
  const int J = j >> 1, K = k >> 1;
  const int cnx = d.nx / 2, cny = d.ny / 2, cnz = d.nz / 2;
  // wrapped or clamped as the fine neighbours are (c may be padded)
  const int Jn = (j & 1) ? (J < cny - 1 ? J + 1 : ((d.wall & 8) ? J : 0))
                         : (J > 0 ? J - 1 : ((d.wall & 4) ? 0 : cny - 1));
  const int Kn = (k & 1) ? (K < cnz - 1 ? K + 1 : ((d.wall & 32) ? K : 0))
                         : (K > 0 ? K - 1 : ((d.wall & 16) ? 0 : cnz - 1));
#pragma unroll
  for (int v = 0; v < V; ++v) {
    const int I = p0 + v < cnx ? p0 + v : cnx - 1;
    const int In = sh ? (I < cnx - 1 ? I + 1 : ((d.wall & 2) ? I : 0))
                      : (I > 0 ? I - 1 : ((d.wall & 1) ? 0 : cnx - 1));
    q.own[v] = coarse_at(c, e, I, J, K);
    q.x[v] = coarse_at(c, e, In, J, K);
    q.y[v] = coarse_at(c, e, I, Jn, K);
    q.z[v] = coarse_at(c, e, I, J, Kn);
  }
}

template <typename T, int V>
__device__ __forceinline__ void add_par(Nb<T, V>& n, const Par<T, V>& q, int j, int k) {
#pragma unroll
  for (int v = 0; v < V; ++v) {
    n.o[v] = n.o[v] + q.own[v];
    n.s[v] = n.s[v] + q.x[v];
    n.yl[v] = n.yl[v] + ((j & 1) ? q.own[v] : q.y[v]);
    n.yh[v] = n.yh[v] + ((j & 1) ? q.y[v] : q.own[v]);
    n.zl[v] = n.zl[v] + ((k & 1) ? q.own[v] : q.z[v]);
    n.zh[v] = n.zh[v] + ((k & 1) ? q.z[v] : q.own[v]);
  }
}

// Which faces of a cell lie on a wall.
struct Walls {
  bool s, yl, yh, zl, zh;
};

__device__ __forceinline__ Walls walls_of(const FlatDims& d, int sh, int p, int j, int k) {
  Walls w;
  w.s = sh ? (d.wall & 2) && p == d.np - 1 : (d.wall & 1) && p == 0;
  w.yl = (d.wall & 4) && j == 0;
  w.yh = (d.wall & 8) && j == d.ny - 1;
  w.zl = (d.wall & 16) && k == 0;
  w.zh = (d.wall & 32) && k == d.nz - 1;
  return w;
}

// A wall face counts twice (phi_ghost = -phi).
template <typename T, int V>
__device__ __forceinline__ T diag_of(const FlatOp<T>& op, const Coef<T, V>& c, int v,
                                     const Walls& w) {
#pragma clang fp contract(off)
  T g = op.a ? c.a[v] : op.alpha;
  g = g + c.o[v];
  g = g + (w.s ? T(2) * c.s[v] : c.s[v]);
  g = g + (w.yl ? T(2) * c.yl[v] : c.yl[v]);
  g = g + (w.yh ? T(2) * c.yh[v] : c.yh[v]);
  g = g + (w.zl ? T(2) * c.zl[v] : c.zl[v]);
  g = g + (w.zh ? T(2) * c.zh[v] : c.zh[v]);
  return g;
}

// ... and has no neighbour: a coefficient of 0.
template <typename T, int V>
__device__ __forceinline__ void drop_walls(Coef<T, V>& c, int v, const Walls& w) {
  c.s[v] = w.s ? T(0) : c.s[v];
  c.yl[v] = w.yl ? T(0) : c.yl[v];
  c.yh[v] = w.yh ? T(0) : c.yh[v];
  c.zl[v] = w.zl ? T(0) : c.zl[v];
  c.zh[v] = w.zh ? T(0) : c.zh[v];
}

// sum of c phi over the neighbours (walls dropped from c)
template <typename T, int V>
__device__ __forceinline__ T off_of(const Coef<T, V>& c, const Nb<T, V>& n, int v) {
#pragma clang fp contract(off)
  T o = c.o[v] * n.o[v];
  o = fma_(c.s[v], n.s[v], o);
  o = fma_(c.yl[v], n.yl[v], o);
  o = fma_(c.yh[v], n.yh[v], o);
  o = fma_(c.zl[v], n.zl[v], o);
  return fma_(c.zh[v], n.zh[v], o);
}

template <typename T>
__device__ __forceinline__ T resid_of(T f, T diag, T v, T off) {
#pragma clang fp contract(off)
  return f - fma_(diag, v, -off);
}

// Blocks are dealt to the 8 XCDs round robin: block b takes tile (b % 8) n/8 +
// b / 8, so that each XCD walks one contiguous part of the level and finds its
// tiles' neighbours in its own L2.
__device__ __forceinline__ int xcd_tile(int n, int reverse) {
  const int b = blockIdx.x, q = n / 8;
  const int t = b < 8 * q ? (b % 8) * q + b / 8 : b;
  return reverse ? n - 1 - t : t;
}

struct Grid2 {
  int lxl;      // log2 of lanes along x
  int nbx, nb;  // blocks along x, in all
  int reverse;
};

// Half-sweep.  Bound by HBM on the finest level: 4.5 values per cell, 604 MB at
// 256^3 FP64, 113 us = 5.3 TB/s (the box form moves 856 MB in 146-170 us); FP32
// 53 us (80).  Blocks are one row group deep along z: the level's planes are
// re-read from the L2 by the neighbouring blocks of the same XCD, and many
// small blocks keep more loads in flight than a march along z.  V pairs per
// lane (flat_width) make 16-byte loads; the block's lanes are 2^lxl along x by
// rows (j + ny k).  ZG: from zero; PE: with the coarse correction; STOP: with
// the norm of the colour's residual before the update.
template <typename T, int V, bool ZG, bool PE, bool STOP, bool NT>
__global__ void __launch_bounds__(256)
    k_flat_half(FlatOp<T> op, Grid2 g, const T* __restrict__ other, T* __restrict__ out,
                const T* __restrict__ f, int colour, FlatDims cd, const T* __restrict__ ec,
                const T* __restrict__ old, unsigned long long* normbits) {
#pragma clang fp contract(off)
  if (op.done && *op.done) return;
  const FlatDims& d = op.d;
  const int t = xcd_tile(g.nb, g.reverse);
  const int p0 = ((t % g.nbx << g.lxl) + (threadIdx.x & ((1 << g.lxl) - 1))) * V;
  const int row = (t / g.nbx) * (256 >> g.lxl) + (threadIdx.x >> g.lxl);
  const bool act = p0 < d.np && row < d.ny * d.nz;
  unsigned long long mx = 0;
  if (act) {
    const int k = row / d.ny, j = row - k * d.ny;
    const int s = (j + k + colour) & 1;
    const int at = p0 + d.sp * row;
    T fv[V], ov[V];
    Coef<T, V> c;
    Nb<T, V> n;
    Par<T, V> q;
    ldv<T, V, NT>(fv, f + colour * d.half + at);
    load_coef<T, V, NT>(c, op, colour, s, p0, j, k);
    if (!ZG) load_nb<T, V>(n, d, other, s, p0, j, k, row_ix(d, j, k));
    if (PE) load_par<T, V>(q, d, cd, ec, s, p0, j, k);
    if (STOP) ldv<T, V, NT>(ov, old + at);
    if (PE) add_par<T, V>(n, q, j, k);
    T nv[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
      const Walls w = walls_of(d, s, p0 + v, j, k);
      const T diag = diag_of<T, V>(op, c, v, w);
      drop_walls<T, V>(c, v, w);
      const T off = ZG ? T(0) : off_of<T, V>(c, n, v);
      nv[v] = (ZG ? fv[v] : fv[v] + off) * (T(1) / diag);
      if (STOP && p0 + v < d.np) {
        const unsigned long long bits = absbits(resid_of(fv[v], diag, ov[v], off));
        mx = bits > mx ? bits : mx;
      }
    }
    stv<T, V>(out + at, nv, d.np - p0);
  }
  if (STOP) block_max_u64(mx, normbits);
}

// Residual and restriction in one pass, red cells only: 4.6 values per fine
// cell, 113 us at 256^3 FP64 (box form, both colours: 148 us).  A lane takes
// coarse cell (I, J, K): the red cells of pair I on rows 2J, 2J + 1 of planes
// 2K, 2K + 1, four stencils in flight at once.
template <typename T, bool NT>
__global__ void __launch_bounds__(256)
    k_flat_restrict(FlatOp<T> op, Grid2 g, const T* __restrict__ v, const T* __restrict__ f,
                    FlatDims cd, T* __restrict__ cf) {
#pragma clang fp contract(off)
  if (op.done && *op.done) return;
  const FlatDims& d = op.d;
  const int t = xcd_tile(g.nb, g.reverse);
  const int I = (t % g.nbx << g.lxl) + (threadIdx.x & ((1 << g.lxl) - 1));
  const int row = (t / g.nbx) * (256 >> g.lxl) + (threadIdx.x >> g.lxl);
  const int cny = d.ny / 2;  // cd may be padded
  if (I >= d.np || row >= cny * (d.nz / 2)) return;
  const int K = row / cny, J = row - K * cny;
  T zs[2];
#pragma unroll
  for (int dk = 0; dk < 2; ++dk) {
    T r[2];
#pragma unroll
    for (int dj = 0; dj < 2; ++dj) {
      const int j = 2 * J + dj, k = 2 * K + dk, s = (dj + dk) & 1;
      const int at = I + d.sp * (j + d.ny * k);
      Coef<T, 1> c;
      Nb<T, 1> n;
      T fv[1];
      ldv<T, 1, NT>(fv, f + at);
      load_coef<T, 1, NT>(c, op, 0, s, I, j, k);
      load_nb<T, 1>(n, d, v + d.half, s, I, j, k, row_ix(d, j, k));
      const Walls w = walls_of(d, s, I, j, k);
      const T diag = diag_of<T, 1>(op, c, 0, w);
      drop_walls<T, 1>(c, 0, w);
      r[dj] = resid_of(fv[0], diag, v[at], off_of<T, 1>(c, n, 0));
    }
    zs[dk] = r[0] + r[1];
  }
  cf[((I + J + K) & 1) * cd.half + (I >> 1) + cd.sp * (J + cd.ny * K)] = (zs[0] + zs[1]) * T(0.125);
}

// UPD (the pass of an FP32 correction): vn = v + e, and the residual of vn.  v and
// e are read at the neighbours too, where the L2 has them, instead of vn
// written by a pass before: 220 us at 256^3 against 65 + 210 for the two passes
// (249 with the non-temporal hint: every face serves a cell of each colour, in
// different rows; 228 with one pair per lane).
template <typename T, typename TO, int V, bool UPD>
__global__ void __launch_bounds__(256)
    k_flat_resid(FlatOp<T> op, Grid2 g, const T* __restrict__ v, const T* __restrict__ f,
                 TO* __restrict__ out, unsigned long long* normbits, double* __restrict__ dots,
                 const float* __restrict__ e, T* __restrict__ vn) {
#pragma clang fp contract(off)
  if (op.done && *op.done) return;
  const FlatDims& d = op.d;
  const int t = xcd_tile(g.nb, g.reverse);
  const int p0 = ((t % g.nbx << g.lxl) + (threadIdx.x & ((1 << g.lxl) - 1))) * V;
  const int row = (t / g.nbx) * (256 >> g.lxl) + (threadIdx.x >> g.lxl);
  unsigned long long mx = 0;
  double dot = 0.0;
  if (p0 < d.np && row < d.ny * d.nz) {
    const int k = row / d.ny, j = row - k * d.ny;
    const int at = p0 + d.sp * row;
    const RowIx rx = row_ix(d, j, k);
#pragma unroll
    for (int colour = 0; colour < 2; ++colour) {
      const int s = (j + k + colour) & 1;
      T fv[V], cv[V];
      TO rv[V];
      Coef<T, V> c;
      Nb<T, V> n;
      if (f) ldv<T, V, false>(fv, f + colour * d.half + at);
      ldv<T, V, false>(cv, v + colour * d.half + at);
      load_coef<T, V, false>(c, op, colour, s, p0, j, k);
      load_nb<T, V>(n, d, v + (1 - colour) * d.half, s, p0, j, k, rx);
      if (UPD) {
        Nb<float, V> ne;
        float ce[V];
        ldv<float, V, false>(ce, e + colour * d.half + at);
        load_nb<float, V>(ne, d, e + (1 - colour) * d.half, s, p0, j, k, rx);
#pragma unroll
        for (int u = 0; u < V; ++u) {
          cv[u] = cv[u] + (T)ce[u];
          n.o[u] = n.o[u] + (T)ne.o[u];
          n.s[u] = n.s[u] + (T)ne.s[u];
          n.yl[u] = n.yl[u] + (T)ne.yl[u];
          n.yh[u] = n.yh[u] + (T)ne.yh[u];
          n.zl[u] = n.zl[u] + (T)ne.zl[u];
          n.zh[u] = n.zh[u] + (T)ne.zh[u];
        }
        stv<T, V>(vn + colour * d.half + at, cv, d.np - p0);
      }
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const Walls w = walls_of(d, s, p0 + u, j, k);
        const T diag = diag_of<T, V>(op, c, u, w);
        drop_walls<T, V>(c, u, w);
        const T off = off_of<T, V>(c, n, u);
        const T r = f ? resid_of(fv[u], diag, cv[u], off) : fma_(diag, cv[u], -off);
        rv[u] = (TO)r;
        if (p0 + u < d.np) {
          const unsigned long long bits = absbits(r);
          mx = bits > mx ? bits : mx;
          if (dots) dot += (double)cv[u] * (double)r;
        }
      }
      if (out) stv<TO, V>(out + colour * d.half + at, rv, d.np - p0);
    }
  }
  if (normbits) block_max_u64(mx, normbits);
  if (dots) {
    __shared__ double red[32];
    int phase = 0;
    dot = block_sum(dot, red, phase);
    if (threadIdx.x == 0) dots[blockIdx.x] = dot;
  }
}

// ---------------------------------------------------------------------------
// A whole sweep (both colours) in one pass over a level that streams from HBM:
// everything is read once, 5.5 values per cell against 9 for two half-sweeps.
// A work-group takes a column of the level, ox pairs by oy rows grown by a rim of
// one pair and two rows, one lane per pair, and marches along z: in step k it
// updates the first colour on plane k and the second on plane k - 1.  A lane's
// neighbours along z are its own earlier and later values (registers), those in
// the plane come through LDS (the first colour's input and its result, two
// planes of each so that a step needs one barrier).  The rim's first-colour cells
// are recomputed by every work-group that needs them; results go to another
// array, because neighbours still read the input.  Coefficients of plane k + 1
// are loaded while plane k is computed.
// 256^3 FP64: 172 us against 2 x 113 for half-sweeps, 650 MB fetched and 134
// written (the arrays are 604 and 134): 4.6 TB/s where a copy reaches 6.2.  What
// is left is the rims, 1.41 of a work-group's loads, and a barrier per plane;
// smaller work-groups, two to a CU, have larger rims (512 lanes, 32 pairs: 198
// us).  Cached loads throughout, since the non-temporal hint on the read-once
// arrays loses the rims as well (185-200 us).
// FP32 93 us against 2 x 52.
struct March {
  int ox, oy;        // pairs and rows a work-group writes
  int gx, gy;        // lanes: ox + 2, oy + 4
  int nbx, nby, nb;  // work-groups along x, y, in all
  int nz;            // planes a work-group writes
};

template <typename T, bool A>
struct MarchIn {
  T o, e0, e1, y[4], z[2], f[2], phi, par, old;
  T a[A ? 2 : 1];
};

template <typename T>
struct MarchCell {
  T o, s, yl, yh, zl, zh, f, rd;
};

template <typename T, bool ZG, bool PE, bool ST, bool A>
__global__ void __launch_bounds__(1024)
    k_flat_march(FlatOp<T> op, March g, const T* __restrict__ src, T* __restrict__ dst,
                 const T* __restrict__ f, int c0, FlatDims cd, const T* __restrict__ ec,
                 const T* __restrict__ old, unsigned long long* normbits) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char flat_lds[];
  const FlatDims& d = op.d;
  const int tid = threadIdx.x;
  // two planes of the input and of the first colour, each with a row before
  // and after
  const int ps = g.gx * (g.gy + 2);
  T* const lin = reinterpret_cast<T*>(flat_lds) + g.gx;
  T* const lfirst = lin + 2 * ps;
  const int t = xcd_tile(g.nb, 0);
  const int bx = t % g.nbx, by = t / g.nbx % g.nby, bz = t / g.nbx / g.nby;
  const int lx = tid % g.gx, ly = tid / g.gx;
  const int z0 = bz * g.nz, z1 = min(z0 + g.nz, d.nz);
  int p = bx * g.ox - 1 + lx, j = by * g.oy - 2 + ly;
  const bool lane = ly < g.gy;
  // the lane's pair belongs to the block (not its rim) and to the domain
  const bool own = lane && lx >= 1 && lx <= g.ox && ly >= 2 && ly < 2 + g.oy && p < d.np && j < d.ny;
  // the outermost rows only hold input
  const bool upd = lane && ly >= 1 && ly < g.gy - 1;
  // wrapped, or clamped: past a wall nothing that is read has a coefficient
  p = (d.wall & 1) ? min(max(p, 0), d.np - 1) : (p % d.np + d.np) % d.np;
  j = (d.wall & 4) ? min(max(j, 0), d.ny - 1) : (j % d.ny + d.ny) % d.ny;
  const int plane = d.sp * d.ny, planey = d.sp * (d.ny + 1);
  const int r0 = p + d.sp * j;
  auto zi = [&](int k) { return (d.wall & 16) ? min(max(k, 0), d.nz - 1) : (k + d.nz) % d.nz; };
  auto input = [&](int k) {
    if (ZG || !lane) return T(0);
    const T v = src[r0 + plane * zi(k)];
    return v;
  };
  auto load = [&](MarchIn<T, A>& in, int k) {
    if (!upd) return;
    const int kz = zi(k), r = r0 + plane * kz, ry = r0 + planey * kz;
    in.o = op.x[d.half + r];
    in.e0 = op.x[r];
    in.e1 = op.x[r + 1];
    // low faces of the first and the second colour's cell, then the high ones
    in.y[0] = op.y[c0 * d.yh + ry];
    in.y[1] = op.y[(1 - c0) * d.yh + ry];
    in.y[2] = op.y[(1 - c0) * d.yh + ry + d.sp];
    in.y[3] = op.y[c0 * d.yh + ry + d.sp];
    // the high z faces, which are plane k + 1's low ones (also for k = -1)
    const int rz = r0 + plane * (k < 0 ? 0 : kz + 1);
    in.z[0] = op.z[c0 * d.zh + rz];
    in.z[1] = op.z[(1 - c0) * d.zh + rz];
    in.f[0] = f[c0 * d.half + r];
    in.f[1] = f[(1 - c0) * d.half + r];
    if (A) {
      in.a[0] = op.a[c0 * d.half + r];
      in.a[A ? 1 : 0] = op.a[(1 - c0) * d.half + r];
    }
    if (ST) in.old = old[r];
  };
  auto parent = [&](int k) {
    return PE && lane ? coarse_at(cd, ec, p, j >> 1, zi(k) >> 1) : T(0);
  };
  const int ka = z0 - 1, kb = z1;
  MarchIn<T, A> pre, cur;
  T ph[3], fi[3];  // input at planes k - 1, k, k + 1; first colour at k - 2, k - 1, k
  T zc[2] = {T(0), T(0)};
  ph[0] = input(ka - 1);
  ph[1] = input(ka);
  ph[2] = input(ka + 1);
  if (PE) {
    ph[0] = ph[0] + parent(ka - 1);
    ph[1] = ph[1] + parent(ka);
    ph[2] = ph[2] + parent(ka + 1);
  }
  T phn = T(0), parn = T(0);  // plane k + 2's, on their way
  if (upd) {
    const int r = r0 + plane * zi(ka);
    zc[0] = op.z[c0 * d.zh + r];
    zc[1] = op.z[(1 - c0) * d.zh + r];
  }
  load(pre, ka);
  fi[0] = fi[1] = fi[2] = T(0);
  MarchCell<T> sec{};  // the second colour's cell on plane k - 1
  for (int q = tid; q < g.gx; q += 1024)
    for (int m = 0; m < 2; ++m) {
      lin[m * ps - g.gx + q] = T(0);
      lin[m * ps + g.gx * g.gy + q] = T(0);
      lfirst[m * ps - g.gx + q] = T(0);
      lfirst[m * ps + g.gx * g.gy + q] = T(0);
    }
  if (lane) {
    lin[tid] = ph[1];
    lfirst[tid] = T(0);
    lfirst[ps + tid] = T(0);
  }
  __syncthreads();
  unsigned long long mx = 0;
  int par = 0;
  for (int k = ka; k <= kb; ++k) {
    cur = pre;
    if (k < kb) {
      load(pre, k + 1);
      phn = input(k + 2);
      if (PE) parn = parent(k + 2);
    }
    const int sh = (j + k + c0) & 1;
    const T* L = lin + par * ps + tid;
    const T* M = lfirst + par * ps + tid;
    MarchCell<T> nxt{};
    if (upd) {
      const bool wy0 = (d.wall & 4) && j == 0, wy1 = (d.wall & 8) && j == d.ny - 1;
      const bool wz0 = (d.wall & 16) && k <= 0, wz1 = (d.wall & 32) && k >= d.nz - 1;
      // both colours' cells of plane k: the first's pair beside lies before
      // (sh = 0) or after, the second's on the other side
      Coef<T, 1> c;
      Walls w;
      c.o[0] = cur.o;
      c.s[0] = sh ? cur.e1 : cur.e0;
      c.yl[0] = cur.y[0];
      c.yh[0] = cur.y[2];
      c.zl[0] = zc[0];
      c.zh[0] = cur.z[1];
      c.a[0] = cur.a[0];
      w.s = sh ? (d.wall & 2) && p == d.np - 1 : (d.wall & 1) && p == 0;
      w.yl = wy0;
      w.yh = wy1;
      w.zl = wz0;
      w.zh = wz1;
      const T diag = diag_of<T, 1>(op, c, 0, w);
      drop_walls<T, 1>(c, 0, w);
      T off = T(0);
      if (!ZG) {
        Nb<T, 1> n;
        n.o[0] = ph[1];
        n.s[0] = L[sh ? 1 : -1];
        n.yl[0] = L[-g.gx];
        n.yh[0] = L[g.gx];
        n.zl[0] = ph[0];
        n.zh[0] = ph[2];
        off = off_of<T, 1>(c, n, 0);
      }
      fi[2] = (ZG ? cur.f[0] : cur.f[0] + off) * (T(1) / diag);
      if (own && k >= z0 && k < z1) {
        const int r = r0 + plane * k;
        dst[c0 * d.half + r] = fi[2];
        if (ST) {
          const unsigned long long b = absbits(resid_of(cur.f[0], diag, cur.old, off));
          mx = b > mx ? b : mx;
        }
      }
      c.o[0] = cur.o;
      c.s[0] = sh ? cur.e0 : cur.e1;
      c.yl[0] = cur.y[1];
      c.yh[0] = cur.y[3];
      c.zl[0] = zc[1];
      c.zh[0] = cur.z[0];
      c.a[0] = cur.a[A ? 1 : 0];
      w.s = sh ? (d.wall & 1) && p == 0 : (d.wall & 2) && p == d.np - 1;
      const T diag2 = diag_of<T, 1>(op, c, 0, w);
      drop_walls<T, 1>(c, 0, w);
      nxt = {c.o[0], c.s[0], c.yl[0], c.yh[0], c.zl[0], c.zh[0], cur.f[1], T(1) / diag2};
      zc[0] = cur.z[0];
      zc[1] = cur.z[1];
    }
    if (own && k - 1 >= z0) {
      // the second colour on plane k - 1 (same side as the first's on plane k)
      T o = sec.o * fi[1];
      o = fma_(sec.s, M[sh ? 1 : -1], o);
      o = fma_(sec.yl, M[-g.gx], o);
      o = fma_(sec.yh, M[g.gx], o);
      o = fma_(sec.zl, fi[0], o);
      o = fma_(sec.zh, fi[2], o);
      dst[(1 - c0) * d.half + r0 + plane * (k - 1)] = (sec.f + o) * sec.rd;
    }
    if (lane) {
      lin[(1 - par) * ps + tid] = ph[2];
      lfirst[(1 - par) * ps + tid] = fi[2];
    }
    __syncthreads();
    par ^= 1;
    sec = nxt;
    ph[0] = ph[1];
    ph[1] = ph[2];
    ph[2] = PE ? phn + parn : phn;
    fi[0] = fi[1];
    fi[1] = fi[2];
  }
  if (ST) block_max_u64(mx, normbits);
}

// ---------------------------------------------------------------------------
// Two sweeps in one launch, for levels whose passes are launches rather than
// memory traffic.  A work-group takes a block of OP pairs by OY by OZ rows,
// grown by 4 cells on every side, and runs the half-sweeps on the grown block:
// every half-sweep spoils one more layer of its rim, so the block itself comes
// out right, and no work-group needs another's values.  A lane keeps its
// pairs' coefficients in registers; the values are in LDS.  The results go to
// other arrays than the values came from (neighbouring work-groups still read
// those).
// MODE 0: pre-smoothing from zero (red, black, red, black), then the red
// residual's restriction; MODE 1: the same after a red half-sweep done elsewhere
// (black, red, black; src its red half); MODE 2: post-smoothing, colour C0
// first (src the other colour's half, to which the coarse correction is added
// as it is loaded).
// One work-group per CU (94 VGPRs, 1024 lanes; FP32 60, two); a block takes 6.5
// to 8 us, of which the coefficients' loads 2-3.  32^3 FP64 7.3 us for five
// launches of 3.6-6.7 us, 16^3 6.5.  A second round of blocks loses the gain:
// 64^3 FP64 (512 blocks) 20-21 us against 25 (pre) and 19 (post) for the separate
// launches; blocks of 8 pairs (one round) spill there and take 22.  FP32's fit:
// 64^3 11 us against 15 in two rounds of 4 and 22 for the launches.
// Blocks of OP pairs by 8 rows by 8 planes.
constexpr int kBlkOY = 8, kBlkOZ = 8, kBlkH = 4, kBlkLanes = 1024;
template <int OP>
struct Blk {
  static constexpr int GX = OP + kBlkH, GY = kBlkOY + 2 * kBlkH, GZ = kBlkOZ + 2 * kBlkH;
  static constexpr int NP = GX * GY * GZ, M = NP / kBlkLanes;
  static constexpr int PAD = GX * GY;  // neighbour reads past the block's ends
  static_assert(NP % kBlkLanes == 0, "whole pairs per lane");
};

template <typename T>
struct BlkPair {
  Coef<T, 1> c[2];
  T f[2], rdiag[2], diag;  // diag: the red cell's
  int side[2];             // LDS offset of the pair beside the colour's cell
  int at;                  // element in the level's arrays
  int rim;                 // layers outside the block (<= 0: inside)
  bool in;                 // a pair of the domain (or its periodic image)
};

template <typename T, int OP, int COLOUR>
__device__ __forceinline__ T blk_off(const BlkPair<T>& b, const T* O) {
  constexpr int GX = Blk<OP>::GX, GXY = GX * Blk<OP>::GY;
  Nb<T, 1> n;
  n.o[0] = O[0];
  n.s[0] = O[b.side[COLOUR]];
  n.yl[0] = O[-GX];
  n.yh[0] = O[GX];
  n.zl[0] = O[-GXY];
  n.zh[0] = O[GXY];
  return off_of<T, 1>(b.c[COLOUR], n, 0);
}

template <typename T, int OP, int MODE, int C0>
__global__ void __launch_bounds__(kBlkLanes)
    k_flat_block(FlatOp<T> op, int nbx, int nby, const T* __restrict__ src,
                 const T* __restrict__ f, T* __restrict__ dst, FlatDims cd, T* __restrict__ cf,
                 const T* __restrict__ ec) {
#pragma clang fp contract(off)
  using B = Blk<OP>;
  constexpr int kBlkGX = B::GX, kBlkGY = B::GY, kBlkNP = B::NP, kBlkM = B::M, kBlkPad = B::PAD,
                kBlkOP = OP;
  __shared__ T lds[2][kBlkNP + 2 * kBlkPad];
  T* const e[2] = {lds[0] + kBlkPad, lds[1] + kBlkPad};
  if (op.done && *op.done) return;
  const FlatDims& d = op.d;
  const int tid = threadIdx.x;
  const int bx = blockIdx.x % nbx, by = blockIdx.x / nbx % nby, bz = blockIdx.x / nbx / nby;
  const int p0 = bx * kBlkOP, y0 = by * kBlkOY, z0 = bz * kBlkOZ;
  BlkPair<T> b[kBlkM];
#pragma unroll
  for (int m = 0; m < kBlkM; ++m) {
    const int q = tid + m * kBlkLanes;
    const int lx = q % kBlkGX, ly = q / kBlkGX % kBlkGY, lz = q / (kBlkGX * kBlkGY);
    int p = p0 - kBlkH / 2 + lx, j = y0 - kBlkH + ly, k = z0 - kBlkH + lz;
    // along x the nearer cell of the pair counts
    b[m].rim = max(max(2 * max(kBlkH / 2 - lx, lx - (kBlkH / 2 + kBlkOP - 1)) - 1,
                       max(kBlkH - ly, ly - (kBlkH + kBlkOY - 1))),
                   max(kBlkH - lz, lz - (kBlkH + kBlkOZ - 1)));
    bool in = true;
    if (d.wall & 1)
      in = in && p >= 0 && p < d.np;
    else
      p = (p % d.np + d.np) % d.np;
    if (d.wall & 4)
      in = in && j >= 0 && j < d.ny;
    else
      j = (j % d.ny + d.ny) % d.ny;
    if (d.wall & 16)
      in = in && k >= 0 && k < d.nz;
    else
      k = (k % d.nz + d.nz) % d.nz;
    b[m].in = in;
    b[m].at = 0;
    T v = T(0);
    if (in) {
      const int at = p + d.sp * (j + d.ny * k);
      b[m].at = at;
      if (MODE == 1) v = src[at];
      if (MODE == 2) v = src[at] + coarse_at(cd, ec, p, j >> 1, k >> 1);
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const int sh = (j + k + c) & 1;
        b[m].f[c] = f[c * d.half + at];
        load_coef<T, 1, false>(b[m].c[c], op, c, sh, p, j, k);
        const Walls w = walls_of(d, sh, p, j, k);
        const T diag = diag_of<T, 1>(op, b[m].c[c], 0, w);
        drop_walls<T, 1>(b[m].c[c], 0, w);
        b[m].rdiag[c] = T(1) / diag;
        if (c == 0) b[m].diag = diag;
        b[m].side[c] = sh ? 1 : -1;
      }
    }
    // slots outside the domain are read with a coefficient of 0
    e[MODE == 2 ? 1 - C0 : 0][q] = v;
    e[MODE == 2 ? C0 : 1][q] = T(0);
  }
  for (int q = tid; q < kBlkPad; q += kBlkLanes)
    for (int c = 0; c < 2; ++c) {
      e[c][q - kBlkPad] = T(0);
      e[c][kBlkNP + q] = T(0);
    }
  __syncthreads();
  // half-sweep number t (0 ..) of a run that ends on the block itself after
  // the last: layers beyond `layers` are spoiled by then and skipped
#define BLK_HALF(COL, ZG, LAYERS)                                                              \
  {                                                                                            \
    _Pragma("unroll") for (int m = 0; m < kBlkM; ++m) {                                        \
      const int q = tid + m * kBlkLanes;                                                       \
      if (b[m].in && b[m].rim <= LAYERS)                                                       \
        e[COL][q] = (ZG ? b[m].f[COL] : b[m].f[COL] + blk_off<T, OP, COL>(b[m], e[1 - (COL)] + q)) * \
                    b[m].rdiag[COL];                                                           \
    }                                                                                          \
    __syncthreads();                                                                           \
  }
  if (MODE == 0) BLK_HALF(0, true, 4)
  if (MODE <= 1) {
    BLK_HALF(1, false, 3)
    BLK_HALF(0, false, 2)
    BLK_HALF(1, false, 1)
  } else {
    BLK_HALF(C0, false, 3)
    BLK_HALF(1 - C0, false, 2)
    BLK_HALF(C0, false, 1)
    BLK_HALF(1 - C0, false, 0)
  }
#undef BLK_HALF
  T r[kBlkM];
#pragma unroll
  for (int m = 0; m < kBlkM; ++m) {
    const int q = tid + m * kBlkLanes;
    // inside the block and, for periodic domains too, not a wrapped image
    const int lx = q % kBlkGX, ly = q / kBlkGX % kBlkGY, lz = q / (kBlkGX * kBlkGY);
    const bool own = b[m].rim <= 0 && p0 - kBlkH / 2 + lx < d.np && y0 - kBlkH + ly < d.ny &&
                     z0 - kBlkH + lz < d.nz;
    r[m] = T(0);
    if (own) {
      dst[b[m].at] = e[0][q];
      dst[d.half + b[m].at] = e[1][q];
      if (MODE <= 1)
        r[m] = resid_of(b[m].f[0], b[m].diag, e[0][q], blk_off<T, OP, 0>(b[m], e[1] + q));
    }
  }
  if (MODE <= 1) {
    __syncthreads();
#pragma unroll
    for (int m = 0; m < kBlkM; ++m) e[0][tid + m * kBlkLanes] = r[m];
    __syncthreads();
    if (tid < kBlkOP * (kBlkOY / 2) * (kBlkOZ / 2)) {
      const int cx = tid % kBlkOP, cy = tid / kBlkOP % (kBlkOY / 2), cz = tid / (kBlkOP * (kBlkOY / 2));
      const int I = p0 + cx, J = y0 / 2 + cy, K = z0 / 2 + cz;
      if (2 * I < d.nx && 2 * J < d.ny && 2 * K < d.nz) {
        const int q = kBlkH / 2 + cx + kBlkGX * (kBlkH + 2 * cy + kBlkGY * (kBlkH + 2 * cz));
        const T zl = e[0][q] + e[0][q + kBlkGX];
        const T zh = e[0][q + kBlkGX * kBlkGY] + e[0][q + kBlkGX * kBlkGY + kBlkGX];
        cf[((I + J + K) & 1) * cd.half + (I >> 1) + cd.sp * (J + cd.ny * K)] = (zl + zh) * T(0.125);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Between box arrays and the split-colour layout; grid.y = box, lanes stride
// the box's cells or faces.

__device__ __forceinline__ int split_at(const FlatDims& d, int i, int j, int k) {
  return ((i + j + k) & 1) * d.half + (i >> 1) + d.sp * (j + d.ny * k);
}
__device__ __forceinline__ int xface_at(const FlatDims& d, int i, int j, int k) {
  return (i & 1) * d.half + (i >> 1) + d.sp * (j + d.ny * k);
}
__device__ __forceinline__ int yface_at(const FlatDims& d, int i, int j, int k) {
  return ((i + j + k) & 1) * d.yh + (i >> 1) + d.sp * (j + (d.ny + 1) * k);
}
__device__ __forceinline__ int zface_at(const FlatDims& d, int i, int j, int k) {
  return ((i + j + k) & 1) * d.zh + (i >> 1) + d.sp * (j + d.ny * k);
}
__device__ __forceinline__ int face_at(const FlatDims& d, int dir, const int (&c)[3]) {
  return dir == 0 ? xface_at(d, c[0], c[1], c[2])
                  : dir == 1 ? yface_at(d, c[0], c[1], c[2]) : zface_at(d, c[0], c[1], c[2]);
}

// GHOSTS (scatter): the ghost layer too, wrapped along periodic directions; what
// lies past a wall is left as it is.
template <typename T, bool GATHER, bool GHOSTS>
__global__ void __launch_bounds__(256)
    k_flat_boxes(const BoxInfo* __restrict__ boxes, int3 lo, FlatDims d, const T* src, T* dst,
                 int ng, unsigned long long* normbits) {
  const BoxInfo B = boxes[blockIdx.y];
  const int nx = B.hi[0] - B.lo[0] + 1, ny = B.hi[1] - B.lo[1] + 1, nz = B.hi[2] - B.lo[2] + 1;
  const long long off = ng ? B.off_g1 : B.off_g0;
  const int sy = nx + 2 * ng;
  const long long sz = (long long)sy * (ny + 2 * ng);
  if (GHOSTS) {
    const int n0 = nx + 2, n1 = ny + 2;
    const unsigned all = (unsigned)n0 * n1 * (nz + 2);
    for (unsigned e = blockIdx.x * 256 + threadIdx.x; e < all; e += gridDim.x * 256) {
      const unsigned t = e / n0, gk = t / n1;
      int i = (int)(e - t * n0) - 1 + B.lo[0] - lo.x, j = (int)(t - gk * n1) - 1 + B.lo[1] - lo.y,
          k = (int)gk - 1 + B.lo[2] - lo.z;
      const bool in = ((d.wall & 1) == 0 || (i >= 0 && i < d.nx)) &&
                      ((d.wall & 4) == 0 || (j >= 0 && j < d.ny)) &&
                      ((d.wall & 16) == 0 || (k >= 0 && k < d.nz));
      i = i < 0 ? i + d.nx : i >= d.nx ? i - d.nx : i;
      j = j < 0 ? j + d.ny : j >= d.ny ? j - d.ny : j;
      k = k < 0 ? k + d.nz : k >= d.nz ? k - d.nz : k;
      if (in) dst[off + e] = src[split_at(d, i, j, k)];
    }
    return;
  }
  const unsigned total = nx * ny * nz;
  unsigned long long mx = 0;
  for (unsigned e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int t = e / nx, il = e - t * nx, kl = t / ny, jl = t - kl * ny;
    const long long b = off + (il + ng) + (long long)sy * (jl + ng) + sz * (kl + ng);
    const int q = split_at(d, B.lo[0] - lo.x + il, B.lo[1] - lo.y + jl, B.lo[2] - lo.z + kl);
    if (GATHER) {
      const T v = src[b];
      dst[q] = v;
      const unsigned long long bits = absbits(v);
      mx = bits > mx ? bits : mx;
    } else {
      dst[b] = src[q];
    }
  }
  if (GATHER && normbits) block_max_u64(mx, normbits);
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_flat_faces(const BoxInfo* __restrict__ boxes, int3 lo, FlatDims d, int dir,
                 const T* __restrict__ b, T beta, T ih, T* __restrict__ dst) {
#pragma clang fp contract(off)
  const BoxInfo B = boxes[blockIdx.y];
  int n[3];
  for (int a = 0; a < 3; ++a) n[a] = B.hi[a] - B.lo[a] + 1 + (a == dir ? 1 : 0);
  const int dn[3] = {d.nx, d.ny, d.nz};
  const int l[3] = {lo.x, lo.y, lo.z};
  const unsigned total = n[0] * n[1] * n[2];
  for (unsigned e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    int q[3];
    const int t = e / n[0];
    q[0] = e - t * n[0];
    q[2] = t / n[1];
    q[1] = t - q[2] * n[1];
    // a box's last face is the next box's first, unless the domain ends there
    if (q[dir] == n[dir] - 1 && B.hi[dir] - l[dir] + 1 != dn[dir]) continue;
    for (int a = 0; a < 3; ++a) q[a] += B.lo[a] - l[a];
    dst[face_at(d, dir, q)] = (beta * b[B.off_f[dir] + e]) * ih;
  }
}

// grid.z = direction, grid.y = box; lanes stride the box's last plane of faces.
// They are a 65th of the faces of 64^3 boxes, along x one cache line each: 23 us at
// 256^3, 11.5 at 128^3.  Up to four units in the last place count as the same:
// less than what the operator's own products round, and what two boxes' owners
// may differ by that computed the face each in its own way.
template <typename T>
struct BoxFaces {
  const T* b[3];
  T ih[3];
};
template <typename T>
__global__ void __launch_bounds__(256)
    k_flat_shared(const BoxInfo* __restrict__ boxes, int3 lo, FlatOp<T> op, BoxFaces<T> faces,
                  T beta, unsigned long long* differ) {
#pragma clang fp contract(off)
  const FlatDims& d = op.d;
  const int dir = blockIdx.z, u = dir == 0 ? 1 : 0, v = dir == 2 ? 1 : 2;
  const BoxInfo B = boxes[blockIdx.y];
  int n[3];
  for (int a = 0; a < 3; ++a) n[a] = B.hi[a] - B.lo[a] + 1 + (a == dir ? 1 : 0);
  const int dn[3] = {d.nx, d.ny, d.nz};
  const int l[3] = {lo.x, lo.y, lo.z};
  const bool end = B.hi[dir] - l[dir] + 1 == dn[dir];
  if (end && (d.wall >> (2 * dir) & 1)) return;
  const T* b = (dir == 0 ? faces.b[0] : dir == 1 ? faces.b[1] : faces.b[2]) + B.off_f[dir];
  const T* c = dir == 0 ? op.x : dir == 1 ? op.y : op.z;
  const T ih = dir == 0 ? faces.ih[0] : dir == 1 ? faces.ih[1] : faces.ih[2];
  const T ulps = sizeof(T) == 8 ? T(0x1p-50) : T(0x1p-21);
  bool bad = false;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < n[u] * n[v]; e += gridDim.x * 256) {
    int q[3];
    q[dir] = n[dir] - 1;
    q[v] = e / n[u];
    q[u] = e - q[v] * n[u];
    const T own = (beta * b[q[0] + n[0] * ((long long)q[1] + n[1] * (long long)q[2])]) * ih;
    for (int a = 0; a < 3; ++a) q[a] += B.lo[a] - l[a];
    if (end) q[dir] = 0;
    const T other = c[face_at(d, dir, q)];
    bad = bad || !(own == other || fabs(own - other) <= ulps * fabs(other));
  }
  if (bad) atomicOr(differ, 1ull);
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_flat_acoef(const BoxInfo* __restrict__ boxes, int3 lo, FlatDims d, const T* __restrict__ a,
                 T alpha, T* __restrict__ dst) {
  const BoxInfo B = boxes[blockIdx.y];
  const int nx = B.hi[0] - B.lo[0] + 1, ny = B.hi[1] - B.lo[1] + 1, nz = B.hi[2] - B.lo[2] + 1;
  const unsigned total = nx * ny * nz;
  for (unsigned e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
    const int t = e / nx, il = e - t * nx, kl = t / ny, jl = t - kl * ny;
    dst[split_at(d, B.lo[0] - lo.x + il, B.lo[1] - lo.y + jl, B.lo[2] - lo.z + kl)] =
        alpha * a[B.off_g0 + e];
  }
}

// ---------------------------------------------------------------------------
// Vectors: both halves of an array as one run of n elements (a multiple of 4),
// padding included.  The padding is 0 for good: no gather, sweep or residual
// writes it and the sums below read it, so what a solve that fails leaves there
// would fail every later one.  A finite factor times 0 keeps it; where the
// factor is not finite (a uniform branch) the update skips it.
__device__ __forceinline__ bool is_cell(const FlatDims& d, long long e) {
  if (e >= d.half) e -= d.half;
  return e < (long long)d.sp * d.ny * d.nz && (int)e % d.sp < d.np;
}

template <typename TZ>
__global__ void __launch_bounds__(256)
    k_flat_dot(long long n, const double* __restrict__ a, const TZ* __restrict__ z,
               double* __restrict__ partials) {
  __shared__ double red[32];
  int phase = 0;
  double s0 = 0.0, s1 = 0.0;
  const long long step = (long long)gridDim.x * 512;
  for (long long e = (blockIdx.x * 256ll + threadIdx.x) * 2; e < n; e += step) {
    double av[2];
    TZ zv[2];
    ldv<double, 2, false>(av, a + e);
    ldv<TZ, 2, false>(zv, z + e);
    s0 += av[0] * (double)zv[0];
    s1 += av[1] * (double)zv[1];
  }
  const double s = block_sum(s0 + s1, red, phase);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

template <typename TZ>
__global__ void __launch_bounds__(256)
    k_flat_cg_p(FlatDims d, double* __restrict__ p, const TZ* __restrict__ z, const double* num,
                const double* den, int first) {
  const long long n = 2ll * d.half;
  const double be = first ? 0.0 : *num / *den;
  const bool all = isfinite(be);
  for (long long e = (blockIdx.x * 256ll + threadIdx.x) * 2; e < n; e += gridDim.x * 512ll) {
    TZ zv[2];
    double pv[2] = {0.0, 0.0};
    ldv<TZ, 2, false>(zv, z + e);
    if (!first) ldv<double, 2, false>(pv, p + e);
    for (int v = 0; v < 2; ++v)
      if (all || is_cell(d, e + v))
        pv[v] = first ? (double)zv[v] : (double)zv[v] + be * pv[v];
    stv<double, 2>(p + e, pv, 2);
  }
}

__global__ void __launch_bounds__(256)
    k_flat_cg_xr(FlatDims d, double* __restrict__ x, const double* __restrict__ p,
                 double* __restrict__ r, const double* __restrict__ q, const double* num,
                 const double* den, unsigned long long* normbits, float* __restrict__ r32) {
  const long long n = 2ll * d.half;
  const double al = *num / *den;
  const bool all = isfinite(al);
  unsigned long long mx = 0;
  for (long long e = (blockIdx.x * 256ll + threadIdx.x) * 2; e < n; e += gridDim.x * 512ll) {
    double xv[2], pv[2], rv[2], qv[2];
    ldv<double, 2, false>(xv, x + e);
    ldv<double, 2, false>(pv, p + e);
    ldv<double, 2, false>(rv, r + e);
    ldv<double, 2, false>(qv, q + e);
    float rs[2];
    for (int v = 0; v < 2; ++v) {
      if (all || is_cell(d, e + v)) {
        xv[v] += al * pv[v];
        rv[v] -= al * qv[v];
      }
      rs[v] = (float)rv[v];
      const unsigned long long bits = absbits(rv[v]);
      mx = bits > mx ? bits : mx;
    }
    stv<double, 2>(x + e, xv, 2);
    stv<double, 2>(r + e, rv, 2);
    if (r32) stv<float, 2>(r32 + e, rs, 2);
  }
  block_max_u64(mx, normbits);
}

__global__ void __launch_bounds__(256)
    k_flat_sum(long long n, const double* __restrict__ v, double* __restrict__ partials) {
  __shared__ double red[32];
  int phase = 0;
  double s = 0.0;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll) s += v[e];
  s = block_sum(s, red, phase);
  if (threadIdx.x == 0) partials[blockIdx.x] = s;
}

// grid.y = half
__global__ void __launch_bounds__(256)
    k_flat_shift(FlatDims d, double* __restrict__ v, const double* sum) {
  const double m = *sum / ((double)d.nx * d.ny * d.nz);
  double* h = v + (long long)blockIdx.y * d.half;
  const unsigned total = d.sp * d.ny * d.nz;
  for (unsigned e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256)
    if (e % d.sp < d.np) h[e] -= m;
}

__global__ void __launch_bounds__(256)
    k_flat_maxabs(long long n, const double* __restrict__ v, unsigned long long* normbits) {
  unsigned long long mx = 0;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll) {
    const unsigned long long bits = absbits(v[e]);
    mx = bits > mx ? bits : mx;
  }
  block_max_u64(mx, normbits);
}

// ---------------------------------------------------------------------------
// The tail.

// LDS (elements) of one tail level: e and f (both halves), r (red half).
__host__ __device__ inline int tail_elems(const FlatDims& d) { return 5 * d.half; }

// Pointers read from the plan are known to be global, so that their loads do
// not share a wait counter with LDS.
template <typename T>
__device__ __forceinline__ T* as_global(T* p) {
  return (T*)(__attribute__((address_space(1))) T*)p;
}

template <typename T>
__device__ __forceinline__ FlatOp<T> tail_op(const FlatTail<T>* tp, int l) {
  FlatOp<T> op = tp->lev[l].op;
  op.x = as_global(op.x);
  op.y = as_global(op.y);
  op.z = as_global(op.z);
  op.a = as_global(op.a);
  return op;
}

// A level's arrays: both halves of e and f, r the red half.
template <typename T>
struct TailArr {
  T *e, *f, *r;
};

template <typename T, bool LDS>
__device__ __forceinline__ TailArr<T> tail_arr(const FlatTail<T>* tp, T* lds, int l) {
  TailArr<T> a;
  if (LDS) {
    // one level after the other, then the bottom's e, f and the CG's p
    int o = 0;
    for (int m = 0; m < l; ++m) o += tail_elems(tp->lev[m].op.d);
    const int h = tp->lev[l].op.d.half;
    a.e = lds + o;
    a.f = a.e + 2 * h;
    a.r = a.f + 2 * h;
  } else {
    a.e = as_global(tp->lev[l].e);
    a.f = as_global(tp->lev[l].f);
    a.r = as_global(tp->lev[l].r);
  }
  return a;
}

// A pair of the level and both its cells' coefficients (walls dropped) and
// diagonals.
template <typename T>
struct TailPair {
  Coef<T, 1> c[2];
  T diag, rdiag[2];  // diag: the red cell's
  int p, j, k;
};

template <typename T>
__device__ __forceinline__ TailPair<T> tail_pair(const FlatOp<T>& op, int q) {
  TailPair<T> m;
  const FlatDims& d = op.d;
  const int t = q / d.np;
  m.p = q - t * d.np;
  m.k = t / d.ny;
  m.j = t - m.k * d.ny;
#pragma unroll
  for (int c = 0; c < 2; ++c) {
    const int sh = (m.j + m.k + c) & 1;
    load_coef<T, 1, false>(m.c[c], op, c, sh, m.p, m.j, m.k);
    const Walls w = walls_of(d, sh, m.p, m.j, m.k);
    const T diag = diag_of<T, 1>(op, m.c[c], 0, w);
    drop_walls<T, 1>(m.c[c], 0, w);
    m.rdiag[c] = T(1) / diag;
    if (c == 0) m.diag = diag;
  }
  return m;
}

// The update of the colour's cell of a pair.
template <typename T, int COLOUR, bool ZG, bool PE>
__device__ __forceinline__ void tail_update(const FlatOp<T>& op, const TailArr<T>& A,
                                            const TailPair<T>& m, const FlatDims& cd,
                                            const T* ec) {
#pragma clang fp contract(off)
  const FlatDims& d = op.d;
  const Coef<T, 1>& c = m.c[COLOUR];
  const int s = (m.j + m.k + COLOUR) & 1;
  const int at = m.p + d.sp * (m.j + d.ny * m.k);
  T off = T(0);
  if (!ZG) {
    Nb<T, 1> n;
    load_nb<T, 1>(n, d, A.e + (1 - COLOUR) * d.half, s, m.p, m.j, m.k, row_ix(d, m.j, m.k));
    if (PE) {
      Par<T, 1> q;
      load_par<T, 1>(q, d, cd, ec, s, m.p, m.j, m.k);
      add_par<T, 1>(n, q, m.j, m.k);
    }
    off = off_of<T, 1>(c, n, 0);
  }
  const T fv = A.f[COLOUR * d.half + at];
  A.e[COLOUR * d.half + at] = (ZG ? fv : fv + off) * m.rdiag[COLOUR];
}

// One half-sweep of the work-group.  own: the lane's pair where the level has
// at most one per lane, else unused.
template <typename T, int COLOUR, bool ZG, bool PE, int NT>
__device__ __forceinline__ void tail_half(const FlatOp<T>& op, const TailArr<T>& A,
                                          const TailPair<T>& own, int npair, const FlatDims& cd,
                                          const T* ec) {
  if (npair <= NT) {
    if ((int)threadIdx.x < npair) tail_update<T, COLOUR, ZG, PE>(op, A, own, cd, ec);
  } else {
    for (int q = threadIdx.x; q < npair; q += NT)
      tail_update<T, COLOUR, ZG, PE>(op, A, tail_pair(op, q), cd, ec);
  }
  __syncthreads();
}

// The coarsest levels and the CG in one work-group, latency bound: a barrier and
// one LDS round trip per half-sweep, since a lane keeps its pair's coefficients
// in registers for the whole visit of a level and e, f and r are in LDS.  8^3
// and 4^3 cells FP64: 20 us, the CG's iterations most of it (the box form,
// arrays in the L2: 36 us; with the plan as a by-value argument the compiler
// spilled: 81 us).  NT lanes: 512 where every level has at most that many
// pairs and the bottom that many cells, else 1024.
template <typename T, bool LDS, int NT>
__global__ void __launch_bounds__(NT) k_flat_tail(const FlatTail<T>* __restrict__ tp) {
#pragma clang fp contract(off)
  extern __shared__ __align__(16) unsigned char flat_lds[];
  __shared__ double red[32];
  T* const lds = reinterpret_cast<T*>(flat_lds);
  const int tid = threadIdx.x;
  const int nlev = tp->nlev;
  if (tp->bt.done && *as_global(tp->bt.done)) return;
  if (LDS) {
    // the first level's right-hand side
    const int n = 2 * tp->lev[0].op.d.half;
    const T* f = as_global(tp->lev[0].f);
    T* to = tail_arr<T, LDS>(tp, lds, 0).f;
    for (int e = tid; e < n; e += NT) to[e] = f[e];
    __syncthreads();
  }
  for (int l = 0; l < nlev; ++l) {
    const FlatOp<T> op = tail_op(tp, l);
    const FlatDims& d = op.d;
    const FlatDims cd = tp->lev[l + 1].op.d;
    const TailArr<T> A = tail_arr<T, LDS>(tp, lds, l), C = tail_arr<T, LDS>(tp, lds, l + 1);
    const int npair = d.np * d.ny * d.nz;
    TailPair<T> own;
    if (npair <= NT && tid < npair) own = tail_pair(op, tid);
    for (int k = 0; k < tp->nu1; ++k) {
      if (k == 0)
        tail_half<T, 0, true, false, NT>(op, A, own, npair, cd, nullptr);
      else
        tail_half<T, 0, false, false, NT>(op, A, own, npair, cd, nullptr);
      tail_half<T, 1, false, false, NT>(op, A, own, npair, cd, nullptr);
    }
    // cells added to the coarser level have no right-hand side
    if (LDS && (2 * cd.nx != d.nx || 2 * cd.ny != d.ny || 2 * cd.nz != d.nz))
      for (int e = tid; e < 2 * cd.half; e += NT) C.f[e] = T(0);
    // residual of the red cells (the black ones' is zero)
    for (int q = tid; q < npair; q += NT) {
      if (npair > NT) own = tail_pair(op, q);
      const int s = (own.j + own.k) & 1, at = own.p + d.sp * (own.j + d.ny * own.k);
      Nb<T, 1> n;
      load_nb<T, 1>(n, d, A.e + d.half, s, own.p, own.j, own.k, row_ix(d, own.j, own.k));
      A.r[at] = resid_of(A.f[at], own.diag, A.e[at], off_of<T, 1>(own.c[0], n, 0));
    }
    __syncthreads();
    const int cny = d.ny / 2, ncell = d.np * cny * (d.nz / 2);  // cd may be padded
    for (int q = tid; q < ncell; q += NT) {
      const int t = q / d.np, I = q - t * d.np, K = t / cny, J = t - K * cny;
      const int b = I + d.sp * (2 * J + d.ny * 2 * K);
      const int bz = d.sp * d.ny;
      const T z0 = A.r[b] + A.r[b + d.sp];
      const T z1 = A.r[b + bz] + A.r[b + bz + d.sp];
      C.f[((I + J + K) & 1) * cd.half + (I >> 1) + cd.sp * (J + cd.ny * K)] = (z0 + z1) * T(0.125);
    }
    __syncthreads();
  }
  {
    const TailArr<T> B = tail_arr<T, LDS>(tp, lds, nlev);
    T* p = LDS ? B.f + 2 * tp->lev[nlev].op.d.half : lds;
    BottomTables bt = tp->bt;
    bt.nbr = as_global(bt.nbr);
    bt.map_rhs = as_global(bt.map_rhs);
    bt.map_out = as_global(bt.map_out);
    const T* diag = as_global(tp->bdiag);
    const T* coef = as_global(tp->bcoef);
    if (bt.n <= 64) {
      if (tid < 64)
        cg_lds_run<T, 1, true>(bt, diag, coef, B.f, B.e, 0, tp->tol, tp->maxiter, tp->singular,
                               as_global(tp->iters), p, red, 64, 1);
    } else {
      cg_lds_run<T, 1>(bt, diag, coef, B.f, B.e, 0, tp->tol, tp->maxiter, tp->singular,
                       as_global(tp->iters), p, red, NT, (bt.n + 63) / 64);
    }
  }
  __syncthreads();
  const bool reverse = tp->reverse != 0;
  for (int l = nlev - 1; l >= 0; --l) {
    const FlatOp<T> op = tail_op(tp, l);
    const FlatDims& d = op.d;
    const FlatDims cd = tp->lev[l + 1].op.d;
    const TailArr<T> A = tail_arr<T, LDS>(tp, lds, l);
    const T* ec = tail_arr<T, LDS>(tp, lds, l + 1).e;
    const int npair = d.np * d.ny * d.nz;
    TailPair<T> own;
    if (npair <= NT && tid < npair) own = tail_pair(op, tid);
    if (reverse) {
      for (int k = 0; k < tp->nu2; ++k) {
        if (k == 0)
          tail_half<T, 1, false, true, NT>(op, A, own, npair, cd, ec);
        else
          tail_half<T, 1, false, false, NT>(op, A, own, npair, cd, ec);
        tail_half<T, 0, false, false, NT>(op, A, own, npair, cd, ec);
      }
    } else {
      for (int k = 0; k < tp->nu2; ++k) {
        if (k == 0)
          tail_half<T, 0, false, true, NT>(op, A, own, npair, cd, ec);
        else
          tail_half<T, 0, false, false, NT>(op, A, own, npair, cd, ec);
        tail_half<T, 1, false, false, NT>(op, A, own, npair, cd, ec);
      }
    }
  }
  if (LDS) {
    const FlatDims d = tp->lev[0].op.d;
    const T* e = tail_arr<T, LDS>(tp, lds, 0).e;
    T* to = as_global(tp->lev[0].e);
    for (int q = tid; q < d.np * d.ny * d.nz; q += NT) {
      const int t = q / d.np, at = q - t * d.np + d.sp * t;
      to[at] = e[at];
      to[d.half + at] = e[d.half + at];
    }
  }
}

// ---------------------------------------------------------------------------
// Deep bottom: setup of the coarsenings and the vector passes of the iteration.
// Latency bound: a bottom of 28^3 takes nine launches of 4 to 18 us an iteration
// and 4 to 6 iterations (0.35 ms a cycle) where one work-group's CG from the L2
// took 12 ms.  A reduction ends in the block that finishes last, so that a dot
// product is one launch and its result decides on the device whether the rest
// of the iteration does anything.

__device__ __forceinline__ int3 cell_of(const FlatDims& d, int at) {
  const int colour = at >= d.half, e = at - colour * d.half;
  const int p = e % d.sp, row = e / d.sp, j = row % d.ny, k = row / d.ny;
  return make_int3(2 * p + ((j + k + colour) & 1), j, k);
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_fill(BottomTables bt, StencilArgs<T> op, FlatDims d, int3 pad, T* __restrict__ x,
                T* __restrict__ y, T* __restrict__ z, T* __restrict__ mass,
                T* __restrict__ wall) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= bt.n) return;
  const int at = bt.map_out[c];
  const int3 q = cell_of(d, at);
  const int ix[3] = {q.x, q.y, q.z}, N[3] = {d.nx, d.ny, d.nz}, m[3] = {pad.x, pad.y, pad.z};
  const T* bs[3] = {op.b0, op.b1, op.b2};
  const T ih[3] = {op.ih0, op.ih1, op.ih2};
  T* dst[3] = {x, y, z};
  T w = T(0);
#pragma unroll
  for (int dir = 0; dir < 3; ++dir) {
    const int lo = 2 * dir * bt.n + c, hi = lo + bt.n;
    const T cl = (op.beta * bs[dir][bt.fidx[lo]]) * ih[dir];
    if (bt.nbr[hi] < 0) w = w + T(2) * ((op.beta * bs[dir][bt.fidx[hi]]) * ih[dir]);
    if (bt.nbr[lo] < 0) {
      w = w + T(2) * cl;
    } else if (ix[dir] > 0) {
      dst[dir][face_at(d, dir, ix)] = cl;
    } else {
      // the link from the last cell, in m + 1 pieces
      int f[3] = {ix[0], ix[1], ix[2]};
      const T v = T(m[dir] + 1) * cl;
      dst[dir][face_at(d, dir, f)] = v;
      for (f[dir] = N[dir] - m[dir]; f[dir] <= N[dir]; ++f[dir]) dst[dir][face_at(d, dir, f)] = v;
    }
  }
  mass[at] = op.a ? op.alpha * op.a[bt.aidx[c]] : op.alpha;
  wall[at] = w;
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_diag(FlatDims d, const T* __restrict__ x, const T* __restrict__ y,
                const T* __restrict__ z, const T* __restrict__ mass, const T* __restrict__ wall,
                T* __restrict__ a) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= d.nx * d.ny * d.nz) return;
  const int i = c % d.nx, j = c / d.nx % d.ny, k = c / d.nx / d.ny;
  const int at = split_at(d, i, j, k);
  const T s = x[xface_at(d, i, j, k)] + x[xface_at(d, i + 1, j, k)] + y[yface_at(d, i, j, k)] +
              y[yface_at(d, i, j + 1, k)] + z[zface_at(d, i, j, k)] + z[zface_at(d, i, j, k + 1)];
  const T v = mass[at] + wall[at];
  a[at] = v == T(0) && s == T(0) ? T(1) : v;
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_coarsen(FlatDims d, const T* __restrict__ x, const T* __restrict__ y,
                   const T* __restrict__ z, const T* __restrict__ mass,
                   const T* __restrict__ wall, FlatDims cd, int3 pad, T* __restrict__ cx,
                   T* __restrict__ cy, T* __restrict__ cz, T* __restrict__ cmass,
                   T* __restrict__ cwall) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  const int n[3] = {d.nx / 2, d.ny / 2, d.nz / 2};  // without the cells added
  const int per = ~d.wall, nx = n[0] + 1, ny = n[1] + 1;
  if (c >= nx * ny * (n[2] + 1)) return;
  const int I = c % nx, J = c / nx % ny, K = c / nx / ny;
  const int i = 2 * I, j = 2 * J, k = 2 * K;
  // ends of a periodic direction: the link in pad + 1 pieces
  if (J < n[1] && K < n[2]) {
    const bool link = (per & 1) && pad.x && (I == 0 || I == n[0]);
    const T v = T(link ? 0.125 : 0.0625) *
                ((x[xface_at(d, i, j, k)] + x[xface_at(d, i, j + 1, k)]) +
                 (x[xface_at(d, i, j, k + 1)] + x[xface_at(d, i, j + 1, k + 1)]));
    cx[xface_at(cd, I, J, K)] = v;
    if (link && I) cx[xface_at(cd, I + 1, J, K)] = v;
  }
  if (I < n[0] && K < n[2]) {
    const bool link = (per & 4) && pad.y && (J == 0 || J == n[1]);
    const T v = T(link ? 0.125 : 0.0625) *
                ((y[yface_at(d, i, j, k)] + y[yface_at(d, i + 1, j, k)]) +
                 (y[yface_at(d, i, j, k + 1)] + y[yface_at(d, i + 1, j, k + 1)]));
    cy[yface_at(cd, I, J, K)] = v;
    if (link && J) cy[yface_at(cd, I, J + 1, K)] = v;
  }
  if (I < n[0] && J < n[1]) {
    const bool link = (per & 16) && pad.z && (K == 0 || K == n[2]);
    const T v = T(link ? 0.125 : 0.0625) *
                ((z[zface_at(d, i, j, k)] + z[zface_at(d, i + 1, j, k)]) +
                 (z[zface_at(d, i, j + 1, k)] + z[zface_at(d, i + 1, j + 1, k)]));
    cz[zface_at(cd, I, J, K)] = v;
    if (link && K) cz[zface_at(cd, I, J, K + 1)] = v;
  }
  if (I < n[0] && J < n[1] && K < n[2]) {
    T m = T(0), w = T(0);
    for (int u = 0; u < 8; ++u) {
      const int at = split_at(d, i + (u & 1), j + (u >> 1 & 1), k + (u >> 2));
      m = m + mass[at];
      w = w + wall[at];
    }
    const int at = split_at(cd, I, J, K);
    cmass[at] = T(0.125) * m;
    cwall[at] = T(0.0625) * w;
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_bottom(BottomTables bt, FlatOp<T> op, T* __restrict__ diag, T* __restrict__ coef) {
  const int c = blockIdx.x * 256 + threadIdx.x;
  if (c >= bt.n) return;
  const FlatDims& d = op.d;
  const int at = bt.map_out[c];
  const int3 q = cell_of(d, at);
  const T f[6] = {op.x[xface_at(d, q.x, q.y, q.z)],     op.x[xface_at(d, q.x + 1, q.y, q.z)],
                  op.y[yface_at(d, q.x, q.y, q.z)],     op.y[yface_at(d, q.x, q.y + 1, q.z)],
                  op.z[zface_at(d, q.x, q.y, q.z)],     op.z[zface_at(d, q.x, q.y, q.z + 1)]};
  T g = op.a[at];
#pragma unroll
  for (int u = 0; u < 6; ++u) {
    g = g + f[u];
    coef[u * bt.n + c] = bt.nbr[u * bt.n + c] < 0 ? T(0) : f[u];
  }
  diag[c] = g;
}

// The launch's partial sums s (one per block, all lanes hold it): true in the
// block that finishes last, with their sum in *total, added in block order.
__device__ __forceinline__ bool deep_total(double s, double* partials, unsigned* count,
                                           double* red, int& phase, double* total) {
  __shared__ bool last;
  if (threadIdx.x == 0) {
    partials[blockIdx.x] = s;
    __threadfence();
    last = atomicAdd(count, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return false;
  __threadfence();
  double t = 0.0;
  for (int b = threadIdx.x; b < (int)gridDim.x; b += 256) t += partials[b];
  *total = block_sum(t, red, phase);
  if (threadIdx.x == 0) *count = 0;
  return true;
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_init(long long n, const T* __restrict__ f, T* __restrict__ r, T* __restrict__ x,
                T* __restrict__ p, double* __restrict__ partials, DeepState* st) {
  __shared__ double red[32];
  int phase = 0;
  double s = 0.0;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll) {
    const T v = f[e];
    r[e] = v;
    x[e] = T(0);
    p[e] = T(0);
    s += (double)v * (double)v;
  }
  s = block_sum(s, red, phase);
  double b2;
  if (deep_total(s, partials, &st->count, red, phase, &b2) && threadIdx.x == 0) {
    st->rho = 0.0;
    st->b2 = b2;
    st->it = 0;
    st->done = b2 > 0.0 ? 0 : 1;
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_rz(long long n, const T* __restrict__ r, const T* __restrict__ z,
              double* __restrict__ partials, DeepState* st) {
  __shared__ double red[32];
  if (st->done) return;
  int phase = 0;
  double s = 0.0;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll)
    s += (double)r[e] * (double)z[e];
  s = block_sum(s, red, phase);
  double rho;
  if (deep_total(s, partials, &st->count, red, phase, &rho) && threadIdx.x == 0) {
    st->beta = st->it > 0 ? rho / st->rho : 0.0;
    st->rho = rho;
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_p(long long n, const T* __restrict__ z, T* __restrict__ p, const DeepState* st) {
  if (st->done) return;
  const T be = (T)st->beta;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll)
    p[e] = z[e] + be * p[e];
}

template <typename T>
__global__ void __launch_bounds__(256)
    k_deep_xr(long long n, T* __restrict__ x, const T* __restrict__ p, T* __restrict__ r,
              const T* __restrict__ q, const double* __restrict__ pqs, int npq, double tol2,
              double* __restrict__ partials, DeepState* st) {
  __shared__ double red[32];
  if (st->done) return;
  int phase = 0;
  double s = 0.0;
  for (int b = threadIdx.x; b < npq; b += 256) s += pqs[b];
  const double pq = block_sum(s, red, phase), al = st->rho / pq;
  const bool ok = pq > 0.0 && fabs(al) < 1e300;
  const T alT = ok ? (T)al : T(0);
  s = 0.0;
  if (ok)
    for (long long e = blockIdx.x * 256ll + threadIdx.x; e < n; e += gridDim.x * 256ll) {
      x[e] = x[e] + alT * p[e];
      const T rv = r[e] - alT * q[e];
      r[e] = rv;
      s += (double)rv * (double)rv;
    }
  s = block_sum(s, red, phase);
  double rr;
  if (deep_total(s, partials, &st->count, red, phase, &rr) && threadIdx.x == 0) {
    if (ok) ++st->it;
    st->done = !ok ? 2 : !(rr > tol2 * st->b2) ? 1 : 0;
  }
}

// Lanes along x for `width` work items per row: the smallest power of two that
// covers them, at most a wavefront (a wavefront's loads are then one run).
Grid2 grid_of(int width, int rows, int reverse) {
  Grid2 g;
  g.lxl = 0;
  while (g.lxl < 6 && (1 << g.lxl) < width) ++g.lxl;
  const int lx = 1 << g.lxl, ly = 256 / lx;
  g.nbx = (width + lx - 1) / lx;
  g.nb = g.nbx * ((rows + ly - 1) / ly);
  g.reverse = reverse;
  return g;
}

// Pairs per lane: two FP64 or four FP32 make 16-byte loads.  One where a
// periodic row is no multiple of that (the group's last neighbour wraps), and
// on levels too small to fill the chip that way.
template <typename T>
int flat_width(const FlatDims& d) {
  const int v = 16 / (int)sizeof(T);
  if (!(d.wall & 2) && d.np % v) return 1;
  return (long long)d.np * d.ny * d.nz >= v * 262144ll ? v : 1;
}

int vec_blocks(long long n) { return (int)std::min<long long>((n + 511) / 512, 4096); }

// Rows of at least a cache line start on one; shorter rows (whole levels of
// which the tail keeps in LDS) on 16 bytes.
int flat_pitch(int nx, int elem) {
  const int need = nx / 2 + 1, to = need >= 128 / elem ? 128 / elem : 16 / elem;
  return (need + to - 1) / to * to;
}

}  // namespace

FlatDims flat_dims(const int n[3], const int periodic[3], int elem) {
  FlatDims d;
  d.nx = n[0];
  d.ny = n[1];
  d.nz = n[2];
  d.np = (n[0] + 1) / 2;
  const int line = 128 / elem;
  d.sp = flat_pitch(n[0], elem);
  d.wall = 0;
  for (int a = 0; a < 3; ++a)
    if (!periodic[a]) d.wall |= 3 << (2 * a);
  // past the end: the widest load that starts inside a row
  auto up = [&](long long v) { return (int)((v + line + 63) / 64 * 64); };
  d.half = up((long long)d.sp * d.ny * d.nz);
  d.yh = up((long long)d.sp * (d.ny + 1) * d.nz);
  d.zh = up((long long)d.sp * d.ny * (d.nz + 1));
  return d;
}

bool flat_fits(const int n[3], int elem) {
  const int line = 128 / elem;
  const long long sp = flat_pitch(n[0], elem);
  return 2 * (sp * (n[1] + 1) * (n[2] + 1) + line + 64) < (1ll << 31);
}

template <typename T>
hipError_t launch_flat_half(hipStream_t st, const FlatOp<T>& op, FlatPass ps, const T* other,
                            T* out, const T* f, int colour, bool zero_guess, const FlatDims* cd,
                            const T* ec, const T* old, unsigned long long* normbits) {
  const FlatDims c = cd ? *cd : FlatDims{};
  const int V = flat_width<T>(op.d);
  const Grid2 g = grid_of((op.d.np + V - 1) / V, op.d.ny * op.d.nz, ps.reverse);
#define FH2(W, ZG, PE, SP, NT)                                                                 \
  hipLaunchKernelGGL((k_flat_half<T, W, ZG, PE, SP, NT>), dim3(g.nb), dim3(256), 0, st, op, g, \
                     other, out, f, colour, c, ec, old, normbits)
#define FH1(W, NT)                                                                 \
  if (zero_guess) FH2(W, true, false, false, NT);                                  \
  else if (ec) FH2(W, false, true, false, NT);                                     \
  else if (old) FH2(W, false, false, true, NT);                                    \
  else FH2(W, false, false, false, NT)
  constexpr int W = 16 / sizeof(T);
  if (V == 1) {
    FH1(1, false);
  } else if (ps.stream) {
    FH1(W, true);
  } else {
    FH1(W, false);
  }
#undef FH1
#undef FH2
  return hipGetLastError();
}

// Whether cd holds the coarsening of d, as it is or padded at its high ends.
static bool coarse_fits(const FlatDims& d, const FlatDims& cd) {
  return d.nx % 2 == 0 && d.ny % 2 == 0 && d.nz % 2 == 0 && 2 * cd.nx >= d.nx &&
         2 * cd.ny >= d.ny && 2 * cd.nz >= d.nz;
}

template <typename T>
hipError_t launch_flat_restrict(hipStream_t st, const FlatOp<T>& op, FlatPass ps, const T* v,
                                const T* f, const FlatDims& cd, T* cf) {
  if (!coarse_fits(op.d, cd)) return hipErrorInvalidValue;
  const Grid2 g = grid_of(op.d.np, op.d.ny / 2 * (op.d.nz / 2), ps.reverse);
  if (ps.stream)
    hipLaunchKernelGGL((k_flat_restrict<T, true>), dim3(g.nb), dim3(256), 0, st, op, g, v, f, cd,
                       cf);
  else
    hipLaunchKernelGGL((k_flat_restrict<T, false>), dim3(g.nb), dim3(256), 0, st, op, g, v, f, cd,
                       cf);
  return hipGetLastError();
}

// Work-groups of a march: tiles at most 64 pairs wide (at 256^3 FP64 194 us with
// 32 pairs, 172 with 64: a row's two rim pairs cost a cache line each where the
// neighbour's copy has left the L2; 280 with rows off the lines at 43, 350 with
// whole rows of 128, which leave 3 of 7 rows to write), as many rows as 1024 lanes
// hold, and as many planes each as fill the chip evenly (`resident` work-groups
// at a time).
static March march_of(const FlatDims& d, int resident) {
  March m{};
  m.nbx = (d.np + 63) / 64;
  m.ox = (d.np + m.nbx - 1) / m.nbx;
  m.gx = m.ox + 2;
  const int rows = std::min(1024 / m.gx - 4, d.ny);
  m.nby = (d.ny + rows - 1) / rows;
  m.oy = (d.ny + m.nby - 1) / m.nby;
  m.gy = m.oy + 4;
  double cost = 0;
  for (int ns = 1; ns <= d.nz; ++ns) {
    const int nz = (d.nz + ns - 1) / ns;
    const int n = m.nbx * m.nby * ((d.nz + nz - 1) / nz);
    // rounds, each as long as its planes and the two of the rim
    const double c = double((n + resident - 1) / resident) * (nz + 4.0);
    if (cost == 0 || c < cost) {
      cost = c;
      m.nz = nz;
      m.nb = n;
    }
  }
  return m;
}

template <typename T>
hipError_t launch_flat_sweep(hipStream_t st, const FlatOp<T>& op, const T* src, T* dst, const T* f,
                             int c0, bool zero_guess, const FlatDims* cd, const T* ec,
                             const T* old, unsigned long long* normbits) {
  const FlatDims& d = op.d;
  const FlatDims c = cd ? *cd : FlatDims{};
  // FP64 100-120 VGPRs: one work-group per CU; FP32 up to 66: two of most forms
  const March m = march_of(d, sizeof(T) == 8 ? 256 : 512);
  if (m.nb <= 0) return hipErrorInvalidValue;
  const size_t lds = sizeof(T) * 4 * (size_t)m.gx * (m.gy + 2);
  if (lds > 65536) return hipErrorInvalidValue;
  const T* in = zero_guess ? nullptr : src + (1 - c0) * (size_t)d.half;
#define FM2(Z, P, S, A)                                                                        \
  hipLaunchKernelGGL((k_flat_march<T, Z, P, S, A>), dim3(m.nb), dim3(1024), lds, st, op, m, in, \
                     dst, f, c0, c, ec, old, normbits)
#define FM(A)                                  \
  if (zero_guess) FM2(true, false, false, A);  \
  else if (ec) FM2(false, true, false, A);     \
  else if (old) FM2(false, false, true, A);    \
  else FM2(false, false, false, A)
  if (op.a) {
    FM(true);
  } else {
    FM(false);
  }
#undef FM
#undef FM2
  return hipGetLastError();
}

// Blocks of OP pairs that cover a level.
static long long blocks_of(const FlatDims& d, int op) {
  return (long long)((d.np + op - 1) / op) * ((d.ny + kBlkOY - 1) / kBlkOY) *
         ((d.nz + kBlkOZ - 1) / kBlkOZ);
}

int flat_block_pairs(const FlatDims& d, int elem) {
  if (blocks_of(d, 4) <= 256) return 4;
  return elem == 4 && blocks_of(d, 8) <= 256 ? 8 : 0;
}

template <typename T>
hipError_t launch_flat_block(hipStream_t st, const FlatOp<T>& op, FlatBlockMode mode, const T* src,
                             const T* f, T* dst, const FlatDims& cd, T* cf, const T* ec) {
  const FlatDims& d = op.d;
  if (!coarse_fits(d, cd)) return hipErrorInvalidValue;
  const int w = flat_block_pairs(d, sizeof(T));
  if (w == 0) return hipErrorInvalidValue;
  const int nbx = (d.np + w - 1) / w, nby = (d.ny + kBlkOY - 1) / kBlkOY;
  const dim3 grid((unsigned)blocks_of(d, w));
#define FBK(W, M, C)                                                                               \
  hipLaunchKernelGGL((k_flat_block<T, W, M, C>), grid, dim3(kBlkLanes), 0, st, op, nbx, nby, src, \
                     f, dst, cd, cf, ec)
#define FB(M, C)                          \
  if constexpr (sizeof(T) == 4) {         \
    if (w == 8) FBK(8, M, C);             \
    else FBK(4, M, C);                    \
  } else {                                \
    FBK(4, M, C);                         \
  }
  switch (mode) {
    case FlatBlockMode::pre_zero: FB(0, 0) break;
    case FlatBlockMode::pre_after_red: FB(1, 0) break;
    case FlatBlockMode::post_red: src += d.half; FB(2, 0) break;
    case FlatBlockMode::post_black: FB(2, 1) break;
  }
#undef FB
#undef FBK
  return hipGetLastError();
}

int flat_resid_blocks(const FlatDims& d) { return grid_of(d.np, d.ny * d.nz, 0).nb; }

template <typename T, typename TO>
hipError_t launch_flat_resid(hipStream_t st, const FlatOp<T>& op, FlatPass ps, const T* v,
                             const T* f, TO* out, unsigned long long* normbits, double* dots) {
  const Grid2 g = grid_of(op.d.np, op.d.ny * op.d.nz, ps.reverse);
  hipLaunchKernelGGL((k_flat_resid<T, TO, 1, false>), dim3(g.nb), dim3(256), 0, st, op, g, v, f,
                     out, normbits, dots, (const float*)nullptr, (T*)nullptr);
  return hipGetLastError();
}

hipError_t launch_flat_update_resid(hipStream_t st, const FlatOp<double>& op, FlatPass ps,
                                    const double* v, const float* e, double* vn, const double* f,
                                    float* out, unsigned long long* normbits) {
  const int V = flat_width<double>(op.d);
  const Grid2 g = grid_of((op.d.np + V - 1) / V, op.d.ny * op.d.nz, ps.reverse);
#define FU(V)                                                                                 \
  hipLaunchKernelGGL((k_flat_resid<double, float, V, true>), dim3(g.nb), dim3(256), 0, st, op, \
                     g, v, f, out, normbits, (double*)nullptr, e, vn)
  if (V == 1) FU(1);
  else FU(2);
#undef FU
  return hipGetLastError();
}

static dim3 box_grid(int nbox, int cells) {
  return dim3(std::min((cells + 1023) / 1024, 1024), nbox);
}

template <typename T>
hipError_t launch_flat_gather(hipStream_t st, const BoxInfo* boxes, int nbox, int max_cells,
                              const int lo[3], const FlatDims& d, const T* src, int ng, T* dst,
                              unsigned long long* normbits) {
  hipLaunchKernelGGL((k_flat_boxes<T, true, false>), box_grid(nbox, max_cells), dim3(256), 0, st, boxes,
                     make_int3(lo[0], lo[1], lo[2]), d, src, dst, ng, normbits);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_flat_scatter(hipStream_t st, const BoxInfo* boxes, int nbox, int max_cells,
                               const int lo[3], const FlatDims& d, const T* src, T* dst, int ng,
                               bool ghosts) {
  if (ghosts && ng != 1) return hipErrorInvalidValue;
  const int3 l = make_int3(lo[0], lo[1], lo[2]);
  if (ghosts)
    hipLaunchKernelGGL((k_flat_boxes<T, false, true>), box_grid(nbox, max_cells), dim3(256), 0, st,
                       boxes, l, d, src, dst, ng, nullptr);
  else
    hipLaunchKernelGGL((k_flat_boxes<T, false, false>), box_grid(nbox, max_cells), dim3(256), 0,
                       st, boxes, l, d, src, dst, ng, nullptr);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_flat_faces(hipStream_t st, const BoxInfo* boxes, int nbox, int max_faces,
                             const int lo[3], const FlatDims& d, int dir, const T* b, T beta, T ih,
                             T* dst) {
  hipLaunchKernelGGL((k_flat_faces<T>), box_grid(nbox, max_faces), dim3(256), 0, st, boxes,
                     make_int3(lo[0], lo[1], lo[2]), d, dir, b, beta, ih, dst);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_flat_shared(hipStream_t st, const BoxInfo* boxes, int nbox, int max_plane,
                              const int lo[3], const FlatOp<T>& op, const T* const b[3], T beta,
                              const T ih[3], unsigned long long* differ) {
  dim3 g = box_grid(nbox, max_plane);
  g.z = 3;
  BoxFaces<T> f;
  for (int a = 0; a < 3; ++a) {
    f.b[a] = b[a];
    f.ih[a] = ih[a];
  }
  hipLaunchKernelGGL((k_flat_shared<T>), g, dim3(256), 0, st, boxes,
                     make_int3(lo[0], lo[1], lo[2]), op, f, beta, differ);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_flat_acoef(hipStream_t st, const BoxInfo* boxes, int nbox, int max_cells,
                             const int lo[3], const FlatDims& d, const T* a, T alpha, T* dst) {
  hipLaunchKernelGGL((k_flat_acoef<T>), box_grid(nbox, max_cells), dim3(256), 0, st, boxes,
                     make_int3(lo[0], lo[1], lo[2]), d, a, alpha, dst);
  return hipGetLastError();
}

template <typename TZ>
hipError_t launch_flat_dot(hipStream_t st, long long n, const double* a, const TZ* z,
                           double* partials, double* out) {
  const int nb = std::min(vec_blocks(n), kFlatDotBlocks);
  hipLaunchKernelGGL((k_flat_dot<TZ>), dim3(nb), dim3(256), 0, st, n, a, z, partials);
  const hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_sum_final(st, partials, nb, out);
}

template <typename TZ>
hipError_t launch_flat_cg_p(hipStream_t st, const FlatDims& d, double* p, const TZ* z,
                            const double* num, const double* den, int first) {
  hipLaunchKernelGGL((k_flat_cg_p<TZ>), dim3(vec_blocks(2ll * d.half)), dim3(256), 0, st, d, p, z,
                     num, den, first);
  return hipGetLastError();
}

hipError_t launch_flat_cg_xr(hipStream_t st, const FlatDims& d, double* x, const double* p,
                             double* r, const double* q, const double* num, const double* den,
                             unsigned long long* normbits, float* r32) {
  hipLaunchKernelGGL(k_flat_cg_xr, dim3(vec_blocks(2ll * d.half)), dim3(256), 0, st, d, x, p, r, q,
                     num, den, normbits, r32);
  return hipGetLastError();
}

hipError_t launch_flat_remove_mean(hipStream_t st, const FlatDims& d, double* v, double* partials,
                                   double* sum) {
  const long long n = 2ll * d.half;
  const int nb = std::min(vec_blocks(n), kFlatDotBlocks);
  hipLaunchKernelGGL(k_flat_sum, dim3(nb), dim3(256), 0, st, n, v, partials);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess) e = launch_sum_final(st, partials, nb, sum);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_flat_shift, dim3(vec_blocks(d.half), 2), dim3(256), 0, st, d, v, sum);
  return hipGetLastError();
}

hipError_t launch_flat_maxabs(hipStream_t st, long long n, const double* v,
                              unsigned long long* normbits) {
  hipLaunchKernelGGL(k_flat_maxabs, dim3(vec_blocks(n)), dim3(256), 0, st, n, v, normbits);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_flat_tail(hipStream_t st, const FlatTail<T>& t, const FlatTail<T>* dt) {
  if (!dt || t.nlev < 1 || t.nlev > kTailMaxLevels || t.bt.n < 1 || t.bt.n > kTailMaxBottom)
    return hipErrorInvalidValue;
  long long el = 4ll * t.lev[t.nlev].op.d.half + t.bt.n;
  for (int l = 0; l < t.nlev; ++l) el += tail_elems(t.lev[l].op.d);
  bool small = t.bt.n <= 512;
  for (int l = 0; l < t.nlev; ++l) {
    const FlatDims& d = t.lev[l].op.d;
    small = small && d.np * d.ny * d.nz <= 512;
  }
  const bool fits = el * (long long)sizeof(T) <= 60 * 1024;
#define FT(L, N, BYTES) \
  hipLaunchKernelGGL((k_flat_tail<T, L, N>), dim3(1), dim3(N), BYTES, st, dt)
  if (fits && small) FT(true, 512, el * sizeof(T));
  else if (fits) FT(true, 1024, el * sizeof(T));
  else FT(false, 1024, t.bt.n * sizeof(T));
#undef FT
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_fill(hipStream_t st, const BottomTables& bt, const StencilArgs<T>& op,
                            const FlatDims& d, const int pad[3], T* x, T* y, T* z, T* mass,
                            T* wall) {
  hipLaunchKernelGGL(k_deep_fill<T>, dim3((bt.n + 255) / 256), dim3(256), 0, st, bt, op, d,
                     make_int3(pad[0], pad[1], pad[2]), x, y, z, mass, wall);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_diag(hipStream_t st, const FlatDims& d, const T* x, const T* y, const T* z,
                            const T* mass, const T* wall, T* a) {
  hipLaunchKernelGGL(k_deep_diag<T>, dim3((d.nx * d.ny * d.nz + 255) / 256), dim3(256), 0, st, d, x,
                     y, z, mass, wall, a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_coarsen(hipStream_t st, const FlatDims& d, const T* x, const T* y,
                               const T* z, const T* mass, const T* wall, const FlatDims& cd,
                               const int pad[3], T* cx, T* cy, T* cz, T* cmass, T* cwall) {
  if (!coarse_fits(d, cd) || 2 * (cd.nx - pad[0]) != d.nx || 2 * (cd.ny - pad[1]) != d.ny ||
      2 * (cd.nz - pad[2]) != d.nz || std::max({pad[0], pad[1], pad[2]}) > 1)
    return hipErrorInvalidValue;
  const int n = (d.nx / 2 + 1) * (d.ny / 2 + 1) * (d.nz / 2 + 1);
  hipLaunchKernelGGL(k_deep_coarsen<T>, dim3((n + 255) / 256), dim3(256), 0, st, d, x, y, z, mass,
                     wall, cd, make_int3(pad[0], pad[1], pad[2]), cx, cy, cz, cmass, cwall);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_bottom(hipStream_t st, const BottomTables& bt, const FlatOp<T>& op, T* diag,
                              T* coef) {
  hipLaunchKernelGGL(k_deep_bottom<T>, dim3((bt.n + 255) / 256), dim3(256), 0, st, bt, op, diag,
                     coef);
  return hipGetLastError();
}

static int deep_blocks(long long n) {
  return (int)std::min<long long>((n + 1023) / 1024, kDeepBlocks);
}

template <typename T>
hipError_t launch_deep_init(hipStream_t st, long long n, const T* f, T* r, T* x, T* p,
                            double* partials, DeepState* s) {
  hipLaunchKernelGGL(k_deep_init<T>, dim3(deep_blocks(n)), dim3(256), 0, st, n, f, r, x, p,
                     partials, s);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_rz(hipStream_t st, long long n, const T* r, const T* z, double* partials,
                          DeepState* s) {
  hipLaunchKernelGGL(k_deep_rz<T>, dim3(deep_blocks(n)), dim3(256), 0, st, n, r, z, partials, s);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_p(hipStream_t st, long long n, const T* z, T* p, const DeepState* s) {
  hipLaunchKernelGGL(k_deep_p<T>, dim3(deep_blocks(n)), dim3(256), 0, st, n, z, p, s);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_deep_xr(hipStream_t st, long long n, T* x, const T* p, T* r, const T* q,
                          const double* pq, int npq, double tol2, double* partials, DeepState* s) {
  hipLaunchKernelGGL(k_deep_xr<T>, dim3(deep_blocks(n)), dim3(256), 0, st, n, x, p, r, q, pq, npq,
                     tol2, partials, s);
  return hipGetLastError();
}

#define INST(T)                                                                                    \
  template hipError_t launch_deep_fill<T>(hipStream_t, const BottomTables&, const StencilArgs<T>&, \
                                          const FlatDims&, const int*, T*, T*, T*, T*, T*);        \
  template hipError_t launch_deep_diag<T>(hipStream_t, const FlatDims&, const T*, const T*,        \
                                          const T*, const T*, const T*, T*);                       \
  template hipError_t launch_deep_coarsen<T>(hipStream_t, const FlatDims&, const T*, const T*,     \
                                             const T*, const T*, const T*, const FlatDims&,        \
                                             const int*, T*, T*, T*, T*, T*);                      \
  template hipError_t launch_deep_bottom<T>(hipStream_t, const BottomTables&, const FlatOp<T>&,    \
                                            T*, T*);                                               \
  template hipError_t launch_deep_init<T>(hipStream_t, long long, const T*, T*, T*, T*, double*,   \
                                          DeepState*);                                             \
  template hipError_t launch_deep_rz<T>(hipStream_t, long long, const T*, const T*, double*,       \
                                        DeepState*);                                               \
  template hipError_t launch_deep_p<T>(hipStream_t, long long, const T*, T*, const DeepState*);    \
  template hipError_t launch_deep_xr<T>(hipStream_t, long long, T*, const T*, T*, const T*,        \
                                        const double*, int, double, double*, DeepState*);          \
  template hipError_t launch_flat_half<T>(hipStream_t, const FlatOp<T>&, FlatPass, const T*, T*,   \
                                          const T*, int, bool, const FlatDims*, const T*,          \
                                          const T*, unsigned long long*);                          \
  template hipError_t launch_flat_restrict<T>(hipStream_t, const FlatOp<T>&, FlatPass, const T*,   \
                                              const T*, const FlatDims&, T*);                      \
  template hipError_t launch_flat_gather<T>(hipStream_t, const BoxInfo*, int, int, const int*,     \
                                            const FlatDims&, const T*, int, T*,                    \
                                            unsigned long long*);                                  \
  template hipError_t launch_flat_scatter<T>(hipStream_t, const BoxInfo*, int, int, const int*,    \
                                             const FlatDims&, const T*, T*, int, bool);            \
  template hipError_t launch_flat_faces<T>(hipStream_t, const BoxInfo*, int, int, const int*,      \
                                           const FlatDims&, int, const T*, T, T, T*);              \
  template hipError_t launch_flat_shared<T>(hipStream_t, const BoxInfo*, int, int, const int*,     \
                                            const FlatOp<T>&, const T* const*, T, const T*,        \
                                            unsigned long long*);                                  \
  template hipError_t launch_flat_acoef<T>(hipStream_t, const BoxInfo*, int, int, const int*,      \
                                           const FlatDims&, const T*, T, T*);                      \
  template hipError_t launch_flat_dot<T>(hipStream_t, long long, const double*, const T*, double*, \
                                         double*);                                                 \
  template hipError_t launch_flat_cg_p<T>(hipStream_t, const FlatDims&, double*, const T*,         \
                                          const double*, const double*, int);                      \
  template hipError_t launch_flat_sweep<T>(hipStream_t, const FlatOp<T>&, const T*, T*, const T*,  \
                                           int, bool, const FlatDims*, const T*, const T*,         \
                                           unsigned long long*);                                   \
  template hipError_t launch_flat_block<T>(hipStream_t, const FlatOp<T>&, FlatBlockMode, const T*, \
                                           const T*, T*, const FlatDims&, T*, const T*);           \
  template hipError_t launch_flat_tail<T>(hipStream_t, const FlatTail<T>&, const FlatTail<T>*);

INST(double)
INST(float)
#undef INST

template hipError_t launch_flat_resid<double, double>(hipStream_t, const FlatOp<double>&, FlatPass,
                                                      const double*, const double*, double*,
                                                      unsigned long long*, double*);
template hipError_t launch_flat_resid<float, float>(hipStream_t, const FlatOp<float>&, FlatPass,
                                                    const float*, const float*, float*,
                                                    unsigned long long*, double*);
template hipError_t launch_flat_resid<double, float>(hipStream_t, const FlatOp<double>&, FlatPass,
                                                     const double*, const double*, float*,
                                                     unsigned long long*, double*);

}  // namespace amrmg
