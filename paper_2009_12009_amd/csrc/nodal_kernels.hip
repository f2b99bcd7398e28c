// gfx950 kernels of the node-centred finite-element solve (the nodal solver
// of the paper's "Linear Solvers" section).
//
// Finest level: (A phi)_u = sum over the 8 cells s at node u of sigma_s times
// the cell's stiffness row, (1/V) sum_{corners b} K_{1-s, b} phi(u + b + s - 1);
// K depends only on which coordinates of the two corners differ, so the
// kernel takes the 8 values kappa[pattern] (K / V).  Coarse levels: 27
// couplings per node, 14 stored (offsets >= 0 in (z, y, x) order, the centre
// first), the other 13 read from the neighbour they couple to.
//
// Work-groups are 64 x 4 lanes (x contiguous across a wavefront) marching
// tz planes along z.  On the finest level the 3 x 3 x 3 block of phi and the
// 2 x 2 x 2 block of sigma a node needs are kept in registers from plane to
// plane, so a step loads one new plane of each.
#include <hip/hip_runtime.h>

#include "device.hpp"
#include "nodal.hpp"

namespace amrmg {

namespace {

__device__ __forceinline__ int pidx(const NdGeo& g, int x, int y, int z) {
  // padded element of unknown (x, y, z); x, y, z in [-1, m]
  return (x + 1) + g.px * ((y + 1) + g.py * (z + 1));
}

// Work-groups go to the 8 XCDs round robin (block b to XCD b % 8), and each
// XCD has its own L2.  The tiled kernels take their tile from a 1-D grid of
// 8 * ceil(n / 8) blocks so that every XCD runs one contiguous run of the
// tile order (x fastest, then y, then z): tiles that share halo rows and
// planes then share an L2.  A block past the last tile has no work.
constexpr int kNdXcds = 8;

__device__ __forceinline__ bool nd_tile(int ntx, int nty, int ntz, int& tx, int& ty, int& tz) {
  const int n = ntx * nty * ntz;
  const int per = (n + kNdXcds - 1) / kNdXcds;
  const int b = (int)blockIdx.x;
  const int t = (b % kNdXcds) * per + b / kNdXcds;
  if (t >= n) return false;
  tx = t % ntx;
  const int r = t / ntx;
  ty = r % nty;
  tz = r / nty;
  return true;
}

__device__ __forceinline__ int nd_ntx(const NdGeo& g) { return (g.mx + 63) / 64; }
__device__ __forceinline__ int nd_nty(const NdGeo& g) { return (g.my + 3) / 4; }
__device__ __forceinline__ int nd_ntz(const NdGeo& g) { return (g.mz + g.tz - 1) / g.tz; }

// Unsigned max of a per-lane value over the work-group, folded into way
// (blockIdx % kNdNormWays) of the slot at dst (skipped when the way already
// holds at least that value).
__device__ void nd_block_max(unsigned long long v, unsigned long long* dst) {
  const int nb = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
  dst += kNdNormStride * (nb % kNdNormWays);
  __shared__ unsigned long long red[16];
  for (int o = 32; o > 0; o >>= 1) {
    const unsigned long long w = (unsigned long long)__shfl_xor((long long)v, o);
    v = w > v ? w : v;
  }
  const int tid = threadIdx.x + blockDim.x * threadIdx.y;
  const int nw = (blockDim.x * blockDim.y + 63) / 64;
  if ((tid & 63) == 0) red[tid >> 6] = v;
  __syncthreads();
  if (tid == 0) {
    unsigned long long m = red[0];
    for (int w = 1; w < nw; ++w) m = red[w] > m ? red[w] : m;
    if (m > __hip_atomic_load(dst, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(dst, m);
  }
}

// The 14 stored offsets, centre first, then (z, y, x) lexicographic.
__device__ constexpr int kUp[kNdStored][3] = {
    {0, 0, 0},  {1, 0, 0},  {-1, 1, 0}, {0, 1, 0},  {1, 1, 0}, {-1, -1, 1}, {0, -1, 1},
    {1, -1, 1}, {-1, 0, 1}, {0, 0, 1},  {1, 0, 1},  {-1, 1, 1}, {0, 1, 1},  {1, 1, 1}};

// A phi at the centre of a 3 x 3 x 3 block P, from the 2 x 2 x 2 cells S around
// it: the coupling to a neighbour is kappa[pattern] times the sum of the cells
// that hold both nodes.
__device__ __forceinline__ double nd_apply0(const NdKappa& kap, const double (&P)[3][3][3],
                                            const double (&S)[2][2][2], double& diag) {
  double t[8] = {};
  double e[2][2], sum = 0.0;
  // faces, edges and corners off each plane of cells, pattern bit 2 (z)
#pragma unroll
  for (int cz = 0; cz < 2; ++cz) {
    const int z = 2 * cz;
    const double x0 = S[cz][0][0] + S[cz][1][0], x1 = S[cz][0][1] + S[cz][1][1];
    const double y0 = S[cz][0][0] + S[cz][0][1], y1 = S[cz][1][0] + S[cz][1][1];
    const double all = x0 + x1;
    e[cz][0] = x0;
    e[cz][1] = x1;
    sum += all;
    t[4] += all * P[z][1][1];
    t[5] += x0 * P[z][1][0];
    t[5] += x1 * P[z][1][2];
    t[6] += y0 * P[z][0][1];
    t[6] += y1 * P[z][2][1];
    t[7] += S[cz][0][0] * P[z][0][0];
    t[7] += S[cz][0][1] * P[z][0][2];
    t[7] += S[cz][1][0] * P[z][2][0];
    t[7] += S[cz][1][1] * P[z][2][2];
  }
  t[0] = sum * P[1][1][1];
  t[1] = (e[0][0] + e[1][0]) * P[1][1][0];
  t[1] += (e[0][1] + e[1][1]) * P[1][1][2];
#pragma unroll
  for (int cy = 0; cy < 2; ++cy) {
    const double a = S[0][cy][0] + S[1][cy][0], b = S[0][cy][1] + S[1][cy][1];
    t[2] += (a + b) * P[1][2 * cy][1];
    t[3] += a * P[1][2 * cy][0];
    t[3] += b * P[1][2 * cy][2];
  }
  diag = kap.k[0] * sum;
  double ap = 0.0;
#pragma unroll
  for (int q = 7; q >= 0; --q) ap += kap.k[q] * t[q];
  return ap;
}

// The value of the lane to the left (right) in the wavefront, `edge` in lane 0
// (63).
template <int CTRL>
__device__ __forceinline__ double lane_shift(double v, double edge) {
  const long long b = __double_as_longlong(v), e = __double_as_longlong(edge);
  const int lo = __builtin_amdgcn_update_dpp((int)e, (int)b, CTRL, 0xf, 0xf, false);
  const int hi =
      __builtin_amdgcn_update_dpp((int)(e >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_left(double v, double edge) {
  return lane_shift<0x138>(v, edge);  // wave_shr:1
}
__device__ __forceinline__ double from_right(double v, double edge) {
  return lane_shift<0x130>(v, edge);  // wave_shl:1
}
__device__ __forceinline__ double lane_of(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Finest-level sweep, see nd_launch_sweep0.  A wavefront is one row of 64 nodes:
// of a plane it loads its own three rows of phi and two of sigma, the
// neighbours along x come from the lanes beside (DPP), and one load of eight
// lanes brings what lies past the row's ends (lanes 2 r + 0 / 1: left and right
// of phi row r; lanes 6 + r: right of sigma row r).  Own loads of all thirteen
// values took 207 accesses of the L1 per row and step, half the time of the
// pass.  Now 134 MB an array four times in 140 us at 256^3 (Jacobi; 164 before,
// residual 162 -> 134 to 137, apply 141 -> 121), 3.8 TB/s.
// DOT: the block's part of phi . A phi (ND_APPLY) or f . out (ND_JACOBI).
template <int MODE, bool NORM, bool DOT>
__global__ void __launch_bounds__(256)
    k_nd_sweep0(NdGeo g, NdKappa kap, const double* __restrict__ sig,
                const double* __restrict__ phi, const double* __restrict__ f,
                double* __restrict__ out, double omega, unsigned long long* norm,
                double* __restrict__ part) {
  int tx, ty, tz;
  if (!nd_tile(nd_ntx(g), nd_nty(g), nd_ntz(g), tx, ty, tz)) {  // whole block
    if (DOT && threadIdx.x == 0 && threadIdx.y == 0) part[blockIdx.x] = 0.0;
    return;
  }
  const int lane = threadIdx.x;
  const int ux = tx * 64 + lane;
  const int uy = ty * 4 + threadIdx.y;
  const int z0 = tz * g.tz;
  unsigned long long mx = 0;
  double dot = 0.0;
  if (uy < g.my && z0 < g.mz) {  // whole wavefronts
    const int z1 = min(z0 + g.tz, g.mz);
    const int sx = g.mx + 1, sy = g.my + 1;  // sigma pitches
    // lanes past the row read its ghost, the last node's right neighbour
    const int xc = min(ux, g.mx);
    const int pz = g.px * g.py, sz = sx * sy;
    const double* const pp = phi + pidx(g, xc, uy - 1, 0);
    const double* const ss = sig + (xc + sx * uy);
    const double* const fp = f + pidx(g, xc, uy, 0);
    const int xr = min(tx * 64 + 64, g.mx);
    const double* ep = ss;
    int ez = 0;
    if (lane < 6) {
      ep = phi + pidx(g, lane & 1 ? xr : tx * 64 - 1, uy - 1 + (lane >> 1), 0);
      ez = pz;
    } else if (lane < 8) {
      ep = sig + (xr + sx * (uy + lane - 6));
      ez = sz;
    }
    double P[3][3][3];  // [z - uz + 1][y - uy + 1][x - ux + 1]
    double S[2][2][2];  // sigma of cells [z][y][x] = u + s
    struct Plane {
      double p[3], s[2], e;
    };
    // phi plane z, sigma plane zs and the ends of both
    auto load = [&](Plane& n, int z, int zs) {
      if (MODE != ND_ZERO) {
#pragma unroll
        for (int dy = 0; dy < 3; ++dy) n.p[dy] = pp[g.px * dy + pz * z];
      }
#pragma unroll
      for (int cy = 0; cy < 2; ++cy) n.s[cy] = ss[sx * cy + sz * zs];
      n.e = 0.0;
      if (lane < 8 && (MODE != ND_ZERO || lane >= 6)) n.e = ep[ez * (lane < 6 ? z : zs)];
    };
    auto spread_p = [&](double (&d)[3][3], const Plane& n) {
#pragma unroll
      for (int dy = 0; dy < 3; ++dy) {
        d[dy][0] = from_left(n.p[dy], lane_of(n.e, 2 * dy));
        d[dy][1] = n.p[dy];
        d[dy][2] = from_right(n.p[dy], lane_of(n.e, 2 * dy + 1));
      }
    };
    auto spread_s = [&](double (&d)[2][2], const Plane& n) {
#pragma unroll
      for (int cy = 0; cy < 2; ++cy) {
        d[cy][0] = n.s[cy];
        d[cy][1] = from_right(n.s[cy], lane_of(n.e, 6 + cy));
      }
    };
    Plane n;
    load(n, z0 - 1, z0);
    if (MODE != ND_ZERO) spread_p(P[1], n);
    spread_s(S[1], n);
    if (MODE != ND_ZERO) {
      Plane m;
      load(m, z0, z0);
      spread_p(P[2], m);
    }
    load(n, z0 + 1, z0 + 1);
    double fn = fp[pz * z0];
    for (int uz = z0; uz < z1; ++uz) {
      if (MODE != ND_ZERO) {
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
          for (int dx = 0; dx < 3; ++dx) {
            P[0][dy][dx] = P[1][dy][dx];
            P[1][dy][dx] = P[2][dy][dx];
          }
        spread_p(P[2], n);
      }
#pragma unroll
      for (int cy = 0; cy < 2; ++cy)
#pragma unroll
        for (int cx = 0; cx < 2; ++cx) S[0][cy][cx] = S[1][cy][cx];
      spread_s(S[1], n);
      const double fv = fn;
      // the next step's planes are loaded while this one's are worked on (past
      // the last step an in-range plane, not used)
      const int zn = min(uz + 2, g.mz);
      load(n, zn, zn);
      fn = fp[pz * min(uz + 1, g.mz)];
      double v;
      if (MODE == ND_ZERO) {
        double ssum = 0.0;
#pragma unroll
        for (int c = 0; c < 8; ++c) ssum += S[c >> 2][c >> 1 & 1][c & 1];
        v = omega * fv / (kap.k[0] * ssum);
      } else {
        double diag;
        const double ap = nd_apply0(kap, P, S, diag);
        const double r = fv - ap;
        if (NORM && ux < g.mx) {
          const unsigned long long b = absbits(r);
          mx = b > mx ? b : mx;
        }
        v = MODE == ND_RESID ? r : (MODE == ND_APPLY ? ap : P[1][1][1] + omega * r / diag);
      }
      if (ux < g.mx) {
        out[pidx(g, ux, uy, uz)] = v;
        if (DOT) dot += MODE == ND_APPLY ? P[1][1][1] * v : fv * v;
      }
    }
  }
  if (NORM) nd_block_max(mx, norm);
  if (DOT) {
    __shared__ double red[4];
    dot = wave_sum(dot);
    if (lane == 0) red[threadIdx.y] = dot;
    __syncthreads();
    if (lane == 0 && threadIdx.y == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
  }
}

// Coarse-level sweep (stored couplings), see nd_launch_sweep_st.
template <int MODE, bool NORM>
__global__ void __launch_bounds__(256)
    k_nd_sweep_st(NdGeo g, NdStencilC s, const double* __restrict__ phi,
                  const double* __restrict__ f, double* __restrict__ out, double omega,
                  unsigned long long* norm) {
  int tx, ty, tz;
  if (!nd_tile(nd_ntx(g), nd_nty(g), nd_ntz(g), tx, ty, tz)) return;  // whole block
  const int ux = tx * 64 + threadIdx.x;
  const int uy = ty * 4 + threadIdx.y;
  const int z0 = tz * g.tz;
  const bool act = ux < g.mx && uy < g.my && z0 < g.mz;
  unsigned long long mx = 0;
  if (act) {
    const int z1 = min(z0 + g.tz, g.mz);
    for (int uz = z0; uz < z1; ++uz) {
      const int c = pidx(g, ux, uy, uz);
      const double fv = f[c];
      const double diag = s.w[0][c];
      double v;
      if (MODE == ND_ZERO) {
        v = omega * fv / diag;
      } else {
        double ap = diag * phi[c];
#pragma unroll
        for (int q = 1; q < kNdStored; ++q) {
          const int d = kUp[q][0] + g.px * (kUp[q][1] + g.py * kUp[q][2]);
          ap += s.w[q][c] * phi[c + d];
          ap += s.w[q][c - d] * phi[c - d];
        }
        const double r = fv - ap;
        if (NORM) {
          const unsigned long long b = absbits(r);
          mx = b > mx ? b : mx;
        }
        v = MODE == ND_RESID ? r : (MODE == ND_APPLY ? ap : phi[c] + omega * r / diag);
      }
      out[c] = v;
    }
  }
  if (NORM) nd_block_max(mx, norm);
}

// Index along one direction of fine unknown 2 G + u for coarse unknown I
// (G = I + off, off = 1 on a Dirichlet direction), wrapped when periodic.
__device__ __forceinline__ int fine_of(int I, int u, bool per, int mf) {
  int q = 2 * I + (per ? 0 : 1) + u;
  if (per) q = q < 0 ? q + mf : (q >= mf ? q - mf : q);
  return q;
}

__device__ __forceinline__ double pw1(int t) { return t == 0 ? 1.0 : ((t == 1 || t == -1) ? 0.5 : 0.0); }

__global__ void __launch_bounds__(256)
    k_nd_restrict(NdGeo gf, NdGeo gc, const double* __restrict__ rf, double* __restrict__ rc) {
  int tx, ty, K;
  if (!nd_tile(nd_ntx(gc), nd_nty(gc), gc.mz, tx, ty, K)) return;
  const int I = tx * 64 + threadIdx.x;
  const int J = ty * 4 + threadIdx.y;
  if (I >= gc.mx || J >= gc.my) return;
  double acc = 0.0;
#pragma unroll
  for (int uz = -1; uz <= 1; ++uz) {
    const int z = fine_of(K, uz, gf.per & 4, gf.mz);
#pragma unroll
    for (int uy = -1; uy <= 1; ++uy) {
      const int y = fine_of(J, uy, gf.per & 2, gf.my);
#pragma unroll
      for (int ux = -1; ux <= 1; ++ux) {
        const int x = fine_of(I, ux, gf.per & 1, gf.mx);
        acc += (pw1(ux) * pw1(uy) * pw1(uz)) * rf[pidx(gf, x, y, z)];
      }
    }
  }
  rc[pidx(gc, I, J, K)] = acc * 0.125;
}

// One direction of the trilinear interpolation at fine unknown q: the coarse
// unknowns (ia, ib) and weights (wa, wb); a wall node gets weight 0.
__device__ __forceinline__ void interp1(int q, bool per, int mc, int& ia, int& ib, double& wa,
                                        double& wb) {
  const int G = q + (per ? 0 : 1);  // global fine node
  const int off = per ? 0 : 1;
  if ((G & 1) == 0) {
    ia = G / 2 - off;
    ib = ia;
    wa = 1.0;
    wb = 0.0;
  } else {
    ia = (G - 1) / 2 - off;
    ib = (G + 1) / 2 - off;
    wa = 0.5;
    wb = 0.5;
  }
  if (per) {
    ia = ia < 0 ? ia + mc : (ia >= mc ? ia - mc : ia);
    ib = ib < 0 ? ib + mc : (ib >= mc ? ib - mc : ib);
  } else {
    if (ia < 0 || ia >= mc) { wa = 0.0; ia = 0; }
    if (ib < 0 || ib >= mc) { wb = 0.0; ib = 0; }
  }
}

__global__ void __launch_bounds__(256)
    k_nd_interp_add(NdGeo gf, NdGeo gc, const double* __restrict__ ec, double* __restrict__ pf) {
  // lanes along x, gf.tz planes per work-group; every lane interpolates coarse
  // planes at its (x, y) from four values (a term of weight 0 reads a valid
  // node and adds 0 exactly, so neighbouring lanes of both parities take the
  // same path), a fine plane takes one of them or the mean of two, and the
  // upper one serves the next plane too (eight values for every fine node: 118 us
  // at 256^3 instead of 65, 13.5 at 128^3 instead of 9)
  int tx, ty, tz;
  if (!nd_tile(nd_ntx(gf), nd_nty(gf), nd_ntz(gf), tx, ty, tz)) return;
  const int x = tx * 64 + threadIdx.x;
  const int y = ty * 4 + threadIdx.y;
  const int z0 = tz * gf.tz;
  if (x >= gf.mx || y >= gf.my || z0 >= gf.mz) return;
  int ix[2], iy[2];
  double wx[2], wy[2];
  interp1(x, gf.per & 1, gc.mx, ix[0], ix[1], wx[0], wx[1]);
  interp1(y, gf.per & 2, gc.my, iy[0], iy[1], wy[0], wy[1]);
  const bool per = gf.per & 4;
  const int off = per ? 0 : 1;
  int at[2][2];
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int a = 0; a < 2; ++a) at[b][a] = pidx(gc, ix[a], iy[b], 0);
  const int pz = gc.px * gc.py;
  // the coarse plane of (even) global fine node 2 K, 0 past a wall
  auto plane = [&](int K) -> double {
    K -= off;
    if (per) K = K < 0 ? K + gc.mz : (K >= gc.mz ? K - gc.mz : K);
    const bool in = K >= 0 && K < gc.mz;
    const int o = in ? pz * K : 0;
    double v = 0.0;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int a = 0; a < 2; ++a) v += (wx[a] * wy[b]) * ec[at[b][a] + o];
    return in ? v : 0.0;
  };
  const int z1 = min(z0 + gf.tz, gf.mz);
  double lo = plane((z0 + off) >> 1);
  double* p = pf + pidx(gf, x, y, z0);
  for (int z = z0; z < z1; ++z, p += gf.px * gf.py) {
    const int G = z + off;
    if (G & 1) {
      const double hi = plane((G + 1) >> 1);
      *p += 0.5 * lo + 0.5 * hi;
      lo = hi;
    } else {
      *p += lo;
    }
  }
}

// Ghosts of direction d from the opposite valid layer; grid covers the
// padded extent of the other two directions.
__global__ void __launch_bounds__(256) k_nd_fill_ghosts(NdGeo g, double* a, int d) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  const int pz = g.mz + 2;
  int n1, n2;
  if (d == 0) { n1 = g.py; n2 = pz; }
  else if (d == 1) { n1 = g.px; n2 = pz; }
  else { n1 = g.px; n2 = g.py; }
  if (i >= n1 * n2) return;
  const int p = i % n1, q = i / n1;
  const int m = d == 0 ? g.mx : (d == 1 ? g.my : g.mz);
  auto at = [&](int t) -> int {
    // padded coordinates: t along d, (p, q) along the others
    if (d == 0) return t + g.px * (p + g.py * q);
    if (d == 1) return p + g.px * (t + g.py * q);
    return p + g.px * (q + g.py * t);
  };
  a[at(0)] = a[at(m)];
  a[at(m + 1)] = a[at(1)];
}

// Galerkin product: for coarse node (I, J, K) and each stored offset o,
// 1/8 sum_u r(u) sum_v W_f(2I + u, v) P(u + v - 2o).  FROM_SIGMA: W_f from
// the finest level's cells; else from the finer level's stored couplings.
template <bool FROM_SIGMA>
__global__ void __launch_bounds__(256)
    k_nd_rap(NdGeo gf, NdGeo gc, NdKappa kap, const double* __restrict__ sig, NdStencilC in,
             NdStencil out) {
  const int I = blockIdx.x * 64 + threadIdx.x;
  const int J = blockIdx.y * 4 + threadIdx.y;
  const int K = blockIdx.z;
  if (I >= gc.mx || J >= gc.my || K >= gc.mz) return;
  double acc[kNdStored];
#pragma unroll
  for (int q = 0; q < kNdStored; ++q) acc[q] = 0.0;
  const int sx = gf.mx + 1, sy = gf.my + 1;
  for (int u = 0; u < 27; ++u) {
    const int ux = u % 3 - 1, uy = (u / 3) % 3 - 1, uz = u / 9 - 1;
    const int x = fine_of(I, ux, gf.per & 1, gf.mx);
    const int y = fine_of(J, uy, gf.per & 2, gf.my);
    const int z = fine_of(K, uz, gf.per & 4, gf.mz);
    const double ru = pw1(ux) * pw1(uy) * pw1(uz);
    // the fine node's 27 couplings W[v], v = (vx, vy, vz) + 1 indexed vz*9 + vy*3 + vx
    double W[27];
    if (FROM_SIGMA) {
      double S[2][2][2];
#pragma unroll
      for (int cz = 0; cz < 2; ++cz)
#pragma unroll
        for (int cy = 0; cy < 2; ++cy)
#pragma unroll
          for (int cx = 0; cx < 2; ++cx)
            S[cz][cy][cx] = sig[(x + cx) + sx * ((y + cy) + sy * (z + cz))];
#pragma unroll
      for (int v = 0; v < 27; ++v) {
        const int vx = v % 3 - 1, vy = (v / 3) % 3 - 1, vz = v / 9 - 1;
        // cells holding both the node and node + v: s_d = 0 for v_d = -1,
        // 1 for v_d = 1, either for v_d = 0
        double ss = 0.0;
#pragma unroll
        for (int cz = 0; cz < 2; ++cz)
#pragma unroll
          for (int cy = 0; cy < 2; ++cy)
#pragma unroll
            for (int cx = 0; cx < 2; ++cx) {
              const bool ok = (vx == 0 || vx == 2 * cx - 1) && (vy == 0 || vy == 2 * cy - 1) &&
                              (vz == 0 || vz == 2 * cz - 1);
              if (ok) ss += S[cz][cy][cx];
            }
        const int pat = (vx != 0 ? 1 : 0) | (vy != 0 ? 2 : 0) | (vz != 0 ? 4 : 0);
        W[v] = kap.k[pat] * ss;
      }
    } else {
      const int c = pidx(gf, x, y, z);
#pragma unroll
      for (int q = 0; q < kNdStored; ++q) {
        const int vx = kUp[q][0], vy = kUp[q][1], vz = kUp[q][2];
        const int d = vx + gf.px * (vy + gf.py * vz);
        W[(vz + 1) * 9 + (vy + 1) * 3 + (vx + 1)] = in.w[q][c];
        if (q > 0) W[(1 - vz) * 9 + (1 - vy) * 3 + (1 - vx)] = in.w[q][c - d];
      }
    }
#pragma unroll
    for (int q = 0; q < kNdStored; ++q) {
      const int ox = kUp[q][0], oy = kUp[q][1], oz = kUp[q][2];
      double t = 0.0;
#pragma unroll
      for (int v = 0; v < 27; ++v) {
        const int vx = v % 3 - 1, vy = (v / 3) % 3 - 1, vz = v / 9 - 1;
        const double p = pw1(ux + vx - 2 * ox) * pw1(uy + vy - 2 * oy) * pw1(uz + vz - 2 * oz);
        t += p * W[v];
      }
      acc[q] += ru * t;
    }
  }
  const int c = pidx(gc, I, J, K);
#pragma unroll
  for (int q = 0; q < kNdStored; ++q) out.w[q][c] = acc[q] * 0.125;
}

// Block-wide sum in FP64 (all threads get the result).
__device__ double nd_block_sum(double v, double* red) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double s = 0.0;
  for (int i = 0; i < nw; ++i) s += red[i];
  return s;
}

// q = A p on the bottom level (wrapped neighbours; walls skipped).
__device__ double nd_apply_at(const NdGeo& g, const NdStencilC& s, const double* p, int ux, int uy,
                              int uz) {
  const int c = pidx(g, ux, uy, uz);
  double ap = s.w[0][c] * p[c];
  for (int q = 1; q < kNdStored; ++q) {
    const int d = kUp[q][0] + g.px * (kUp[q][1] + g.py * kUp[q][2]);
    ap += s.w[q][c] * p[c + d];
    ap += s.w[q][c - d] * p[c - d];
  }
  return ap;
}

// Whole CG in one work-group of 1024 lanes.  x, r, p, q live in padded
// arrays whose ghosts the work-group keeps wrapped (periodic) or 0 (walls).
__global__ void __launch_bounds__(1024)
    k_nd_bottom_cg(NdGeo g, NdStencilC s, const double* __restrict__ rhs, double* x, double* r,
                   double* p, double* q, double tol, int maxit, int singular, int* iters) {
  __shared__ double red[16];
  const int n = g.mx * g.my * g.mz;
  const int tid = threadIdx.x, nt = blockDim.x;
  auto node = [&](int i, int& ux, int& uy, int& uz) {
    ux = i % g.mx;
    uy = (i / g.mx) % g.my;
    uz = i / (g.mx * g.my);
  };
  auto wrap_fill = [&](double* a) {
    // ghosts along periodic directions, one direction after the other
    for (int d = 0; d < 3; ++d) {
      if (!(g.per & (1 << d))) continue;
      __syncthreads();
      const int pz = g.mz + 2;
      const int n1 = d == 0 ? g.py : g.px;
      const int n2 = d == 2 ? g.py : pz;
      const int m = d == 0 ? g.mx : (d == 1 ? g.my : g.mz);
      for (int i = tid; i < n1 * n2; i += nt) {
        const int pp = i % n1, qq = i / n1;
        int lo, hi, slo, shi;
        if (d == 0) {
          lo = 0 + g.px * (pp + g.py * qq);
          hi = (m + 1) + g.px * (pp + g.py * qq);
          slo = m + g.px * (pp + g.py * qq);
          shi = 1 + g.px * (pp + g.py * qq);
        } else if (d == 1) {
          lo = pp + g.px * (0 + g.py * qq);
          hi = pp + g.px * ((m + 1) + g.py * qq);
          slo = pp + g.px * (m + g.py * qq);
          shi = pp + g.px * (1 + g.py * qq);
        } else {
          lo = pp + g.px * (qq + g.py * 0);
          hi = pp + g.px * (qq + g.py * (m + 1));
          slo = pp + g.px * (qq + g.py * m);
          shi = pp + g.px * (qq + g.py * 1);
        }
        a[lo] = a[slo];
        a[hi] = a[shi];
      }
    }
    __syncthreads();
  };
  // b = rhs (mean removed when singular); x = 0; r = p = b
  double mean = 0.0;
  if (singular) {
    double sm = 0.0;
    for (int i = tid; i < n; i += nt) {
      int ux, uy, uz;
      node(i, ux, uy, uz);
      sm += rhs[pidx(g, ux, uy, uz)];
    }
    mean = nd_block_sum(sm, red) / n;
  }
  double bb = 0.0;
  for (int i = tid; i < n; i += nt) {
    int ux, uy, uz;
    node(i, ux, uy, uz);
    const int c = pidx(g, ux, uy, uz);
    const double b = rhs[c] - mean;
    x[c] = 0.0;
    r[c] = b;
    p[c] = b;
    bb += b * b;
  }
  double rr = nd_block_sum(bb, red);
  const double nb = sqrt(rr);
  wrap_fill(p);
  int it = 0;
  while (nb > 0.0 && it < maxit && sqrt(rr) > tol * nb) {
    double pq = 0.0;
    for (int i = tid; i < n; i += nt) {
      int ux, uy, uz;
      node(i, ux, uy, uz);
      const int c = pidx(g, ux, uy, uz);
      const double v = nd_apply_at(g, s, p, ux, uy, uz);
      q[c] = v;
      pq += p[c] * v;
    }
    pq = nd_block_sum(pq, red);
    const double alpha = rr / pq;
    double rn = 0.0;
    for (int i = tid; i < n; i += nt) {
      int ux, uy, uz;
      node(i, ux, uy, uz);
      const int c = pidx(g, ux, uy, uz);
      x[c] += alpha * p[c];
      r[c] -= alpha * q[c];
      rn += r[c] * r[c];
    }
    rn = nd_block_sum(rn, red);
    const double beta = rn / rr;
    rr = rn;
    for (int i = tid; i < n; i += nt) {
      int ux, uy, uz;
      node(i, ux, uy, uz);
      const int c = pidx(g, ux, uy, uz);
      p[c] = r[c] + beta * p[c];
    }
    wrap_fill(p);
    ++it;
  }
  if (singular) {
    double sm = 0.0;
    for (int i = tid; i < n; i += nt) {
      int ux, uy, uz;
      node(i, ux, uy, uz);
      sm += x[pidx(g, ux, uy, uz)];
    }
    const double mx = nd_block_sum(sm, red) / n;
    for (int i = tid; i < n; i += nt) {
      int ux, uy, uz;
      node(i, ux, uy, uz);
      x[pidx(g, ux, uy, uz)] -= mx;
    }
  }
  if (tid == 0) *iters = it;
}

// ---------------------------------------------------------------------------
// A small level's half of a cycle in one launch, nu1 = nu2 = 2.  A work-group
// takes a tile of the level and recomputes a rim of one node per remaining
// pass, so that the passes need only LDS between them.  Bound by latency and by the
// couplings, which come from the L2 once per pass and node; the tiles are
// small (2^3 coarse nodes, 4^3 nodes), so that a level of 31^3 fills the chip:
// 10 us down and 8 up there, 7 and 6 at 15^3, where the four and three launches
// they replace took 14 to 18 and 12 to 15.

// Regions may be longer than a small periodic level.
__device__ __forceinline__ int wrapped(int x, int m) {
  while (x < 0) x += m;
  while (x >= m) x -= m;
  return x;
}

// Node q of a region of NX x NY x NZ nodes that starts at (x0, y0, z0):
// its padded element, wrapped along periodic directions, -1 past a wall.
template <int NX, int NY>
__device__ __forceinline__ int region_at(const NdGeo& g, int x0, int y0, int z0, int q) {
  int x = x0 + q % NX, y = y0 + q / NX % NY, z = z0 + q / (NX * NY);
  if (g.per & 1) x = wrapped(x, g.mx);
  if (g.per & 2) y = wrapped(y, g.my);
  if (g.per & 4) z = wrapped(z, g.mz);
  const bool in = x >= 0 && x < g.mx && y >= 0 && y < g.my && z >= 0 && z < g.mz;
  return in ? pidx(g, x, y, z) : -1;
}

// A v at padded element c; v: the node's place in an LDS region of row and
// plane pitch NX, NX * NY that holds its neighbours.
template <int NX, int NY>
__device__ __forceinline__ double region_apply(const NdGeo& g, const NdStencilC& s, int c,
                                               double diag, const double* v) {
  double ap = diag * v[0];
#pragma unroll
  for (int q = 1; q < kNdStored; ++q) {
    const int d = kUp[q][0] + g.px * (kUp[q][1] + g.py * kUp[q][2]);
    const int l = kUp[q][0] + NX * (kUp[q][1] + NY * kUp[q][2]);
    ap += s.w[q][c] * v[l];
    ap += s.w[q][c - d] * v[-l];
  }
  return ap;
}

// Two sweeps from zero, residual, restriction: x = the level's iterate, fc =
// the coarser level's right-hand side.  Tile: TX x TY x TZ coarse nodes.
template <int TX, int TY, int TZ>
__global__ void __launch_bounds__(256)
    k_nd_down(NdGeo g, NdGeo gc, int ntx, int nty, NdStencilC s, const double* __restrict__ f,
              double* __restrict__ x, double* __restrict__ fc, double omega) {
  constexpr int RX = 2 * TX + 1, RY = 2 * TY + 1, RZ = 2 * TZ + 1;  // residual
  constexpr int BX = RX + 2, BY = RY + 2, BZ = RZ + 2;              // second sweep
  constexpr int AX = RX + 4, AY = RY + 4, AZ = RZ + 4;              // first sweep
  __shared__ double A[AX * AY * AZ], B[BX * BY * BZ];
  double* const R = A;
  const int t = blockIdx.x;
  const int I0 = t % ntx * TX, J0 = t / ntx % nty * TY, K0 = t / (ntx * nty) * TZ;
  // first node of the residual's region: left of coarse node I0
  const int x0 = 2 * I0 + (g.per & 1 ? 0 : 1) - 1, y0 = 2 * J0 + (g.per & 2 ? 0 : 1) - 1,
            z0 = 2 * K0 + (g.per & 4 ? 0 : 1) - 1;
  for (int q = threadIdx.x; q < AX * AY * AZ; q += 256) {
    const int c = region_at<AX, AY>(g, x0 - 2, y0 - 2, z0 - 2, q);
    A[q] = c >= 0 ? omega * f[c] / s.w[0][c] : 0.0;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < BX * BY * BZ; q += 256) {
    const int c = region_at<BX, BY>(g, x0 - 1, y0 - 1, z0 - 1, q);
    double v = 0.0;
    if (c >= 0) {
      const int bx = q % BX, by = q / BX % BY, bz = q / (BX * BY);
      const double* a = A + (bx + 1) + AX * ((by + 1) + AY * (bz + 1));
      const double diag = s.w[0][c];
      const double r = f[c] - region_apply<AX, AY>(g, s, c, diag, a);
      v = a[0] + omega * r / diag;
    }
    B[q] = v;
  }
  __syncthreads();
  // the tile's own nodes: [x0 + 1, x0 + 2 TX] and so on, the first node of the
  // level along a wall (x0 = 0) and the last ones with the end tiles
  const bool ex = I0 + TX >= gc.mx, ey = J0 + TY >= gc.my, ez = K0 + TZ >= gc.mz;
  for (int q = threadIdx.x; q < RX * RY * RZ; q += 256) {
    const int rx = q % RX, ry = q / RX % RY, rz = q / (RX * RY);
    const int c = region_at<RX, RY>(g, x0, y0, z0, q);
    double r = 0.0;
    if (c >= 0) {
      const double* b = B + (rx + 1) + BX * ((ry + 1) + BY * (rz + 1));
      r = f[c] - region_apply<BX, BY>(g, s, c, s.w[0][c], b);
      // the tile's own nodes: from its first coarse node's left neighbour on
      // along walls (the level's first node is one), from the coarse node on
      // along periodic directions (never a wrapped one)
      const int ux = x0 + rx, uy = y0 + ry, uz = z0 + rz;
      const bool own = ((g.per & 1) ? rx > 0 && ux < g.mx : rx < 2 * TX || ex) &&
                       ((g.per & 2) ? ry > 0 && uy < g.my : ry < 2 * TY || ey) &&
                       ((g.per & 4) ? rz > 0 && uz < g.mz : rz < 2 * TZ || ez);
      if (own) x[c] = b[0];
    }
    R[q] = r;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < TX * TY * TZ; q += 256) {
    const int cx = q % TX, cy = q / TX % TY, cz = q / (TX * TY);
    if (I0 + cx >= gc.mx || J0 + cy >= gc.my || K0 + cz >= gc.mz) continue;
    const double* r = R + (2 * cx + 1) + RX * ((2 * cy + 1) + RY * (2 * cz + 1));
    double acc = 0.0;
#pragma unroll
    for (int uz = -1; uz <= 1; ++uz)
#pragma unroll
      for (int uy = -1; uy <= 1; ++uy)
#pragma unroll
        for (int ux = -1; ux <= 1; ++ux)
          acc += (pw1(ux) * pw1(uy) * pw1(uz)) * r[ux + RX * (uy + RY * uz)];
    fc[pidx(gc, I0 + cx, J0 + cy, K0 + cz)] = acc * 0.125;
  }
}

// Coarse correction added, then two sweeps: out = the level's iterate.  Tile:
// TX x TY x TZ nodes.
template <int TX, int TY, int TZ>
__global__ void __launch_bounds__(256)
    k_nd_up(NdGeo g, NdGeo gc, int ntx, int nty, NdStencilC s, const double* __restrict__ f,
            const double* __restrict__ x, const double* __restrict__ ec,
            double* __restrict__ out, double omega) {
  constexpr int BX = TX + 2, BY = TY + 2, BZ = TZ + 2;
  constexpr int AX = TX + 4, AY = TY + 4, AZ = TZ + 4;
  __shared__ double A[AX * AY * AZ], B[BX * BY * BZ];
  const int t = blockIdx.x;
  const int x0 = t % ntx * TX, y0 = t / ntx % nty * TY, z0 = t / (ntx * nty) * TZ;
  for (int q = threadIdx.x; q < AX * AY * AZ; q += 256) {
    const int c = region_at<AX, AY>(g, x0 - 2, y0 - 2, z0 - 2, q);
    double v = 0.0;
    if (c >= 0) {
      const int cx = c % g.px - 1, cy = c / g.px % g.py - 1, cz = c / (g.px * g.py) - 1;
      int ix[2], iy[2], iz[2];
      double wx[2], wy[2], wz[2];
      interp1(cx, g.per & 1, gc.mx, ix[0], ix[1], wx[0], wx[1]);
      interp1(cy, g.per & 2, gc.my, iy[0], iy[1], wy[0], wy[1]);
      interp1(cz, g.per & 4, gc.mz, iz[0], iz[1], wz[0], wz[1]);
      double p[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        p[k] = 0.0;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int a = 0; a < 2; ++a) p[k] += (wx[a] * wy[b]) * ec[pidx(gc, ix[a], iy[b], iz[k])];
      }
      v = x[c] + (wz[0] * p[0] + wz[1] * p[1]);
    }
    A[q] = v;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < BX * BY * BZ; q += 256) {
    const int c = region_at<BX, BY>(g, x0 - 1, y0 - 1, z0 - 1, q);
    double v = 0.0;
    if (c >= 0) {
      const int bx = q % BX, by = q / BX % BY, bz = q / (BX * BY);
      const double* a = A + (bx + 1) + AX * ((by + 1) + AY * (bz + 1));
      const double diag = s.w[0][c];
      const double r = f[c] - region_apply<AX, AY>(g, s, c, diag, a);
      v = a[0] + omega * r / diag;
    }
    B[q] = v;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < TX * TY * TZ; q += 256) {
    const int ux = x0 + q % TX, uy = y0 + q / TX % TY, uz = z0 + q / (TX * TY);
    if (ux >= g.mx || uy >= g.my || uz >= g.mz) continue;
    const int c = pidx(g, ux, uy, uz);
    const double* b = B + (q % TX + 1) + BX * ((q / TX % TY + 1) + BY * (q / (TX * TY) + 1));
    const double diag = s.w[0][c];
    const double r = f[c] - region_apply<BX, BY>(g, s, c, diag, b);
    out[c] = b[0] + omega * r / diag;
  }
}

// ---------------------------------------------------------------------------
// The tail (nd_launch_tail).  A lane owns one node of a level; its couplings are
// loaded once for the way down and once for the way up, what it reads of its
// neighbours is in LDS, so a pass is 27 LDS reads and a barrier.

template <typename P>
__device__ __forceinline__ P* nd_global(P* p) {
  return (P*)(__attribute__((address_space(1))) P*)p;
}

// The level's LDS arrays: right-hand side and two iterates, padded by the wall
// nodes (zeros).  Periodic neighbours are wrapped in the index, not copied.
struct NdTailNode {
  bool on;
  int c;                       // element of an LDS array, and of the level's own arrays
  int ox[3], oy[3], oz[3];     // element offsets to the neighbours -1, 0, 1
  double w[27];                // couplings by (z + 1) 9 + (y + 1) 3 + (x + 1)
};

__device__ __forceinline__ void nd_tail_place(NdTailNode& n, const NdGeo& g, int i) {
  n.on = i < g.mx * g.my * g.mz;
  const int x = n.on ? i % g.mx : 0, y = n.on ? i / g.mx % g.my : 0,
            z = n.on ? i / (g.mx * g.my) : 0;
  n.c = pidx(g, x, y, z);
  const int py = g.px, pz = g.px * g.py;
  n.ox[0] = x == 0 && (g.per & 1) ? g.mx - 1 : -1;
  n.ox[2] = x == g.mx - 1 && (g.per & 1) ? 1 - g.mx : 1;
  n.oy[0] = y == 0 && (g.per & 2) ? (g.my - 1) * py : -py;
  n.oy[2] = y == g.my - 1 && (g.per & 2) ? (1 - g.my) * py : py;
  n.oz[0] = z == 0 && (g.per & 4) ? (g.mz - 1) * pz : -pz;
  n.oz[2] = z == g.mz - 1 && (g.per & 4) ? (1 - g.mz) * pz : pz;
  n.ox[1] = n.oy[1] = n.oz[1] = 0;
}

__device__ __forceinline__ void nd_tail_load(NdTailNode& n, const NdTail* tp, int l) {
  const NdGeo g = tp->lev[l].g;
#pragma unroll
  for (int q = 0; q < kNdStored; ++q) {
    const double* w = nd_global(tp->lev[l].w.w[q]);
    const int d = kUp[q][0] + g.px * (kUp[q][1] + g.py * kUp[q][2]);
    const int k = 13 + kUp[q][0] + 3 * kUp[q][1] + 9 * kUp[q][2];
    n.w[k] = n.on ? w[n.c] : 0.0;
    if (q > 0) n.w[26 - k] = n.on ? w[n.c - d] : 0.0;
  }
}

__device__ __forceinline__ double nd_tail_apply(const NdTailNode& n, const double* v) {
  double ap = n.w[13] * v[n.c];
#pragma unroll
  for (int q = 1; q < kNdStored; ++q) {
    const int x = kUp[q][0], y = kUp[q][1], z = kUp[q][2], k = 13 + x + 3 * y + 9 * z;
    ap += n.w[k] * v[n.c + n.ox[1 + x] + n.oy[1 + y] + n.oz[1 + z]];
    ap += n.w[26 - k] * v[n.c + n.ox[1 - x] + n.oy[1 - y] + n.oz[1 - z]];
  }
  return ap;
}

__device__ __forceinline__ int nd_padded(const NdGeo& g) { return g.px * g.py * (g.mz + 2); }

// Sum over the work-group; one wavefront needs no barrier.
template <bool ONE>
__device__ __forceinline__ double nd_tail_sum(double v, double* red, int& phase) {
  return ONE ? wave_sum(v) : block_sum_w<true>(v, red, phase, (blockDim.x + 63) / 64);
}

// CG from zero on the bottom: p in LDS (padded), the rest in registers.  ONE: at
// most 64 nodes, wavefront 0 alone.
template <bool ONE>
__device__ __forceinline__ void nd_tail_cg(const NdTail* tp, const double* f, double* x, double* p,
                                           double* red) {
  const NdGeo g = tp->lev[tp->nlev].g;
  const int nn = g.mx * g.my * g.mz;
  NdTailNode n;
  nd_tail_place(n, g, threadIdx.x);
  nd_tail_load(n, tp, tp->nlev);
  int phase = 0;
  auto sync = [&]() {
    if (ONE) {
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    } else {
      __syncthreads();
    }
  };
  double b = n.on ? f[n.c] : 0.0, xv = 0.0;
  if (tp->singular) {
    const double m = nd_tail_sum<ONE>(b, red, phase) / nn;
    b = n.on ? b - m : 0.0;
  }
  double r = b, pv = b;
  double rr = nd_tail_sum<ONE>(r * r, red, phase);
  const double nb = sqrt(rr), tol = tp->tol;
  const int maxit = tp->maxit;
  int it = 0;
  while (nb > 0.0 && it < maxit && sqrt(rr) > tol * nb) {
    if (n.on) p[n.c] = pv;
    sync();
    const double q = n.on ? nd_tail_apply(n, p) : 0.0;
    // (the sum's barrier also keeps the next p from the lanes still reading)
    const double alpha = rr / nd_tail_sum<ONE>(pv * q, red, phase);
    xv += alpha * pv;
    r -= alpha * q;
    const double rn = nd_tail_sum<ONE>(r * r, red, phase);
    const double beta = rn / rr;
    rr = rn;
    pv = r + beta * pv;
    if (ONE) sync();
    ++it;
  }
  if (tp->singular) xv -= nd_tail_sum<ONE>(xv, red, phase) / nn;
  if (n.on) x[n.c] = xv;
  if (threadIdx.x == 0) *nd_global(tp->iters) = it;
}

template <int NT>
__global__ void __launch_bounds__(NT) k_nd_tail(const NdTail* __restrict__ tp) {
  extern __shared__ __align__(16) double nd_lds[];
  __shared__ double red[32];
  const int tid = threadIdx.x, nlev = tp->nlev;
  auto base = [&](int l) {
    int o = 0;
    for (int m = 0; m < l; ++m) o += 3 * nd_padded(tp->lev[m].g);
    return nd_lds + o;
  };
  {
    const int all = (int)(base(nlev + 1) - nd_lds);
    for (int e = tid; e < all; e += NT) nd_lds[e] = 0.0;
    __syncthreads();
    NdTailNode n;
    nd_tail_place(n, tp->lev[0].g, tid);
    if (n.on) nd_lds[n.c] = nd_global(tp->lev[0].f)[n.c];
    __syncthreads();
  }
  const double om = tp->omega;
  for (int l = 0; l < nlev; ++l) {
    const NdGeo g = tp->lev[l].g, gc = tp->lev[l + 1].g;
    const int pad = nd_padded(g);
    double* const f = base(l);
    double* x = f + pad;
    double* y = x + pad;
    NdTailNode n;
    nd_tail_place(n, g, tid);
    nd_tail_load(n, tp, l);
    const double fv = n.on ? f[n.c] : 0.0;
    if (n.on) x[n.c] = om * fv / n.w[13];
    __syncthreads();
    for (int k = 1; k < tp->nu1; ++k) {
      if (n.on) y[n.c] = x[n.c] + om * (fv - nd_tail_apply(n, x)) / n.w[13];
      __syncthreads();
      double* const t = x;
      x = y;
      y = t;
    }
    if (n.on) y[n.c] = fv - nd_tail_apply(n, x);
    __syncthreads();
    NdTailNode m;
    nd_tail_place(m, gc, tid);
    if (m.on) {
      const int I = tid % gc.mx, J = tid / gc.mx % gc.my, K = tid / (gc.mx * gc.my);
      double acc = 0.0;
#pragma unroll
      for (int uz = -1; uz <= 1; ++uz)
#pragma unroll
        for (int uy = -1; uy <= 1; ++uy)
#pragma unroll
          for (int ux = -1; ux <= 1; ++ux)
            acc += (pw1(ux) * pw1(uy) * pw1(uz)) *
                   y[pidx(g, fine_of(I, ux, g.per & 1, g.mx), fine_of(J, uy, g.per & 2, g.my),
                          fine_of(K, uz, g.per & 4, g.mz))];
      base(l + 1)[m.c] = acc * 0.125;
    }
    __syncthreads();
  }
  {
    double* const f = base(nlev);
    const int pad = nd_padded(tp->lev[nlev].g);
    const NdGeo g = tp->lev[nlev].g;
    if (g.mx * g.my * g.mz <= 64) {
      if (tid < 64) nd_tail_cg<true>(tp, f, f + pad, f + 2 * pad, red);
    } else {
      nd_tail_cg<false>(tp, f, f + pad, f + 2 * pad, red);
    }
    __syncthreads();
  }
  // the iterate of a level is x after an odd number of sweeps down, else y
  double* e = base(nlev) + nd_padded(tp->lev[nlev].g);
  for (int l = nlev - 1; l >= 0; --l) {
    const NdGeo g = tp->lev[l].g, gc = tp->lev[l + 1].g;
    const int pad = nd_padded(g);
    double* const f = base(l);
    double* x = f + pad;
    double* y = x + pad;
    if (tp->nu1 % 2 == 0) {
      double* const t = x;
      x = y;
      y = t;
    }
    NdTailNode n;
    nd_tail_place(n, g, tid);
    nd_tail_load(n, tp, l);
    const double fv = n.on ? f[n.c] : 0.0;
    double v = 0.0;
    if (n.on) {
      int ix[2], iy[2], iz[2];
      double wx[2], wy[2], wz[2];
      interp1(tid % g.mx, g.per & 1, gc.mx, ix[0], ix[1], wx[0], wx[1]);
      interp1(tid / g.mx % g.my, g.per & 2, gc.my, iy[0], iy[1], wy[0], wy[1]);
      interp1(tid / (g.mx * g.my), g.per & 4, gc.mz, iz[0], iz[1], wz[0], wz[1]);
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int a = 0; a < 2; ++a)
            v += (wx[a] * wy[b] * wz[c]) * e[pidx(gc, ix[a], iy[b], iz[c])];
      x[n.c] += v;
    }
    __syncthreads();
    for (int k = 0; k < tp->nu2; ++k) {
      if (n.on) y[n.c] = x[n.c] + om * (fv - nd_tail_apply(n, x)) / n.w[13];
      __syncthreads();
      double* const t = x;
      x = y;
      y = t;
    }
    e = x;
  }
  NdTailNode n;
  nd_tail_place(n, tp->lev[0].g, tid);
  if (n.on) nd_global(tp->lev[0].x)[n.c] = e[n.c];
}

__global__ void __launch_bounds__(256)
    k_nd_maxabs(NdGeo g, const double* __restrict__ v, unsigned long long* norm) {
  const int ux = blockIdx.x * 64 + threadIdx.x;
  const int uy = blockIdx.y * 4 + threadIdx.y;
  const int z0 = blockIdx.z * g.tz;
  unsigned long long mx = 0;
  if (ux < g.mx && uy < g.my) {
    const int z1 = min(z0 + g.tz, g.mz);
    for (int uz = z0; uz < z1; ++uz) {
      const unsigned long long b = absbits(v[pidx(g, ux, uy, uz)]);
      mx = b > mx ? b : mx;
    }
  }
  nd_block_max(mx, norm);
}

// Unknown index along d of global node G (relative to the domain), or -1 on
// a wall node; periodic directions wrap.
__device__ __forceinline__ int unknown_of(int G, int n, bool per) {
  if (per) return ((G % n) + n) % n;
  return (G <= 0 || G >= n) ? -1 : G - 1;
}

// grid.y = box; x covers the box's nodes (lo..hi+1 grown by ng)
__global__ void __launch_bounds__(256)
    k_nd_gather(NdGeo g, const NdBox* __restrict__ boxes, int ng, int3 dlo,
                const double* __restrict__ src, double* __restrict__ dst) {
  const NdBox B = boxes[blockIdx.y];
  const int nx = B.hi[0] - B.lo[0] + 2 + 2 * ng, ny = B.hi[1] - B.lo[1] + 2 + 2 * ng;
  const int nz = B.hi[2] - B.lo[2] + 2 + 2 * ng;
  const long long total = (long long)nx * ny * nz;
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < total; e += 256ll * gridDim.x) {
    const int i = (int)(e % nx), j = (int)((e / nx) % ny), k = (int)(e / ((long long)nx * ny));
    // global node of this element; the box owns the nodes of its own cells
    const int G[3] = {B.lo[0] - ng + i, B.lo[1] - ng + j, B.lo[2] - ng + k};
    if (G[0] < B.lo[0] || G[0] > B.hi[0] || G[1] < B.lo[1] || G[1] > B.hi[1] || G[2] < B.lo[2] ||
        G[2] > B.hi[2])
      continue;
    const int u[3] = {G[0] - dlo.x - ((g.per & 1) ? 0 : 1), G[1] - dlo.y - ((g.per & 2) ? 0 : 1),
                      G[2] - dlo.z - ((g.per & 4) ? 0 : 1)};
    if (u[0] < 0 || u[1] < 0 || u[2] < 0) continue;  // wall node
    dst[pidx(g, u[0], u[1], u[2])] = src[B.off + e];
  }
}

__global__ void __launch_bounds__(256)
    k_nd_scatter(NdGeo g, const NdBox* __restrict__ boxes, int ng, int3 dlo, int3 dn,
                 const double* __restrict__ src, double* __restrict__ dst) {
  const NdBox B = boxes[blockIdx.y];
  const int nx = B.hi[0] - B.lo[0] + 2 + 2 * ng, ny = B.hi[1] - B.lo[1] + 2 + 2 * ng;
  const int nz = B.hi[2] - B.lo[2] + 2 + 2 * ng;
  const long long total = (long long)nx * ny * nz;
  const int n[3] = {dn.x, dn.y, dn.z};
  const int lo[3] = {dlo.x, dlo.y, dlo.z};
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < total; e += 256ll * gridDim.x) {
    const int i = (int)(e % nx), j = (int)((e / nx) % ny), k = (int)(e / ((long long)nx * ny));
    const int G[3] = {B.lo[0] - ng + i - lo[0], B.lo[1] - ng + j - lo[1], B.lo[2] - ng + k - lo[2]};
    bool inside = true, wall = false;
    int u[3];
    for (int d = 0; d < 3; ++d) {
      const bool per = g.per & (1 << d);
      if (!per && (G[d] < 0 || G[d] > n[d])) inside = false;
      u[d] = unknown_of(G[d], n[d], per);
      if (u[d] < 0) wall = true;
    }
    if (!inside) continue;  // a ghost node beyond a wall keeps its value
    dst[B.off + e] = wall ? 0.0 : src[pidx(g, u[0], u[1], u[2])];
  }
}

// grid.y = box of the cell MultiFab (ng 0): sigma entry of each cell (and,
// along a periodic direction, the wrapped entry 0 from the last cell).
__global__ void __launch_bounds__(256)
    k_nd_sigma(NdGeo g, const NdBox* __restrict__ boxes, int3 dlo, int3 dn,
               const double* __restrict__ cells, double* __restrict__ sig) {
  const NdBox B = boxes[blockIdx.y];
  const int nx = B.hi[0] - B.lo[0] + 1, ny = B.hi[1] - B.lo[1] + 1, nz = B.hi[2] - B.lo[2] + 1;
  const long long total = (long long)nx * ny * nz;
  const int sx = g.mx + 1, sy = g.my + 1;
  const int n[3] = {dn.x, dn.y, dn.z};
  for (long long e = blockIdx.x * 256ll + threadIdx.x; e < total; e += 256ll * gridDim.x) {
    const int i = (int)(e % nx), j = (int)((e / nx) % ny), k = (int)(e / ((long long)nx * ny));
    const int c[3] = {B.lo[0] + i - dlo.x, B.lo[1] + j - dlo.y, B.lo[2] + k - dlo.z};
    const double v = cells[B.off + e];
    // entry index: the cell itself on a Dirichlet direction, cell + 1 on a
    // periodic one (entry 0 holds the last cell)
    int a[3], nw = 1;
    int alt[3] = {-1, -1, -1};
    for (int d = 0; d < 3; ++d) {
      const bool per = g.per & (1 << d);
      a[d] = per ? c[d] + 1 : c[d];
      if (per && c[d] == n[d] - 1) alt[d] = 0;
    }
    // write every combination of the entry and its wrapped copy
    for (int m = 0; m < 8; ++m) {
      int q[3];
      bool ok = true;
      for (int d = 0; d < 3; ++d) {
        if (m & (1 << d)) {
          if (alt[d] < 0) ok = false;
          q[d] = alt[d];
        } else {
          q[d] = a[d];
        }
      }
      if (!ok) continue;
      sig[q[0] + sx * (q[1] + sy * q[2])] = v;
    }
    (void)nw;
  }
}

// Partial sums of the valid nodes, one per work-group (FP64, fixed order).
__global__ void __launch_bounds__(256)
    k_nd_sum_partials(NdGeo g, const double* __restrict__ v, double* __restrict__ part) {
  __shared__ double red[4];
  const int ux = blockIdx.x * 64 + threadIdx.x;
  const int uy = blockIdx.y * 4 + threadIdx.y;
  const int z0 = blockIdx.z * g.tz;
  double sm = 0.0;
  if (ux < g.mx && uy < g.my) {
    const int z1 = min(z0 + g.tz, g.mz);
    for (int uz = z0; uz < z1; ++uz) sm += v[pidx(g, ux, uy, uz)];
  }
  for (int o = 32; o > 0; o >>= 1) sm += __shfl_xor(sm, o);
  if (threadIdx.x == 0) red[threadIdx.y] = sm;
  __syncthreads();
  if (threadIdx.x == 0 && threadIdx.y == 0)
    part[blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)] =
        (red[0] + red[1]) + (red[2] + red[3]);
}

// v -= (sum of the partials) / (number of unknowns) on every valid node; the
// partials are summed by every work-group in the same order.
__global__ void __launch_bounds__(256)
    k_nd_shift(NdGeo g, double* __restrict__ v, const double* __restrict__ part, int npart) {
  __shared__ double mean;
  if (threadIdx.x == 0 && threadIdx.y == 0) {
    double s = 0.0;
    for (int i = 0; i < npart; ++i) s += part[i];
    mean = s / ((double)g.mx * g.my * g.mz);
  }
  __syncthreads();
  const int ux = blockIdx.x * 64 + threadIdx.x;
  const int uy = blockIdx.y * 4 + threadIdx.y;
  const int z0 = blockIdx.z * g.tz;
  if (ux < g.mx && uy < g.my) {
    const int z1 = min(z0 + g.tz, g.mz);
    for (int uz = z0; uz < z1; ++uz) v[pidx(g, ux, uy, uz)] -= mean;
  }
}

// Partial sums of a.b over the valid nodes, one per work-group.
__global__ void __launch_bounds__(256)
    k_nd_dot_partials(NdGeo g, const double* __restrict__ a, const double* __restrict__ b,
                      double* __restrict__ part) {
  __shared__ double red[4];
  const int ux = blockIdx.x * 64 + threadIdx.x;
  const int uy = blockIdx.y * 4 + threadIdx.y;
  const int z0 = blockIdx.z * g.tz;
  double sm = 0.0;
  if (ux < g.mx && uy < g.my) {
    const int z1 = min(z0 + g.tz, g.mz);
    for (int uz = z0; uz < z1; ++uz) {
      const int c = pidx(g, ux, uy, uz);
      sm += a[c] * b[c];
    }
  }
  for (int o = 32; o > 0; o >>= 1) sm += __shfl_xor(sm, o);
  if (threadIdx.x == 0) red[threadIdx.y] = sm;
  __syncthreads();
  if (threadIdx.x == 0 && threadIdx.y == 0)
    part[blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)] =
        (red[0] + red[1]) + (red[2] + red[3]);
}

// out = sum of n partials (one work-group, fixed order).
__global__ void __launch_bounds__(256)
    k_nd_sum_final(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double red[4];
  double sm = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) sm += part[i];
  for (int o = 32; o > 0; o >>= 1) sm += __shfl_xor(sm, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sm;
  __syncthreads();
  if (threadIdx.x == 0) *out = (red[0] + red[1]) + (red[2] + red[3]);
}

// p = z (restart) or z + (rho / rho_old) p.
__global__ void __launch_bounds__(256)
    k_nd_cg_p(NdGeo g, double* __restrict__ p, const double* __restrict__ z,
              const double* __restrict__ rho, const double* __restrict__ rho_old, int restart) {
  const int ux = blockIdx.x * 64 + threadIdx.x;
  const int uy = blockIdx.y * 4 + threadIdx.y;
  const int z0 = blockIdx.z * g.tz;
  if (ux >= g.mx || uy >= g.my) return;
  const double beta = restart ? 0.0 : *rho / *rho_old;
  const int z1 = min(z0 + g.tz, g.mz);
  for (int uz = z0; uz < z1; ++uz) {
    const int c = pidx(g, ux, uy, uz);
    p[c] = restart ? z[c] : z[c] + beta * p[c];
  }
}

// alpha = rho / pq; x += alpha p; r -= alpha q; max |r| into norm.
__global__ void __launch_bounds__(256)
    k_nd_cg_xr(NdGeo g, double* __restrict__ x, const double* __restrict__ p,
               double* __restrict__ r, const double* __restrict__ q,
               const double* __restrict__ rho, const double* __restrict__ pq,
               unsigned long long* norm) {
  const int ux = blockIdx.x * 64 + threadIdx.x;
  const int uy = blockIdx.y * 4 + threadIdx.y;
  const int z0 = blockIdx.z * g.tz;
  unsigned long long mx = 0;
  if (ux < g.mx && uy < g.my) {
    const double alpha = *rho / *pq;
    const int z1 = min(z0 + g.tz, g.mz);
    for (int uz = z0; uz < z1; ++uz) {
      const int c = pidx(g, ux, uy, uz);
      x[c] += alpha * p[c];
      const double rv = r[c] - alpha * q[c];
      r[c] = rv;
      const unsigned long long b = absbits(rv);
      mx = b > mx ? b : mx;
    }
  }
  nd_block_max(mx, norm);
}

__global__ void k_nd_fill(double* a, long long n, double v) {
  const long long i = blockIdx.x * 256ll + threadIdx.x;
  if (i < n) a[i] = v;
}

__global__ void k_nd_fill_u64(unsigned long long* a, int n, unsigned long long v) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) a[i] = v;
}

dim3 sweep_grid(const NdGeo& g) {
  return dim3((g.mx + 63) / 64, (g.my + 3) / 4, (g.mz + g.tz - 1) / g.tz);
}
dim3 plane_grid(const NdGeo& g) { return dim3((g.mx + 63) / 64, (g.my + 3) / 4, g.mz); }
// 1-D grids of the XCD-grouped tile order (nd_tile)
dim3 xcd_grid(long long ntiles) {
  return dim3((unsigned)(kNdXcds * ((ntiles + kNdXcds - 1) / kNdXcds)));
}
dim3 sweep_grid_xcd(const NdGeo& g) {
  const dim3 t = sweep_grid(g);
  return xcd_grid((long long)t.x * t.y * t.z);
}
dim3 plane_grid_xcd(const NdGeo& g) {
  const dim3 t = plane_grid(g);
  return xcd_grid((long long)t.x * t.y * t.z);
}

}  // namespace

hipError_t nd_launch_sweep0(hipStream_t st, const NdGeo& g, const NdKappa& k, const double* sig,
                            const double* phi, const double* f, double* out, double omega,
                            int mode, unsigned long long* norm, double* part, double* dot) {
  const dim3 b(64, 4), gr = sweep_grid_xcd(g);
#define L0(M, N, D)                                                                            \
  hipLaunchKernelGGL((k_nd_sweep0<M, N, D>), gr, b, 0, st, g, k, sig, phi, f, out, omega, norm, \
                     part)
  if (dot) {
    if (norm || (mode != ND_APPLY && mode != ND_JACOBI)) return hipErrorInvalidValue;
    if (mode == ND_APPLY) L0(ND_APPLY, false, true);
    else L0(ND_JACOBI, false, true);
    hipLaunchKernelGGL(k_nd_sum_final, dim3(1), dim3(256), 0, st, part, (int)gr.x, dot);
  } else if (mode == ND_ZERO) L0(ND_ZERO, false, false);
  else if (mode == ND_APPLY) L0(ND_APPLY, false, false);
  else if (mode == ND_RESID) { if (norm) L0(ND_RESID, true, false); else L0(ND_RESID, false, false); }
  else { if (norm) L0(ND_JACOBI, true, false); else L0(ND_JACOBI, false, false); }
#undef L0
  return hipGetLastError();
}

hipError_t nd_launch_sweep_st(hipStream_t st, const NdGeo& g, const NdStencilC& s,
                              const double* phi, const double* f, double* out, double omega,
                              int mode, unsigned long long* norm) {
  const dim3 b(64, 4);
#define LS(M, N) \
  hipLaunchKernelGGL((k_nd_sweep_st<M, N>), sweep_grid_xcd(g), b, 0, st, g, s, phi, f, out, omega, norm)
  if (mode == ND_ZERO) LS(ND_ZERO, false);
  else if (mode == ND_APPLY) LS(ND_APPLY, false);
  else if (mode == ND_RESID) { if (norm) LS(ND_RESID, true); else LS(ND_RESID, false); }
  else { if (norm) LS(ND_JACOBI, true); else LS(ND_JACOBI, false); }
#undef LS
  return hipGetLastError();
}

hipError_t nd_launch_restrict(hipStream_t st, const NdGeo& gf, const NdGeo& gc, const double* rf,
                              double* rc) {
  hipLaunchKernelGGL(k_nd_restrict, plane_grid_xcd(gc), dim3(64, 4), 0, st, gf, gc, rf, rc);
  return hipGetLastError();
}

hipError_t nd_launch_interp_add(hipStream_t st, const NdGeo& gf, const NdGeo& gc,
                                const double* ec, double* phif) {
  hipLaunchKernelGGL(k_nd_interp_add, sweep_grid_xcd(gf), dim3(64, 4), 0, st, gf, gc, ec, phif);
  return hipGetLastError();
}

hipError_t nd_launch_down(hipStream_t st, const NdGeo& g, const NdGeo& gc, const NdStencilC& s,
                          const double* f, double* x, double* fc, double omega) {
  const int ntx = (gc.mx + 1) / 2, nty = (gc.my + 1) / 2, ntz = (gc.mz + 1) / 2;
  hipLaunchKernelGGL((k_nd_down<2, 2, 2>), dim3(ntx * nty * ntz), dim3(256), 0, st, g, gc, ntx, nty,
                     s, f, x, fc, omega);
  return hipGetLastError();
}

hipError_t nd_launch_up(hipStream_t st, const NdGeo& g, const NdGeo& gc, const NdStencilC& s,
                        const double* f, const double* x, const double* ec, double* out,
                        double omega) {
  const int ntx = (g.mx + 3) / 4, nty = (g.my + 3) / 4, ntz = (g.mz + 3) / 4;
  hipLaunchKernelGGL((k_nd_up<4, 4, 4>), dim3(ntx * nty * ntz), dim3(256), 0, st, g, gc, ntx, nty, s,
                     f, x, ec, out, omega);
  return hipGetLastError();
}

hipError_t nd_launch_fill_ghosts(hipStream_t st, const NdGeo& g, double* a) {
  for (int d = 0; d < 3; ++d) {
    if (!(g.per & (1 << d))) continue;
    const int pz = g.mz + 2;
    const int n = d == 0 ? g.py * pz : (d == 1 ? g.px * pz : g.px * g.py);
    hipLaunchKernelGGL(k_nd_fill_ghosts, dim3((n + 255) / 256), dim3(256), 0, st, g, a, d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t nd_launch_rap0(hipStream_t st, const NdGeo& gf, const NdGeo& gc, const NdKappa& k,
                          const double* sig, const NdStencil& out) {
  NdStencilC none{};
  hipLaunchKernelGGL(k_nd_rap<true>, plane_grid(gc), dim3(64, 4), 0, st, gf, gc, k, sig, none,
                     out);
  return hipGetLastError();
}

hipError_t nd_launch_rap(hipStream_t st, const NdGeo& gf, const NdGeo& gc, const NdStencilC& in,
                         const NdStencil& out) {
  NdKappa k{};
  hipLaunchKernelGGL(k_nd_rap<false>, plane_grid(gc), dim3(64, 4), 0, st, gf, gc, k, nullptr, in,
                     out);
  return hipGetLastError();
}

hipError_t nd_launch_bottom_cg(hipStream_t st, const NdGeo& g, const NdStencilC& s,
                               const double* rhs, double* x, double* work, double tol, int maxit,
                               int singular, int* iters) {
  const long long sz = (long long)g.px * g.py * (g.mz + 2);
  hipLaunchKernelGGL(k_nd_bottom_cg, dim3(1), dim3(1024), 0, st, g, s, rhs, x, work,
                     work + sz, work + 2 * sz, tol, maxit, singular, iters);
  return hipGetLastError();
}

int nd_tail_lds(const NdTail& t) {
  long long el = 0;
  for (int l = 0; l <= t.nlev; ++l) {
    const NdGeo& g = t.lev[l].g;
    if ((long long)g.mx * g.my * g.mz > kNdTailNodes) return -1;
    el += 3ll * g.px * g.py * (g.mz + 2);
  }
  return el * 8 <= 60 * 1024 ? (int)(el * 8) : -1;
}

hipError_t nd_launch_tail(hipStream_t st, const NdTail& t, const NdTail* dt) {
  const int lds = nd_tail_lds(t);
  if (!dt || t.nlev < 0 || t.nlev > kNdTailLevels || lds < 0) return hipErrorInvalidValue;
  const NdGeo& g = t.lev[0].g;
  if (g.mx * g.my * g.mz <= 512)
    hipLaunchKernelGGL(k_nd_tail<512>, dim3(1), dim3(512), lds, st, dt);
  else
    hipLaunchKernelGGL(k_nd_tail<1024>, dim3(1), dim3(1024), lds, st, dt);
  return hipGetLastError();
}

hipError_t nd_launch_maxabs(hipStream_t st, const NdGeo& g, const double* v,
                            unsigned long long* norm) {
  hipLaunchKernelGGL(k_nd_maxabs, sweep_grid(g), dim3(64, 4), 0, st, g, v, norm);
  return hipGetLastError();
}

hipError_t nd_launch_gather(hipStream_t st, const NdGeo& g, const NdBox* boxes, int nbox,
                            int maxnodes, int ng, const int dom_lo[3], const double* src,
                            double* dst) {
  if (nbox <= 0) return hipSuccess;
  int gx = (maxnodes + 255) / 256;
  gx = gx < 1 ? 1 : (gx > 4096 ? 4096 : gx);
  hipLaunchKernelGGL(k_nd_gather, dim3(gx, nbox), dim3(256), 0, st, g, boxes, ng,
                     make_int3(dom_lo[0], dom_lo[1], dom_lo[2]), src, dst);
  return hipGetLastError();
}

hipError_t nd_launch_scatter(hipStream_t st, const NdGeo& g, const NdBox* boxes, int nbox,
                             int maxnodes, int ng, const int dom_lo[3], const int dom_n[3],
                             const double* src, double* dst) {
  if (nbox <= 0) return hipSuccess;
  int gx = (maxnodes + 255) / 256;
  gx = gx < 1 ? 1 : (gx > 4096 ? 4096 : gx);
  hipLaunchKernelGGL(k_nd_scatter, dim3(gx, nbox), dim3(256), 0, st, g, boxes, ng,
                     make_int3(dom_lo[0], dom_lo[1], dom_lo[2]),
                     make_int3(dom_n[0], dom_n[1], dom_n[2]), src, dst);
  return hipGetLastError();
}

hipError_t nd_launch_sigma(hipStream_t st, const NdGeo& g, const NdBox* boxes, int nbox,
                           int maxcells, const int dom_lo[3], const int dom_n[3],
                           const double* cells, double* sig) {
  if (nbox <= 0) return hipSuccess;
  int gx = (maxcells + 255) / 256;
  gx = gx < 1 ? 1 : (gx > 4096 ? 4096 : gx);
  hipLaunchKernelGGL(k_nd_sigma, dim3(gx, nbox), dim3(256), 0, st, g, boxes,
                     make_int3(dom_lo[0], dom_lo[1], dom_lo[2]),
                     make_int3(dom_n[0], dom_n[1], dom_n[2]), cells, sig);
  return hipGetLastError();
}

int nd_sum_partials_count(const NdGeo& g) {
  const dim3 gr = sweep_grid(g);
  return (int)(gr.x * gr.y * gr.z);
}

hipError_t nd_launch_remove_mean(hipStream_t st, const NdGeo& g, double* v, double* part) {
  hipLaunchKernelGGL(k_nd_sum_partials, sweep_grid(g), dim3(64, 4), 0, st, g, v, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_nd_shift, sweep_grid(g), dim3(64, 4), 0, st, g, v, part,
                     nd_sum_partials_count(g));
  return hipGetLastError();
}

hipError_t nd_launch_dot(hipStream_t st, const NdGeo& g, const double* a, const double* b,
                         double* part, double* out) {
  hipLaunchKernelGGL(k_nd_dot_partials, sweep_grid(g), dim3(64, 4), 0, st, g, a, b, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_nd_sum_final, dim3(1), dim3(256), 0, st, part, nd_sum_partials_count(g),
                     out);
  return hipGetLastError();
}

hipError_t nd_launch_cg_p(hipStream_t st, const NdGeo& g, double* p, const double* z,
                          const double* rho, const double* rho_old, int restart) {
  hipLaunchKernelGGL(k_nd_cg_p, sweep_grid(g), dim3(64, 4), 0, st, g, p, z, rho, rho_old,
                     restart);
  return hipGetLastError();
}

hipError_t nd_launch_cg_xr(hipStream_t st, const NdGeo& g, double* x, const double* p, double* r,
                           const double* q, const double* rho, const double* pq,
                           unsigned long long* norm) {
  hipLaunchKernelGGL(k_nd_cg_xr, sweep_grid(g), dim3(64, 4), 0, st, g, x, p, r, q, rho, pq, norm);
  return hipGetLastError();
}

hipError_t nd_launch_fill(hipStream_t st, double* a, long long n, double v) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_nd_fill, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, a, n, v);
  return hipGetLastError();
}

hipError_t nd_launch_fill_u64(hipStream_t st, unsigned long long* a, int n,
                              unsigned long long v) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_nd_fill_u64, dim3((n + 255) / 256), dim3(256), 0, st, a, n, v);
  return hipGetLastError();
}

}  // namespace amrmg
