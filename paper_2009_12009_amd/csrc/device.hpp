// Device helpers shared by the kernel files: the max-norm fold, block sums and
// the body of the bottom CG.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.hpp"

namespace amrmg {

namespace {

__device__ __forceinline__ unsigned long long absbits(double v) {
  return (unsigned long long)__double_as_longlong(fabs(v));
}
__device__ __forceinline__ unsigned long long absbits(float v) { return absbits((double)v); }

// Fold a per-lane value into the norm slot at dst as an unsigned max over
// the block, into the block's way of the slot (kNormWays words on separate
// cache lines, so the blocks of a launch do not all meet on one line).  The
// block's atomic is skipped when its way already holds at least its value:
// a way only grows, so a value read at any time that is >= m makes the
// atomic a no-op.
__device__ void block_max_u64(unsigned long long v, unsigned long long* dst) {
  dst += kNormStride * (blockIdx.x % kNormWays);
  __shared__ unsigned long long red[16];
  for (int o = 32; o > 0; o >>= 1) {
    unsigned long long w = (unsigned long long)__shfl_xor((long long)v, o);
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

// v of the lane that DPP control CTRL pairs with this one.
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

__device__ __forceinline__ double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)b, lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Sum over a wavefront (all 64 lanes active), the same bits in every lane:
// inside rows of 16 lanes by DPP (neighbours, pairs, mirrored halves, mirrored
// row), then the four rows' sums.  A butterfly of shuffles goes through LDS six
// times, which is most of a small CG iteration.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp<0xB1>(v);   // quad_perm [1, 0, 3, 2]
  v += dpp<0x4E>(v);   // quad_perm [2, 3, 0, 1]
  v += dpp<0x141>(v);  // row_half_mirror
  v += dpp<0x140>(v);  // row_mirror
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Block sum in a fixed order: lanes by butterfly, or by wave_sum with FAST, then
// the first nw waves in index order (every wave of the work-group takes part in
// the barrier; later waves' sums are left out).
template <bool FAST = false>
__device__ double block_sum_w(double v, double* red, int& phase, int nw) {
  if (FAST)
    v = wave_sum(v);
  else
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  const int tid = threadIdx.x + blockDim.x * threadIdx.y;
  double* buf = red + phase * 16;
  phase ^= 1;
  if ((tid & 63) == 0) buf[tid >> 6] = v;
  __syncthreads();
  double s = buf[0];
  for (int w = 1; w < nw; ++w) s += buf[w];
  return s;
}

// ... over every wave of the work-group.
__device__ double block_sum(double v, double* red, int& phase) {
  return block_sum_w(v, red, phase, (blockDim.x * blockDim.y + 63) / 64);
}

// The body runs on any work-group: lanes stride the cells by nt (lane l owns
// l, l+nt, ...), the dot products add the first nw waves' sums, and every
// wave takes part in the barriers (lanes past the cells hold zeros).  p:
// n values of LDS.
// The CG's sums and barriers.  ONE_WAVE: the CG runs in wavefront 0 alone
// (n <= 64, lanes 0..63): wave_sum leaves the sum in every lane (the value
// the work-group form reads back for one wave) and LDS needs only
// wave-level ordering.
template <bool ONE_WAVE>
__device__ __forceinline__ double cg_sum(double v, double* red, int& phase, int nw) {
  if (ONE_WAVE) {
    return wave_sum(v);
  }
  return block_sum_w<true>(v, red, phase, nw);
}

template <bool ONE_WAVE>
__device__ __forceinline__ void cg_sync() {
  if (ONE_WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// Scale of the bottom CGs' scalars r.r, a power of two: right-hand sides below
// some 1e-140 bring tol^2 r.r and 1 / r.r to the ends of the range, where the one
// underflows and the other overflows.  A factor costs a multiplication; a branch
// with the square root and the quotient of the plain forms in the loop cost the
// kernels that use all their registers 8 % of their time.
__device__ __forceinline__ double cg_scale(double rho) { return rho < 0x1p-700 ? 0x1p600 : 1.0; }

template <typename T, int CPT, bool ONE_WAVE = false>
__device__ __forceinline__ void cg_lds_run(const BottomTables& bt, const T* __restrict__ diag,
                                           const T* __restrict__ coef, const T* __restrict__ rhs,
                                           T* __restrict__ out, int accumulate, double tol,
                                           int maxiter, int singular, int* iters_out, T* p,
                                           double* red, int nt, int nw) {
  // no multiply-add fusion: whether the compiler fuses a product into an
  // addition depends on the code around it, and the work-group and the
  // one-wavefront forms (and every kernel that runs this body) must round
  // the same way
#pragma clang fp contract(off)
  int phase = 0;
  const int n = bt.n;
  const int tid = threadIdx.x;
  // stencil in registers up to two cells per lane (more would spill)
  constexpr bool REG = CPT <= 2;
  constexpr int RC = REG ? CPT : 1;
  T x[CPT], r[CPT], q[CPT], dg[RC], cf[RC][6];
  int nb[RC][6];
  double s = 0.0;
#pragma unroll
  for (int m = 0; m < CPT; ++m) {
    const int c = tid + m * nt;
    x[m] = T(0);
    r[m] = T(0);
    if (c < n) {
      r[m] = rhs[bt.map_rhs[c]];
      s += (double)r[m];
    }
    if (REG) {
      dg[m % RC] = c < n ? diag[c] : T(1);
      for (int f = 0; f < 6; ++f) {
        nb[m % RC][f] = c < n ? bt.nbr[f * n + c] : -1;
        cf[m % RC][f] = c < n ? coef[f * n + c] : T(0);
      }
    }
  }
  if (singular) {
    s = cg_sum<ONE_WAVE>(s, red, phase, nw);
    const T mean = (T)(s / n);
#pragma unroll
    for (int m = 0; m < CPT; ++m)
      if (tid + m * nt < n) r[m] = r[m] - mean;
  }
  s = 0.0;
#pragma unroll
  for (int m = 0; m < CPT; ++m) s += (double)r[m] * (double)r[m];
  double rho = cg_sum<ONE_WAVE>(s, red, phase, nw);
  // stop at ||r|| <= tol ||rhs||, compared as squares
  const double sc = cg_scale(rho), stop = tol * tol * (sc * rho);
  int it = 0;
  if (rho > 0.0) {
#pragma unroll
    for (int m = 0; m < CPT; ++m)
      if (tid + m * nt < n) p[tid + m * nt] = r[m];
    while (it < maxiter) {
      cg_sync<ONE_WAVE>();
      // off the chain of dependent steps, unlike a quotient by rho below
      const double inv = 1.0 / (sc * rho);
      s = 0.0;
#pragma unroll
      for (int m = 0; m < CPT; ++m) {
        const int c = tid + m * nt;
        q[m] = T(0);
        if (c < n) {
          T off = T(0);
          if (REG) {
#pragma unroll
            for (int f = 0; f < 6; ++f)
              off = off + (nb[m % RC][f] < 0 ? T(0) : cf[m % RC][f] * p[nb[m % RC][f]]);
            q[m] = dg[m % RC] * p[c] - off;
          } else {
            for (int f = 0; f < 6; ++f) {
              const int k = bt.nbr[f * n + c];
              off = off + (k < 0 ? T(0) : coef[f * n + c] * p[k]);
            }
            q[m] = diag[c] * p[c] - off;
          }
          s += (double)p[c] * (double)q[m];
        }
      }
      const double pq = cg_sum<ONE_WAVE>(s, red, phase, nw);
      const T alT = (T)(rho / pq);
      s = 0.0;
#pragma unroll
      for (int m = 0; m < CPT; ++m) {
        const int c = tid + m * nt;
        if (c < n) {
          x[m] = x[m] + alT * p[c];
          r[m] = r[m] - alT * q[m];
          s += (double)r[m] * (double)r[m];
        }
      }
      ++it;
      const double rho_new = cg_sum<ONE_WAVE>(s, red, phase, nw);
      if (!(sc * rho_new > stop)) break;
      const T btT = (T)(sc * rho_new * inv);
#pragma unroll
      for (int m = 0; m < CPT; ++m) {
        const int c = tid + m * nt;
        if (c < n) p[c] = r[m] + btT * p[c];
      }
      rho = rho_new;
    }
  }
  if (singular) {
    s = 0.0;
#pragma unroll
    for (int m = 0; m < CPT; ++m)
      if (tid + m * nt < n) s += (double)x[m];
    s = cg_sum<ONE_WAVE>(s, red, phase, nw);
    const T mean = (T)(s / n);
#pragma unroll
    for (int m = 0; m < CPT; ++m) x[m] = x[m] - mean;
  }
#pragma unroll
  for (int m = 0; m < CPT; ++m) {
    const int c = tid + m * nt;
    if (c < n) {
      const long long o = bt.map_out[c];
      out[o] = accumulate ? out[o] + x[m] : x[m];
    }
  }
  if (tid == 0) *iters_out = it;
}

}  // namespace

}  // namespace amrmg
