// The split-colour layout of a level and the launchers of its kernels.
//
// The level's boxes cover its domain, so the V-cycle keeps each level as one
// grid instead of a list of boxes, and each array as two halves, the red
// cells ((i + j + k) even) and the black ones.  Row (j, k) of a half holds the
// colour's cell of each x-pair p: cell i = 2p + ((j + k + colour) & 1).  A
// half-sweep then reads the other colour, its own right-hand side and every
// face, each as whole lines, and writes its own colour without reading it:
// 4.5 values per cell against 6 where red and black share cache lines.  No
// ghost layer exists (neighbours past a wall are not used, periodic ones wrap),
// so there is no exchange either.
//
// Faces hold the operator's coefficient c = (beta b) / h_d^2.  x faces: the
// even ones [0, half), the odd ones [half, 2 half), rows like a cell row (pair
// p: faces 2p and 2p + 1; face nx is the even entry nx / 2).  y and z faces:
// the half of colour c holds the low face of the colour's cells, with one more
// row (y) or plane (z) for the high boundary, so the high y face of a cell is
// the low face of the other colour's cell above it.
#pragma once

#include <hip/hip_runtime_api.h>

#include "kernels.hpp"
#include "tables.hpp"

namespace amrmg {

// Extents, pitch and array sizes of a level (np = x-pairs per row; sp = row
// pitch in elements, at least nx / 2 + 1; half, yh,
// zh = elements of one half of a cell or x-face, y-face and z-face array).
struct FlatDims {
  int nx, ny, nz, np, sp;
  int wall;  // bit 2d: the low side along d is a wall, 2d + 1: the high side
  int half, yh, zh;
};

// elem: bytes of an element.
FlatDims flat_dims(const int n[3], const int periodic[3], int elem);
// Whether the level's arrays fit the kernels' 32-bit element offsets.
bool flat_fits(const int n[3], int elem);

// The operator on a level.
template <typename T>
struct FlatOp {
  FlatDims d;
  const T* x;
  const T* y;
  const T* z;
  const T* a;  // alpha * a, both halves, or null for a = 1
  T alpha;
  const int* done = nullptr;  // if set and *done is not 0, a pass does nothing
};

// Launch order and cache hints of a pass: stream = the level's arrays exceed
// the last-level cache (read-once loads carry the non-temporal hint); reverse =
// walk the level from its end.
struct FlatPass {
  int stream = 0;
  int reverse = 0;
};

// One half-sweep: out (the colour's half) = (f + sum c other) / diag.  f: both
// halves.  With zero_guess other is taken as 0 and not read.  With ec (both
// halves of the next coarser level's correction, dims cd) every value read of
// the other colour gets its coarse parent's correction added first.  With old
// (the colour's half before the update) max |f - A phi| over the colour's
// cells is folded into *normbits.
template <typename T>
hipError_t launch_flat_half(hipStream_t st, const FlatOp<T>& op, FlatPass ps, const T* other,
                            T* out, const T* f, int colour, bool zero_guess,
                            const FlatDims* cd = nullptr, const T* ec = nullptr,
                            const T* old = nullptr, unsigned long long* normbits = nullptr);

// One sweep, colour c0 then the other, from src into dst (both halves of two
// arrays; of src only the colour that is not updated first is read).  The other
// arguments and the result as for the two half-sweeps.
template <typename T>
hipError_t launch_flat_sweep(hipStream_t st, const FlatOp<T>& op, const T* src, T* dst, const T* f,
                             int c0, bool zero_guess, const FlatDims* cd = nullptr,
                             const T* ec = nullptr, const T* old = nullptr,
                             unsigned long long* normbits = nullptr);

// Coarse right-hand side of a level whose black cells were updated last: their
// residual is zero, so cf = R r sums the red cells' residuals (four of the
// eight children).  v, f: both halves of the fine level, cf both halves of
// the coarse one (dims cd).
template <typename T>
hipError_t launch_flat_restrict(hipStream_t st, const FlatOp<T>& op, FlatPass ps, const T* v,
                                const T* f, const FlatDims& cd, T* cf);

// Two sweeps in one launch on blocks with a rim (nu = 2), dst != src:
// pre_zero: from a zero guess, then cf = R r as launch_flat_restrict;
// pre_after_red: the same where src is the red half after the first half-sweep;
// post_red / post_black: src (both halves of the level's array, of which the
// colour that is not updated first is read) plus the coarse correction ec,
// then two sweeps starting with that colour.  dst: both halves.  cd: the coarser
// level.  Same result as the separate launches.
// Only on levels of at most one block per CU: flat_block_pairs, the pairs of a
// block, is 0 elsewhere (there it costs more than the launches it saves).
int flat_block_pairs(const FlatDims& d, int elem);
enum class FlatBlockMode { pre_zero, pre_after_red, post_red, post_black };
template <typename T>
hipError_t launch_flat_block(hipStream_t st, const FlatOp<T>& op, FlatBlockMode mode, const T* src,
                             const T* f, T* dst, const FlatDims& cd, T* cf, const T* ec);

// out = f - A v (f non-null) or A v (f null) on both colours; out may be null
// (norm only) and narrower than T.  normbits: max |out|; dots (one per block,
// flat_resid_blocks of them): partial sums of v * out.
template <typename T, typename TO>
hipError_t launch_flat_resid(hipStream_t st, const FlatOp<T>& op, FlatPass ps, const T* v,
                             const T* f, TO* out, unsigned long long* normbits, double* dots);
int flat_resid_blocks(const FlatDims& d);
// vn = v + e (vn != v) and out = f - A vn, max |out| as above.
hipError_t launch_flat_update_resid(hipStream_t st, const FlatOp<double>& op, FlatPass ps,
                                    const double* v, const float* e, double* vn, const double* f,
                                    float* out, unsigned long long* normbits);

// Box arrays (ng 0 or 1) <-> the split-colour array, valid cells (scatter with
// ghosts, ng 1: and the ghost cells inside the domain or across periodic faces).
// lo: low corner of the domain.  normbits (gather): max |value|.
template <typename T>
hipError_t launch_flat_gather(hipStream_t st, const BoxInfo* boxes, int nbox, int max_cells,
                              const int lo[3], const FlatDims& d, const T* src, int ng, T* dst,
                              unsigned long long* normbits);
template <typename T>
hipError_t launch_flat_scatter(hipStream_t st, const BoxInfo* boxes, int nbox, int max_cells,
                               const int lo[3], const FlatDims& d, const T* src, T* dst, int ng,
                               bool ghosts);
// Coefficients from a level's box arrays: faces of direction dir scaled by
// (beta b) ih (a face shared by two boxes is taken from the box above it, see
// launch_flat_shared), cell coefficient as alpha * a.
template <typename T>
hipError_t launch_flat_faces(hipStream_t st, const BoxInfo* boxes, int nbox, int max_faces,
                             const int lo[3], const FlatDims& d, int dir, const T* b, T beta, T ih,
                             T* dst);
// *differ = 1 if a box holds another value (scaled as above, beyond four units in
// the last place) for a face than the box above it, or than the other end of a
// periodic direction; b: the level's face
// arrays, op: its faces as launch_flat_faces left them.  max_plane: the most faces
// of a box in one plane.
template <typename T>
hipError_t launch_flat_shared(hipStream_t st, const BoxInfo* boxes, int nbox, int max_plane,
                              const int lo[3], const FlatOp<T>& op, const T* const b[3], T beta,
                              const T ih[3], unsigned long long* differ);
template <typename T>
hipError_t launch_flat_acoef(hipStream_t st, const BoxInfo* boxes, int nbox, int max_cells,
                             const int lo[3], const FlatDims& d, const T* a, T alpha, T* dst);

// Vectors of the level (both halves, n = 2 half elements, padding zero).
constexpr int kFlatDotBlocks = 1024;
// *out = sum a * z (z double or float), partials: kFlatDotBlocks doubles.
template <typename TZ>
hipError_t launch_flat_dot(hipStream_t st, long long n, const double* a, const TZ* z,
                           double* partials, double* out);
// p = z (first) or z + (*num / *den) p; padding stays 0
template <typename TZ>
hipError_t launch_flat_cg_p(hipStream_t st, const FlatDims& d, double* p, const TZ* z,
                            const double* num, const double* den, int first);
// x += al p, r -= al q, al = *num / *den; max |r|; r32 (nullable) = r rounded;
// padding stays 0
hipError_t launch_flat_cg_xr(hipStream_t st, const FlatDims& d, double* x, const double* p,
                             double* r, const double* q, const double* num, const double* den,
                             unsigned long long* normbits, float* r32);
// v -= mean of v over the level's cells (padding untouched); partials and sum
// as in launch_flat_dot
hipError_t launch_flat_remove_mean(hipStream_t st, const FlatDims& d, double* v, double* partials,
                                   double* sum);
hipError_t launch_flat_maxabs(hipStream_t st, long long n, const double* v,
                              unsigned long long* normbits);

// The coarsest levels and a CG bottom of at most kTailMaxBottom cells in one
// work-group: every pass a loop of its lanes with a barrier after it, the
// correction, right-hand side and residual of the levels in LDS where they all
// fit.  Same arithmetic per cell as the launches above.
template <typename T>
struct FlatTailLevel {
  FlatOp<T> op;
  T* e;
  T* f;
  T* r;  // residual of the red cells (one half)
};
template <typename T>
struct FlatTail {
  int nlev, nu1, nu2, reverse;
  FlatTailLevel<T> lev[kTailMaxLevels + 1];  // lev[nlev]: the bottom's extents, e and f
  BottomTables bt;                           // maps into the bottom's f and e
  const T *bdiag, *bcoef;
  double tol;
  int maxiter, singular;
  int* iters;
};
// dt: a copy of t in device memory.
template <typename T>
hipError_t launch_flat_tail(hipStream_t st, const FlatTail<T>& t, const FlatTail<T>* dt);

// ---------------------------------------------------------------------------
// A large CG bottom (deep bottom): conjugate gradients on the bottom's
// cells, preconditioned by one symmetric V-cycle on further coarsenings of it.
// Odd extents of a level are made even by one more cell at the high end:
//  - along a wall a cell without couplings (a = 1, right-hand side 0);
//  - along a periodic direction a cell in the link from the last cell to the
//    first, with no a and no right-hand side and both its links of twice the
//    coefficient: a series of two such links conducts as the one did, so the
//    padded system has the same solution on the level's cells.
// Wall terms are part of a, faces on walls are 0.

// Device state of the iteration, one per handle.  done: 0 going on, 1 converged,
// 2 broken off (p q not positive).
struct DeepState {
  double rho, beta, b2;
  int done, it;
  unsigned count;
};
constexpr int kDeepBlocks = 256;  // partial sums per reduction at most

// Faces and the two parts of a (mass: alpha a, wall: wall terms) of the padded
// bottom, from its stencil; bt.map_out holds the cells' elements.  pad: cells
// added along each direction.
template <typename T>
hipError_t launch_deep_fill(hipStream_t st, const BottomTables& bt, const StencilArgs<T>& op,
                            const FlatDims& d, const int pad[3], T* x, T* y, T* z, T* mass,
                            T* wall);
// a = mass + wall, or 1 for a cell with neither a nor couplings.
template <typename T>
hipError_t launch_deep_diag(hipStream_t st, const FlatDims& d, const T* x, const T* y, const T* z,
                            const T* mass, const T* wall, T* a);
// Faces, mass and wall of the next coarser level: mean face over h_d^2 = a
// sixteenth of the four faces' sum, mean mass, half the mean wall term.
template <typename T>
hipError_t launch_deep_coarsen(hipStream_t st, const FlatDims& d, const T* x, const T* y,
                               const T* z, const T* mass, const T* wall, const FlatDims& cd,
                               const int pad[3], T* cx, T* cy, T* cz, T* cmass, T* cwall);
// diag and coef of launch_bottom_cg for the deepest level.
template <typename T>
hipError_t launch_deep_bottom(hipStream_t st, const BottomTables& bt, const FlatOp<T>& op, T* diag,
                              T* coef);

// The iteration's vector passes (n elements; partials: kDeepBlocks doubles).
// r = f, x = 0, p = 0, |f|^2
template <typename T>
hipError_t launch_deep_init(hipStream_t st, long long n, const T* f, T* r, T* x, T* p,
                            double* partials, DeepState* s);
// rho = r.z and beta
template <typename T>
hipError_t launch_deep_rz(hipStream_t st, long long n, const T* r, const T* z, double* partials,
                          DeepState* s);
// p = z + beta p
template <typename T>
hipError_t launch_deep_p(hipStream_t st, long long n, const T* z, T* p, const DeepState* s);
// x += al p, r -= al q, al = rho / sum of the npq partials of p.q;
// done once |r|^2 <= tol2 |f|^2
template <typename T>
hipError_t launch_deep_xr(hipStream_t st, long long n, T* x, const T* p, T* r, const T* q,
                          const double* pq, int npq, double tol2, double* partials, DeepState* s);

}  // namespace amrmg
