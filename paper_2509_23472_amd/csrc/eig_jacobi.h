// Symmetric positive semidefinite eigendecomposition of a small matrix (order <= LORACT_MAX_RANK)
// by the one-sided (Hestenes) Jacobi method in float64.
//
// Used where an l-column factor is cut to rank k (the randomized-SVD comparator of Section 3.2,
// more sampled rows than the rank, the adaptive rank): with B = Q^T X (l x n) and
// A = B B^T = W diag(lambda) W^T, the k leading left singular vectors of B are the k leading
// columns of W and its singular values are sqrt(lambda).
//
// Method.  A = L L^T is factored first (the Cholesky kernels of ortho_f64.h; a pivot at the rounding
// level of its diagonal entry ends its column with zeros, which is what a semidefinite matrix of that
// rank calls for), because the left singular vectors of L are the eigenvectors of A
// and its singular values their square roots: the iteration then works on a matrix with the
// condition number of B instead of its fourth power, and needs a third of the sweeps.  The columns
// of G = L are then orthogonalised by plane rotations from the right: for a pair (p, q) with
// a = |g_p|^2, b = |g_q|^2, c = g_p . g_q the rotation with tangent
// t = sign(b - a) 2 c / (|b - a| + sqrt((b - a)^2 + 4 c^2)) makes the two columns orthogonal; the
// longer of the two results goes to the lower index (de Rijk's rule, which keeps the columns roughly
// sorted by length and speeds up the convergence on graded matrices).  When all pairs are orthogonal
// G = W diag(sigma) (up to the order and the signs of the columns): lambda_j = |g_j|^2 and
// w_j = g_j / |g_j|.  Nothing besides G is stored -- no accumulated rotation matrix -- and a round of
// disjoint pairs (round-robin tournament order) needs no communication between pairs, only a barrier
// before the next round.  Small columns keep their relative accuracy under rotations with large
// ones, which is what the graded spectra met here (eigenvalue ratios of 1e-12) need.
//
// What bounds it.  A sweep meets every pair once, in rounds of disjoint pairs, and the rounds are sequential:
// each waits for the inner products, a chain of about twenty dependent float64 operations for the rotation, and
// the rotated columns.  So the columns are cut into blocks of 8, and what one round after the other needs
// is kept in registers: for a pair of blocks the 16 x 16 matrix M of inner products is formed once on the matrix
// cores, ONE WAVE runs all rounds of the pair on M alone (64 lanes = 8 x 8 pairs of pairs, a 2 x 2 block of M
// each; a rotation is M <- J^T M J and V <- V J), and the product V of the rotations is applied to the columns
// on the matrix cores.  A round meets columns c and c XOR x, x in Gray code order, so that the next round's
// partners are one exchange between lanes away whose distance is a power of two -- data-parallel
// primitives, no LDS -- and no barrier stands between the rounds.  M is formed afresh from the columns for every
// pair of blocks, and V has the relative accuracy of its rotations, so graded columns stay as accurate as
// with rotations of the columns themselves (CPU model, orders 48 to 264: singular values to the same 1e-14 to
// 5e-14 relative, and a sweep less than the round-robin order of single columns, 7 against 8 or 9).
//   l <= 64   one workgroup, the columns in LDS, a wave per pair of blocks (jacobi_one_kernel).
//   above     a workgroup per pair of blocks; the blocks move on in tournament order through memory
//             (jacobi_blocks_kernel, 5 to 20 workgroups), the matrix products spread over eight waves.
// Measured, with loads and eigenvectors (pairs of columns by 16 or 32 lanes each, every round through LDS, before):
// order 64 284 -> 170 us, order 96 905 -> 390 us, order 264 2.3 -> 1.48 ms.  A round takes 0.23 us (76 instructions of
// one wave and an LDS round trip for the rotations).  A pair of blocks takes 4.0 us at order 64 (0.9 of it matrix
// instructions: 16 for M, 16 for the columns) and 5.6 us at order 264, of which 2.2 are the hand-over through memory.
// The line between the forms: at order 96 six waves on four SIMDs take 8.5 us a step, the block form 6.3.
#pragma once
#include "common.h"
#include "eig_rank.h"

#define EJ_MAX_SWEEPS 30
#define EJ_ROT_TOL 1e-11        // pairs with |c| <= tol sqrt(a b) count as orthogonal
// A sweep is the last one when all its rotations were fine: |c| <= 1e-7 sqrt(a b) and |t| <= ej_fine_t.  A rotation
// puts at most |t| times such a c back into each of the other pairs of its two columns, and a pair that has had its
// turn meets at most 2 (order - 2) more of them in the sweep: 9.5e-12 with this bound on t.  So the sweep leaves
// every pair below EJ_ROT_TOL and need not be followed by one that only finds nothing to do.
#define EJ_FINE_C 1e-7
constexpr double ej_fine_t(int order) { return order <= 47 ? 1e-6 : 4.75e-5 / order; }
constexpr bool ej_fine_holds(int order) { return 2.0 * (order - 2) * EJ_FINE_C * ej_fine_t(order) < 0.99 * EJ_ROT_TOL; }
constexpr bool ej_fine_holds_all() {
  for (int l = 16; l <= LORACT_MAX_RANK; l += 16)
    if (!ej_fine_holds(l)) return false;
  return true;
}
static_assert(ej_fine_holds_all(), "a sweep of fine rotations has to leave every pair below EJ_ROT_TOL");
#define EJ_ONE_MAX 64           // largest order of the one-workgroup form (a pair of blocks per SIMD)
#define EJ_BLOCK 8              // columns per block
#define EJ_SPIN_LIMIT (1 << 23) // polls before a workgroup gives up waiting for a block

// Orders are rounded up to whole pairs of blocks (rows and columns past the matrix are zero), at least one pair.
static inline __host__ __device__ int ej_rows(int l) { return (l + 2 * EJ_BLOCK - 1) / (2 * EJ_BLOCK) * (2 * EJ_BLOCK); }
// (two rows more per column: 16-byte aligned columns whose offsets spread over the LDS banks)
static inline __host__ __device__ int ej_pitch(int l) { return ej_rows(l) + 2; }
// An even number of blocks.
static inline __host__ __device__ int ej_blocks(int l) { return ej_rows(l) / EJ_BLOCK; }
// Words shared by the workgroups of the block form: version of each block, and per sweep whether
// anything was rotated and how many workgroups are through.
#define EJ_WORDS (64 + 2 * EJ_MAX_SWEEPS)
// doubles of global work space: the columns (block form), the eigenvalues, the words above
static inline size_t ej_work_doubles(int l) {
  return (size_t)ej_rows(l) * ej_pitch(l) + LORACT_MAX_RANK + EJ_WORDS;
}

// Value of lane (lane XOR BIT), on the data-parallel-primitive path of the vector unit.
template <int CTRL>
__device__ inline double ej_dpp(double v) {
  union { double d; int i[2]; } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_mov_dpp(a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_mov_dpp(a.i[1], CTRL, 0xf, 0xf, true);
  return b.d;
}
template <int BIT>
__device__ inline double ej_lane_xor(double v, int lane) {
  if constexpr (BIT == 1) return ej_dpp<0xb1>(v);                // quad_perm [1,0,3,2]
  else if constexpr (BIT == 2) return ej_dpp<0x4e>(v);           // quad_perm [2,3,0,1]
  else if constexpr (BIT == 4) return ej_dpp<0x1b>(ej_dpp<0x141>(v));   // row_half_mirror (XOR 7), quad_perm [3,2,1,0]
  else if constexpr (BIT == 8) return ej_dpp<0x128>(v);          // row_ror:8
  else {
    // v_permlane16_swap / v_permlane32_swap of a register with itself: afterwards one result holds the even row
    // (lower half) in both places, the other the odd row (upper half)
    union { double d; unsigned i[2]; } a, r;
    a.d = v;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if constexpr (BIT == 16) {
        const auto x = __builtin_amdgcn_permlane16_swap(a.i[h], a.i[h], false, false);
        r.i[h] = (lane & 16) ? x[0] : x[1];
      } else {
        const auto x = __builtin_amdgcn_permlane32_swap(a.i[h], a.i[h], false, false);
        r.i[h] = (lane & 32) ? x[0] : x[1];
      }
    }
    return r.d;
  }
}
// Sum over the wave, the same bits in every lane.
__device__ inline double ej_wave_sum(double v) {
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
  return v;
}

// The rotation p' = C p + R q, q' = C q - R p that orthogonalises two columns with squared norms a, d and inner
// product c and leaves the longer one in p: with u = 2 c / (|d - a| + sqrt((d - a)^2 + 4 c^2)), cs = 1 / sqrt(1 + u^2)
// and sn = u cs it is (cs, sn) where a > d and the same with a quarter turn, (sn, cs), else.  The tangent u only has to
// be roughly right -- a pair that is left with a residual inner product is met again -- so it is formed from
// the hardware's reciprocal and square root estimates; what must be exact is C^2 + R^2 = 1 (else the columns would
// change length with every rotation), and cs is therefore refined to float64 accuracy (one third-order
// step on the 2^-24 estimate).  Not for c = 0.
__device__ __forceinline__ void ej_rotation(double a, double d, double c, double* C, double* R, double* u) {
  const double dd = d - a, c2 = c + c;
  const double h = fma(dd, dd, c2 * c2);
  const double t = c2 * __builtin_amdgcn_rcp(fma(h, __builtin_amdgcn_rsq(h), fabs(dd)));
  const double x = fma(t, t, 1.0);
  double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  y = fma(y * fma(0.375, e, 0.5), e, y);
  const double z = t * y;
  *C = dd >= 0.0 ? z : y;
  *R = dd >= 0.0 ? y : z;
  *u = t;
}

// LDS of a wave that works on a pair of blocks (columns 0..7 the one, 8..15 the other), in doubles:
// M [16][EJ_MP] | V [16][EJ_VP], V[c][r] = entry (r, c) | the round's rotations (C, R) [64][2], pair i's at 9 i
#define EJ_MP 17
#define EJ_VP 18
#define EJ_WAVE_DOUBLES (16 * EJ_MP + 16 * EJ_VP + 128)

// All rounds whose partners differ first in bit H: columns p (bit H clear) and p XOR x, x = 2^H .. 2^(H+1) - 1,
// eight disjoint pairs in each of the 2^H rounds; H = 3 is every column of the one block with every column of the
// other, H = 0 .. 2 the pairs inside the blocks.  Lane 8 i + j holds the 2 x 2 block of M that pair i and
// pair j have in common, and rows i and i + 8 of V in the columns of pair j.  FIRST: V starts as the
// identity instead of in LDS.  LAST: M is not needed any more.  Was a rotation coarse?
template <int H, bool FIRST, bool LAST>
__device__ __forceinline__ bool ej_rounds(double* w, int lane, double fine_t) {
  double* const M = w;
  double* const V = w + 16 * EJ_MP;
  double* const rot = V + 16 * EJ_VP;
  const int i = lane >> 3, j = lane & 7;
  constexpr int LOW = (1 << H) - 1;
  const int pi = ((i >> H) << (H + 1)) | (i & LOW), pj = ((j >> H) << (H + 1)) | (j & LOW);
  int qi = pi | (1 << H), qj = pj | (1 << H);
  double a = M[pi * EJ_MP + pj], c1 = M[pi * EJ_MP + qj], c2 = M[qi * EJ_MP + pj], d = M[qi * EJ_MP + qj];
  double vp0, vp1, vq0, vq1;
  if (FIRST) {
    vp0 = i == pj ? 1.0 : 0.0; vp1 = i + 8 == pj ? 1.0 : 0.0;
    vq0 = i == qj ? 1.0 : 0.0; vq1 = i + 8 == qj ? 1.0 : 0.0;
  } else {
    vp0 = V[pj * EJ_VP + i]; vp1 = V[pj * EJ_VP + i + 8];
    vq0 = V[qj * EJ_VP + i]; vq1 = V[qj * EJ_VP + i + 8];
  }
  unsigned coarse = 0;
#pragma unroll
  for (int s = 0; s <= LOW; ++s) {
    // the lanes of the diagonal hold a pair's squared norms a, d and inner product c1; the others compute along,
    // which costs less than a branch
    const double ad = a * d, cc = c1 * c1;
    const bool on = cc > (EJ_ROT_TOL * EJ_ROT_TOL) * ad && ad != 0.0;       // (false for NaN)
    double C, R, u;
    ej_rotation(a, d, c1, &C, &R, &u);
    *(double2*)(rot + 2 * lane) = double2{on ? C : 1.0, on ? R : 0.0};
    coarse |= (unsigned)on & ((unsigned)(cc > (EJ_FINE_C * EJ_FINE_C) * ad) | (unsigned)(fabs(u) > fine_t));
    sb_wave_sync();
    const double2 rj = *(const double2*)(rot + 18 * j), ri = *(const double2*)(rot + 18 * i);
    sb_wave_sync();
    const double x0 = fma(rj.x, a, rj.y * c1), x1 = fma(rj.x, c1, -rj.y * a);
    const double y0 = fma(rj.x, c2, rj.y * d), y1 = fma(rj.x, d, -rj.y * c2);
    a = fma(ri.x, x0, ri.y * y0);
    c1 = fma(ri.x, x1, ri.y * y1);
    c2 = fma(ri.x, y0, -ri.y * x0);
    d = fma(ri.x, y1, -ri.y * x1);
    const double t0 = fma(rj.x, vp0, rj.y * vq0), t1 = fma(rj.x, vp1, rj.y * vq1);
    vq0 = fma(rj.x, vq0, -rj.y * vp0);
    vq1 = fma(rj.x, vq1, -rj.y * vp1);
    vp0 = t0;
    vp1 = t1;
    if (s < LOW) {                                     // the next round's partners: q XOR the lowest set bit of s + 1
#define EJ_NEXT(BIT)                                                                                     \
  c1 = ej_lane_xor<BIT>(c1, lane); c2 = ej_lane_xor<8 * BIT>(c2, lane);                                  \
  d = ej_lane_xor<8 * BIT>(ej_lane_xor<BIT>(d, lane), lane);                                             \
  vq0 = ej_lane_xor<BIT>(vq0, lane); vq1 = ej_lane_xor<BIT>(vq1, lane);                                  \
  qi ^= BIT; qj ^= BIT;
      if ((s + 1) & 1) { EJ_NEXT(1) }
      else if ((s + 1) & 2) { EJ_NEXT(2) }
      else { EJ_NEXT(4) }
#undef EJ_NEXT
    }
  }
  if (!LAST) {
    M[pi * EJ_MP + pj] = a; M[pi * EJ_MP + qj] = c1; M[qi * EJ_MP + pj] = c2; M[qi * EJ_MP + qj] = d;
  }
  V[pj * EJ_VP + i] = vp0; V[pj * EJ_VP + i + 8] = vp1;
  V[qj * EJ_VP + i] = vq0; V[qj * EJ_VP + i + 8] = vq1;
  sb_wave_sync();
  return i == j && coarse != 0;
}
// The rounds of a pair of blocks; `inside`: the pairs inside the blocks too (once per sweep).
__device__ __forceinline__ bool ej_solve(double* w, int lane, double fine_t, bool inside) {
  if (!inside) return ej_rounds<3, true, true>(w, lane, fine_t);
  bool coarse = ej_rounds<0, true, false>(w, lane, fine_t);
  coarse |= ej_rounds<1, false, false>(w, lane, fine_t);
  coarse |= ej_rounds<2, false, false>(w, lane, fine_t);
  coarse |= ej_rounds<3, false, true>(w, lane, fine_t);
  return coarse;
}

// Inner products of the 16 columns of a pair of blocks (XP, XQ: 8 columns each, pitch `pitch`) over the 8-row
// steps first, first + STRIDE, ...: register r of lane l is entry (4 r + l / 16, l % 16).  A lane's two rows of a
// step are one 16-byte read and serve two matrix instructions; the order of the rows in the sum is free.
template <int STRIDE>
__device__ __forceinline__ f64x4 ej_gram(const double* XP, const double* XQ, int pitch, int rows, int lane, int first) {
  const int lc = lane & 15, lr = lane >> 4;
  const double* const x = (lc < EJ_BLOCK ? XP + lc * pitch : XQ + (lc - EJ_BLOCK) * pitch) + 2 * lr;
  f64x4 acc = {0.0, 0.0, 0.0, 0.0};
  for (int s = first; s < rows / 8; s += STRIDE) {
    const double2 v = *(const double2*)(x + 8 * s);
    acc = mfma_f64(v.x, v.x, acc);
    acc = mfma_f64(v.y, v.y, acc);
  }
  return acc;
}
// Rows 16 t0 .. + 15, 16 (t0 + dt) .., N tiles of them below `tiles`, of the columns times V, in place (and to global
// memory, write-through, if out is given: block p's columns from outP, block q's from outQ).  The product is formed
// transposed, so that lanes write along a column; N independent chains of matrix instructions.
template <int N>
__device__ __forceinline__ void ej_apply(double* XP, double* XQ, int pitch, const double* V, int lane, int t0, int dt,
                                         int tiles, double* outP, double* outQ) {
  const int lc = lane & 15, lr = lane >> 4;
  double va[4], xb[N][4];
#pragma unroll
  for (int k = 0; k < 4; ++k) va[k] = V[lc * EJ_VP + 4 * k + lr];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int t = t0 + u * dt < tiles ? t0 + u * dt : t0;
#pragma unroll
    for (int k = 0; k < 4; ++k) xb[u][k] = (k < 2 ? XP + (4 * k + lr) * pitch : XQ + (4 * k - 8 + lr) * pitch)[16 * t + lc];
  }
  f64x4 o[N];
#pragma unroll
  for (int u = 0; u < N; ++u) o[u] = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int u = 0; u < N; ++u) o[u] = mfma_f64(va[k], xb[u][k], o[u]);
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int t = t0 + u * dt;
    if (t >= tiles) break;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int at = (r < 2 ? 4 * r + lr : 4 * r - 8 + lr) * pitch + 16 * t + lc;
      (r < 2 ? XP : XQ)[at] = o[u][r];
      if (outP) __hip_atomic_store((r < 2 ? outP : outQ) + at, o[u][r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

// Entry (r, c) of the Cholesky factor: strict lower triangle in L (pitch kp), the diagonal as the
// reciprocal of the inverted diagonal blocks' own.
__device__ inline double ej_factor_entry(const double* L, const double* Dinv, int kp, int l, int r, int c) {
  if (r >= l || c >= l || r < c) return 0.0;
  if (r > c) return L[(int64_t)r * kp + c];
  const double d = Dinv[(int64_t)(r >> 4) * 256 + (r & 15) * 17];
  return d != 0.0 ? 1.0 / d : 0.0;
}

// Ranks lam[0 .. l-1] (descending, ties by index) into order[]; the first wave picks the number of columns to
// keep.  Adaptive rank (energy_rank): with s_i = sqrt(lambda_i) in descending order -- the singular
// values of the factor whose Gram matrix A is -- the smallest count with s_1 + ... + s_k_eff >=
// energy * (s_1 + ... + s_l), at most k (the retained-energy count of Section 2).  The sums run in that order; the
// roots are taken a lane each (one thread, root after root, takes 10 us at order 64).  sv: l doubles of LDS.
__device__ inline void ej_rank(const double* lam, int* order, double* sv, int* keep_out, int l, int k, double energy,
                               bool energy_rank, int threads) {
  for (int i = threadIdx.x; i < l; i += threads) {
    const int r = ej_rank_of(lam, l, i);
    order[r] = i;
    sv[r] = sqrt(lam[i]);
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    int keep = k;
    if (energy_rank) {
      const int lane = threadIdx.x;
      double total = 0.0;
      for (int i0 = 0; i0 < l; i0 += 64) {
        const double v = i0 + lane < l ? sv[i0 + lane] : 0.0;
#pragma unroll 8
        for (int u = 0; u < 64; ++u) total += readlane_f64(v, u);        // (zeros past the last)
      }
      const double goal = energy * total;
      double run = 0.0;
      keep = l;
      for (int i0 = 0; i0 < l && keep == l; i0 += 64) {
        const double v = i0 + lane < l ? sv[i0 + lane] : 0.0;
#pragma unroll 8
        for (int u = 0; u < 64; ++u) {
          run += readlane_f64(v, u);
          if (run >= goal && i0 + u + 1 < keep) keep = i0 + u + 1;
        }
      }
      if (keep > k) keep = k;
    }
    if (threadIdx.x == 0) *keep_out = keep;
  }
  __syncthreads();
}

struct EjArgs {
  const double* L;       // Cholesky factor of A: strict lower triangle, pitch kp
  const double* Dinv;    // inverted 16 x 16 diagonal blocks
  double* work;          // ej_work_doubles(l) doubles
  double* Wk;            // l x k out: eigenvectors of the k largest eigenvalues, descending (zero where the eigenvalue is)
  int l, k, kp;
  double energy;
  int32_t* k_out;        // adaptive rank: out, else null (columns of Wk past the rank are zero)
  int32_t* status;
};
__host__ __device__ inline double* ej_lam(const EjArgs& g) {
  return g.work + (size_t)ej_rows(g.l) * ej_pitch(g.l);
}
__host__ __device__ inline int32_t* ej_words(const EjArgs& g) { return (int32_t*)(ej_lam(g) + LORACT_MAX_RANK); }

// ---------------------------------------------------------------------------------------------
// Orders up to EJ_ONE_MAX: one workgroup, the columns in LDS, wave w on the w-th pair of blocks of a step.  One
// barrier per step: a pair's columns are its wave's alone until the next.  (Waves without a pair help to load and
// to write.)
#define EJ_ONE_THREADS 512
__global__ __launch_bounds__(EJ_ONE_THREADS) void jacobi_one_kernel(EjArgs g) {
  extern __shared__ __attribute__((aligned(16))) double ej_smem[];
  __shared__ int rotated, k_eff;
  const int l = g.l, rows = ej_rows(l), pitch = ej_pitch(l), nb = ej_blocks(l), t = threadIdx.x;
  const int lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  double* const X = ej_smem;                           // [rows columns][pitch]
  double* const lam = X + rows * pitch;                // the squared norms at the end
  double* const sv = lam + rows;
  int* const order = (int*)(sv + rows);                // rows words, an even number
  double* const w = sv + rows + rows / 2 + wave * EJ_WAVE_DOUBLES;
  // row by row of L: coalesced reads, four in flight
  for (int e0 = t; e0 < rows * rows; e0 += 4 * EJ_ONE_THREADS) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * EJ_ONE_THREADS, r = e / rows, c = e - r * rows;
      v[u] = ej_factor_entry(g.L, g.Dinv, g.kp, l, r, c);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + u * EJ_ONE_THREADS, r = e / rows, c = e - r * rows;
      if (e < rows * rows) X[c * pitch + r] = v[u];
    }
  }
  if (t == 0) rotated = 0;
  __syncthreads();
  const double fine_t = ej_fine_t(rows);
  for (int sweep = 0; sweep < EJ_MAX_SWEEPS; ++sweep) {
    bool coarse = false;
    for (int step = 0; step < nb - 1; ++step) {
      if (wave < nb / 2) {
        int p = step + wave, q = step + nb - 1 - wave;
        if (p >= nb - 1) p -= nb - 1;
        if (q >= nb - 1) q -= nb - 1;
        if (wave == 0) q = nb - 1;
        double* const XP = X + (p < q ? p : q) * EJ_BLOCK * pitch;
        double* const XQ = X + (p < q ? q : p) * EJ_BLOCK * pitch;
        const f64x4 m = ej_gram<1>(XP, XQ, pitch, rows, lane, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r) w[(4 * r + (lane >> 4)) * EJ_MP + (lane & 15)] = m[r];
        sb_wave_sync();
        coarse |= ej_solve(w, lane, fine_t, step == 0);
        for (int rt = 0; rt < rows / 16; rt += 2)
          ej_apply<2>(XP, XQ, pitch, w + 16 * EJ_MP, lane, rt, 1, rows / 16, nullptr, nullptr);
      }
      __syncthreads();
    }
    if (coarse) rotated = 1;
    __syncthreads();
    const int again = rotated;
    __syncthreads();
    if (!again) break;
    if (t == 0) rotated = 0;                           // (the next step's barrier comes before the next writing)
  }
  for (int c = wave; c < l; c += EJ_ONE_THREADS / 64) {
    double s = 0.0;
    for (int r = lane; r < rows; r += 64) s = fma(X[c * pitch + r], X[c * pitch + r], s);
    s = ej_wave_sum(s);
    if (lane == 0) lam[c] = s;
  }
  __syncthreads();
  ej_rank(lam, order, sv, &k_eff, l, g.k, g.energy, g.k_out != nullptr, EJ_ONE_THREADS);
  if (t == 0 && g.k_out) *g.k_out = k_eff;
  for (int e = t; e < l * g.k; e += EJ_ONE_THREADS) {
    const int r = e / g.k, c = e - r * g.k;
    double v = 0.0;
    if (c < k_eff && sv[c] > 0.0) v = X[order[c] * pitch + r] / sv[c];
    g.Wk[e] = v;
  }
}
static inline size_t jacobi_one_lds_bytes(int l) {
  const int rows = ej_rows(l);
  return ((size_t)rows * ej_pitch(l) + 2 * rows + rows / 2 + (size_t)(ej_blocks(l) / 2) * EJ_WAVE_DOUBLES) * sizeof(double);
}

// ---------------------------------------------------------------------------------------------
// Orders above: blocks of columns in a work buffer.

// The columns of L; the eigenvalues (which workgroups that give up never write) and the shared words cleared.
__global__ __launch_bounds__(256) void jacobi_init_kernel(EjArgs g) {
  const int cols = ej_rows(g.l), pitch = ej_pitch(g.l);
  for (int e = blockIdx.x * 256 + threadIdx.x; e < cols * pitch; e += gridDim.x * 256) {
    const int r = e / cols, c = e - r * cols;
    g.work[(int64_t)c * pitch + r] = ej_factor_entry(g.L, g.Dinv, g.kp, g.l, r, c);
  }
  if (blockIdx.x == 0) {
    for (int e = threadIdx.x; e < EJ_WORDS; e += 256) ej_words(g)[e] = 0;
    for (int e = threadIdx.x; e < g.l; e += 256) ej_lam(g)[e] = 0.0;
  }
}

// Workgroup w of blocks / 2.  Blocks are handed from workgroup to workgroup through memory: version v
// of a block is complete when its word says so (written after the block's write-through stores have
// completed); one workgroup owns a block at a time, so nothing is overwritten that another still
// reads.  A workgroup waits for the two owners of its next blocks only, and once per sweep for all (has
// anything been rotated?).  The workgroups wait for each other, so all of them have to get a CU; they are
// at most twenty, whatever else runs ends and makes room, and every wait is bounded (then the status
// word says LORACT_STATUS_INTERNAL and the workgroup ends).
#define EJ_BLK_THREADS 512
__global__ __launch_bounds__(EJ_BLK_THREADS) void jacobi_blocks_kernel(EjArgs g) {
  constexpr int THREADS = EJ_BLK_THREADS, NWV = THREADS / 64;
  extern __shared__ __attribute__((aligned(16))) double ej_smem[];
  __shared__ int rotated, go_on;
  const int rows = ej_rows(g.l), pitch = ej_pitch(g.l), nb = ej_blocks(g.l);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int32_t* const version = ej_words(g);
  int32_t* const sweep_rot = version + 64;
  int32_t* const sweep_in = sweep_rot + EJ_MAX_SWEEPS;
  const int block_doubles = EJ_BLOCK * pitch;          // even, so a block is whole 16-byte pieces
  double* const XP = ej_smem;
  double* const XQ = XP + block_doubles;
  double* const part = XQ + block_doubles;             // [NWV][256] shares of M
  double* const w = part + NWV * 256;
  const double fine_t = ej_fine_t(rows);

  // the calling thread polls until `word` has reached `want`; false when the wait ran out
  auto wait_for = [&](const int32_t* word, int want) {
    for (int spin = 0; spin < EJ_SPIN_LIMIT; ++spin) {
      if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want) return true;
      __builtin_amdgcn_s_sleep(1);
    }
    return false;
  };

  int step = 0;
  for (int sweep = 0; sweep < EJ_MAX_SWEEPS; ++sweep) {
    bool coarse = false;
    for (int round = 0; round < nb - 1; ++round, ++step) {
      int p = round + blockIdx.x;
      if (p >= nb - 1) p -= nb - 1;
      int q = round + nb - 1 - blockIdx.x;
      if (q >= nb - 1) q -= nb - 1;
      if (blockIdx.x == 0) q = nb - 1;
      if (p > q) { const int tmp = p; p = q; q = tmp; }
      if (wave == 0) {                                 // lanes 0 and 1 poll for the two blocks side by side
        bool ok = true;
        if (lane < 2) ok = wait_for(version + (lane ? q : p), step);
        const bool all = __all(ok);
        if (lane == 0) go_on = all;
      }
      __syncthreads();
      if (!go_on) break;                               // (uniform)
      double* const gp = g.work + (int64_t)p * block_doubles;
      double* const gq = g.work + (int64_t)q * block_doubles;
      for (int e = wave * 64; e < block_doubles; e += NWV * 64) {      // 64 pieces of 16 bytes per wave, two blocks
        const int piece = e + lane;
        if (piece < block_doubles) {
          const double* src = 2 * piece < block_doubles ? gp + 2 * piece : gq + 2 * piece - block_doubles;
          sb_async16_device(src, (unsigned char*)XP + 16 * e);
        }
      }
      SB_WAIT_VMCNT(0);
      __syncthreads();
      const f64x4 m = ej_gram<NWV>(XP, XQ, pitch, rows, lane, wave);
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave * 256 + 64 * r + lane] = m[r];
      __syncthreads();
      if (t < 256) {                                   // the shares in the order of the waves
        double s = 0.0;
#pragma unroll
        for (int u = 0; u < NWV; ++u) s += part[u * 256 + t];
        w[(t >> 4) * EJ_MP + (t & 15)] = s;
      }
      __syncthreads();
      if (wave == 0) coarse |= ej_solve(w, lane, fine_t, round == 0);
      __syncthreads();
      for (int rt = wave; rt < rows / 16; rt += NWV)
        ej_apply<1>(XP, XQ, pitch, w + 16 * EJ_MP, lane, rt, 1, rt + 1, gp, gq);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();                                 // every wave's stores are complete
      if (t < 2) __hip_atomic_store(version + (t ? q : p), step + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (round == nb - 2) {                           // this sweep's last holder of the blocks: their squared norms
        for (int c = wave; c < 2 * EJ_BLOCK; c += NWV) {
          const double* const x = XP + c * pitch;      // (XQ follows XP)
          double s = 0.0;
          for (int r = lane; r < rows; r += 64) s = fma(x[r], x[r], s);
          s = ej_wave_sum(s);
          const int col = (c < EJ_BLOCK ? p : q - 1) * EJ_BLOCK + c;
          if (lane == 0 && col < g.l) ej_lam(g)[col] = s;
        }
        __syncthreads();                               // before the next copies into XP, XQ
      }
    }
    if (!go_on) break;
    if (t == 0) rotated = 0;
    __syncthreads();
    if (coarse) rotated = 1;
    __syncthreads();
    if (t == 0) {
      if (rotated) __hip_atomic_store(sweep_rot + sweep, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __hip_atomic_fetch_add(sweep_in + sweep, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      go_on = wait_for(sweep_in + sweep, (int)gridDim.x);
      rotated = __hip_atomic_load(sweep_rot + sweep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const bool more = go_on && rotated;
    __syncthreads();                                   // everyone has read what thread 0 writes again in the next sweep
    if (!more) break;
  }
  if (t == 0 && !go_on && g.status) atomicOr(g.status, LORACT_STATUS_INTERNAL);
}
static inline size_t jacobi_blocks_lds_bytes(int l) {
  return ((size_t)2 * EJ_BLOCK * ej_pitch(l) + EJ_BLK_THREADS / 64 * 256 + EJ_WAVE_DOUBLES) * sizeof(double);
}

// Wk from the converged columns: every workgroup ranks the eigenvalues and writes its share.
__global__ __launch_bounds__(256) void jacobi_finish_kernel(EjArgs g) {
  __shared__ double lam[LORACT_MAX_RANK], sv[LORACT_MAX_RANK];
  __shared__ int order[LORACT_MAX_RANK];
  __shared__ int k_eff;
  const int l = g.l, pitch = ej_pitch(l);
  for (int i = threadIdx.x; i < l; i += 256) lam[i] = ej_lam(g)[i];
  __syncthreads();
  ej_rank(lam, order, sv, &k_eff, l, g.k, g.energy, g.k_out != nullptr, 256);
  if (threadIdx.x == 0 && blockIdx.x == 0 && g.k_out) *g.k_out = k_eff;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < l * g.k; e += gridDim.x * 256) {
    const int c = e / l, r = e - c * l;                // down the columns: the reads are the chain
    double v = 0.0;
    if (c < k_eff && sv[c] > 0.0) v = g.work[(int64_t)order[c] * pitch + r] / sv[c];
    g.Wk[r * g.k + c] = v;
  }
}

// L, Dinv: the Cholesky factor of the l x l matrix as the kernels of ortho_f64.h leave it.
static int launch_jacobi_eig(hipStream_t s, const EjArgs& g) {
  if (g.l < 1 || g.l > LORACT_MAX_RANK || g.k < 1 || g.k > g.l) return LORACT_ERR_INVALID_ARG;
  if (g.l <= EJ_ONE_MAX) {
    static std::atomic<bool> attr_done{false};
    if (!attr_done.load(std::memory_order_acquire)) {
      hipError_t e = hipFuncSetAttribute((const void*)jacobi_one_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)jacobi_one_lds_bytes(EJ_ONE_MAX));
      if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(eigensolver LDS)");
      attr_done.store(true, std::memory_order_release);
    }
    LORACT_LAUNCH("jacobi_eig", s, jacobi_one_kernel, dim3(1), dim3(EJ_ONE_THREADS), jacobi_one_lds_bytes(g.l), g);
    return LORACT_OK;
  }
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)jacobi_blocks_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)jacobi_blocks_lds_bytes(LORACT_MAX_RANK));
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(eigensolver LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("jacobi_init", s, jacobi_init_kernel, dim3(64), dim3(256), 0, g);
  LORACT_LAUNCH("jacobi_eig", s, jacobi_blocks_kernel, dim3(ej_blocks(g.l) / 2), dim3(EJ_BLK_THREADS),
                jacobi_blocks_lds_bytes(g.l), g);
  LORACT_LAUNCH("jacobi_finish", s, jacobi_finish_kernel, dim3(64), dim3(256), 0, g);
  return LORACT_OK;
}
