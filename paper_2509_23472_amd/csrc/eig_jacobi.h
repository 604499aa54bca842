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
// What bounds it.  The l - 1 rounds of a sweep are sequential, and so are the sweeps (6 at order 64, 9 to 13
// at orders 97 to 320, for flat, geometric and power-law spectra).  A round costs its dependent chain (a
// dot product, its sum over the lanes, the rotation, a barrier: about 0.4 us) and the passage of the columns
// through a CU: 2 l^2 x 8 bytes, 1 us out of LDS at l = 136 and 15 us out of L2 at l = 264, where they no
// longer fit.  Hence two forms:
//   l <= 96  one workgroup, G in LDS, a pair per 16 lanes (jacobi_one_kernel).
//   above    the columns are cut into blocks of at most 16; a workgroup per pair of blocks holds
//            both in LDS and rotates every column of the one with every column of the other (in the
//            first step of a sweep all pairs among its 32), then the blocks move on in tournament order
//            through memory (jacobi_blocks_kernel, 4 to 10 workgroups).  A pair is handled by 32 lanes, the
//            column of the first block stays in registers through the step, so that only the other one
//            passes through LDS.
// Measured (with the Cholesky kernel where it is a launch of its own; one workgroup with everything in
// LDS up to 141 and out of L2 above, factor included, is what it was before): order 64 457 -> 297 us
// (0.75 us per round: the chain of about thirty dependent float64 operations, and both columns through LDS), order
// 264 39.8 -> 2.5 ms.
// Tried: 8 lanes per pair at order 64 (338 against 282 us) and 16 at order 264 (2.40 against 2.32 ms): fewer
// waves issue less but every chain is longer.
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
static_assert(ej_fine_holds(32) && ej_fine_holds(64) && ej_fine_holds(96) && ej_fine_holds(160) && ej_fine_holds(288) &&
              ej_fine_holds(LORACT_MAX_RANK), "a sweep of fine rotations has to leave every pair below EJ_ROT_TOL");
#define EJ_ONE_MAX 96           // largest order of the one-workgroup form
#define EJ_BLOCK 16             // columns per block, at most
#define EJ_ONE_LPP 16           // lanes per pair, one-workgroup form
#define EJ_BLK_LPP 32           // lanes per pair, block form
#define EJ_SPIN_LIMIT (1 << 23) // polls before a workgroup gives up waiting for a block

// Orders are rounded up to the next of these, so that the rows per lane and every LDS offset are
// compiled in and no lane needs a mask (rows and columns past the matrix are zero).
static inline __host__ __device__ int ej_rows(int l) {
  return l <= 32 ? 32 : l <= 64 ? 64 : l <= 96 ? 96 : l <= 160 ? 160 : l <= 288 ? 288 : 320;
}
// (two rows more per column: 16-byte aligned columns whose offsets spread over the LDS banks)
static inline __host__ __device__ int ej_pitch(int l) { return ej_rows(l) + 2; }
// Blocks of columns: an even number of them, each with ceil(l / blocks) columns (the last ones padded
// with zero columns, which no rotation touches).
static inline __host__ __device__ int ej_blocks(int l) {
  const int nb = (l + EJ_BLOCK - 1) / EJ_BLOCK;
  return l <= EJ_ONE_MAX ? 2 : nb + (nb & 1);
}
static inline __host__ __device__ int ej_block_cols(int l) { return (l + ej_blocks(l) - 1) / ej_blocks(l); }
// Words shared by the workgroups of the block form: version of each block, and per sweep whether
// anything was rotated and how many workgroups are through.
#define EJ_WORDS (64 + 2 * EJ_MAX_SWEEPS)
// doubles of global work space: the columns (block form), the eigenvalues, the words above
static inline size_t ej_work_doubles(int l) {
  return (size_t)ej_blocks(l) * ej_block_cols(l) * ej_pitch(l) + LORACT_MAX_RANK + EJ_WORDS;
}

// Sum over the 16 lanes of a group; every lane gets the total.  Four exchange steps inside a
// row of 16 lanes on the data-parallel-primitive path of the vector unit (no LDS round trip):
// mirror of the row, mirror of each half, reversal and pair swap inside each quad.
template <int CTRL>
__device__ inline double ej_dpp_add(double v) {
  union { double d; int i[2]; } a, b;
  a.d = v;
  b.i[0] = __builtin_amdgcn_mov_dpp(a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_mov_dpp(a.i[1], CTRL, 0xf, 0xf, true);
  return v + b.d;
}
// LPP = 32: two rows of 16, swapped by v_permlane16_swap (afterwards one result holds the even row of
// each pair of rows in both places, the other the odd row).
template <int LPP>
__device__ inline double ej_group_sum(double v) {
  if (LPP >= 16) v = ej_dpp_add<0x140>(v);     // row_mirror:       lane i <- lane 15 - i
  v = ej_dpp_add<0x141>(v);     // row_half_mirror:  lane i <- lane 7 - i inside each half
  v = ej_dpp_add<0x1b>(v);      // quad_perm [3,2,1,0]
  v = ej_dpp_add<0xb1>(v);      // quad_perm [1,0,3,2]
  if (LPP == 32) {
    union { double d; unsigned i[2]; } a, even, odd;
    a.d = v;
    const auto lo = __builtin_amdgcn_permlane16_swap(a.i[0], a.i[0], false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(a.i[1], a.i[1], false, false);
    even.i[0] = lo[0]; even.i[1] = hi[0];
    odd.i[0] = lo[1]; odd.i[1] = hi[1];
    v = even.d + odd.d;
  }
  return v;
}

// cos and sin of the rotation that orthogonalises two columns with squared norms a, b and inner
// product c, and its tangent.  The tangent only has to be roughly right -- a pair that is left with
// a residual inner product is met again -- so it is formed from the hardware's reciprocal and square
// root estimates; what must be exact is cs^2 + sn^2 = 1 (else the columns would change length with
// every rotation), and cs = 1 / sqrt(1 + t^2) is therefore refined to float64 accuracy (one
// third-order step on the 2^-24 estimate).
__device__ inline void ej_rotation(double a, double b, double c, double* cs, double* sn, double* tt) {
  const double d = b - a, c2 = c + c;
  const double h = fma(d, d, c2 * c2);
  const double root = h * __builtin_amdgcn_rsq(h);                 // h > 0: c is not zero
  const double t = (d >= 0.0 ? c2 : -c2) * __builtin_amdgcn_rcp(fabs(d) + root);
  const double x = fma(t, t, 1.0);
  double y = __builtin_amdgcn_rsq(x);
  const double e = fma(-x * y, y, 1.0);
  y = fma(y * fma(0.375, e, 0.5), e, y);
  *cs = y;
  *sn = t * y;
  *tt = t;
}

// One pair: columns in registers (NR rows per lane, zero past the matrix), squared norms a, b.
// Returns whether it was rotated; afterwards the longer column is in gp.  Uniform in the group: every
// lane holds the same bits of a, b and c.  `coarse` is set by a rotation that was not a fine one.
template <int NR, int LPP>
__device__ inline bool ej_pair(double* gp, double* gq, double* a, double* b, bool* coarse) {
  double c0 = 0.0, c1 = 0.0;
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    if (j & 1) c1 = fma(gp[j], gq[j], c1);
    else c0 = fma(gp[j], gq[j], c0);
  }
  const double c = ej_group_sum<LPP>(c0 + c1), ab = *a * *b;
  if (!(c * c > (EJ_ROT_TOL * EJ_ROT_TOL) * ab) || ab == 0.0) return false;
  double cs, sn, tt;
  ej_rotation(*a, *b, c, &cs, &sn, &tt);
  *coarse = *coarse || c * c > (EJ_FINE_C * EJ_FINE_C) * ab || fabs(tt) > ej_fine_t(NR * LPP);
  const double a2 = fmax(*a - tt * c, 0.0), b2 = fmax(*b + tt * c, 0.0);
  const bool swap = a2 < b2;
  const double pp = swap ? sn : cs, pq = swap ? cs : -sn, qp = swap ? cs : sn, qq = swap ? -sn : cs;
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    const double x = gp[j];
    gp[j] = fma(pp, x, pq * gq[j]);
    gq[j] = fma(qp, x, qq * gq[j]);
  }
  *a = swap ? b2 : a2;
  *b = swap ? a2 : b2;
  return true;
}

// Columns of G in LDS, `cols` of them (even), one pair per group of LPP lanes.
template <int NR, int LPP>
struct EjLds {
  static constexpr int PITCH = NR * LPP + 2;
  double* G;
  double* nrm2;
  int grp, li;

  __device__ void load(double* g, int col) const {
    const double* src = G + col * PITCH + li;
#pragma unroll
    for (int j = 0; j < NR; ++j) g[j] = src[LPP * j];
  }
  __device__ void store(const double* g, int col) const {
    double* dst = G + col * PITCH + li;
#pragma unroll
    for (int j = 0; j < NR; ++j) dst[LPP * j] = g[j];
  }
  __device__ void norms(int cols, int groups) const {
    for (int p = grp; p < cols; p += groups) {
      double g[NR], s = 0.0;
      load(g, p);
#pragma unroll
      for (int j = 0; j < NR; ++j) s = fma(g[j], g[j], s);
      s = ej_group_sum<LPP>(s);
      if (li == 0) nrm2[p] = s;
    }
  }
  // all pairs among `cols` columns: cols - 1 rounds of cols / 2 disjoint pairs; was any rotation coarse?
  __device__ bool all_pairs(int cols) const {
    bool coarse = false;
    const int np1 = cols - 1;
    int pn = grp, qn = grp == 0 ? np1 : np1 - grp;  // round r: (r + grp) mod np1 against (r - grp) mod np1
    for (int round = 0; round < np1; ++round) {
      const int p = pn < qn ? pn : qn, q = pn < qn ? qn : pn;
      pn = pn + 1 == np1 ? 0 : pn + 1;              // (worked out before the barrier)
      if (grp != 0) qn = qn + 1 == np1 ? 0 : qn + 1;
      if (grp < cols / 2) {
        double gp[NR], gq[NR];
        load(gp, p);
        load(gq, q);
        double a = nrm2[p], b = nrm2[q];
        if (ej_pair<NR, LPP>(gp, gq, &a, &b, &coarse)) {
          store(gp, p);
          store(gq, q);
          if (li == 0) { nrm2[p] = a; nrm2[q] = b; }
        }
      }
      __syncthreads();
    }
    return coarse;
  }
  // every column 0 .. b-1 with every column b .. 2b-1: b rounds, the first one kept in registers
  __device__ bool cross_pairs(int b) const {
    bool coarse = false;
    double gp[NR], a = 0.0;
    if (grp < b) { load(gp, grp); a = nrm2[grp]; }
    for (int round = 0; round < b; ++round) {
      if (grp < b) {
        int q = grp + round;
        if (q >= b) q -= b;
        q += b;
        double gq[NR];
        load(gq, q);
        double bb = nrm2[q];
        if (ej_pair<NR, LPP>(gp, gq, &a, &bb, &coarse)) {
          store(gq, q);
          if (li == 0) nrm2[q] = bb;
        }
      }
      __syncthreads();
    }
    if (grp < b) {
      store(gp, grp);
      if (li == 0) nrm2[grp] = a;
    }
    __syncthreads();
    return coarse;
  }
};

// Entry (r, c) of the Cholesky factor: strict lower triangle in L (pitch kp), the diagonal as the
// reciprocal of the inverted diagonal blocks' own.
__device__ inline double ej_factor_entry(const double* L, const double* Dinv, int kp, int l, int r, int c) {
  if (r >= l || c >= l || r < c) return 0.0;
  if (r > c) return L[(int64_t)r * kp + c];
  const double d = Dinv[(int64_t)(r >> 4) * 256 + (r & 15) * 17];
  return d != 0.0 ? 1.0 / d : 0.0;
}

// Ranks lam[0 .. l-1] (descending, ties by index) into order[]; thread 0 picks the number of columns to
// keep.  Adaptive rank (energy_rank): with s_i = sqrt(lambda_i) in descending order -- the singular
// values of the factor whose Gram matrix A is -- the smallest count with s_1 + ... + s_k_eff >=
// energy * (s_1 + ... + s_l), at most k (the retained-energy count of Section 2).
__device__ inline void ej_rank(const double* lam, int* order, int* keep_out, int l, int k, double energy,
                               bool energy_rank, int threads) {
  for (int i = threadIdx.x; i < l; i += threads) order[ej_rank_of(lam, l, i)] = i;
  __syncthreads();
  if (threadIdx.x == 0) {
    int keep = k;
    if (energy_rank) {
      double total = 0.0;
      for (int i = 0; i < l; ++i) total += sqrt(lam[order[i]]);
      double run = 0.0;
      keep = l;
      for (int i = 0; i < l; ++i) {
        run += sqrt(lam[order[i]]);
        if (run >= energy * total) { keep = i + 1; break; }
      }
      if (keep > k) keep = k;
    }
    *keep_out = keep;
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
  return g.work + (size_t)ej_blocks(g.l) * ej_block_cols(g.l) * ej_pitch(g.l);
}
__host__ __device__ inline int32_t* ej_words(const EjArgs& g) { return (int32_t*)(ej_lam(g) + LORACT_MAX_RANK); }

// ---------------------------------------------------------------------------------------------
// Orders up to 96: one workgroup, everything in LDS.  NR = rows per lane.
template <int NR, int THREADS>
__global__ __launch_bounds__(THREADS) void jacobi_one_kernel(EjArgs g) {
  extern __shared__ __attribute__((aligned(16))) double ej_smem[];
  __shared__ int rotated, k_eff;
  constexpr int pitch = EjLds<NR, EJ_ONE_LPP>::PITCH;
  const int l = g.l, cols = l + (l & 1), t = threadIdx.x;
  EjLds<NR, EJ_ONE_LPP> m;
  m.G = ej_smem;
  m.nrm2 = ej_smem + cols * pitch;
  m.grp = t / EJ_ONE_LPP; m.li = t % EJ_ONE_LPP;
  double* const lam = m.nrm2;                          // the squared norms at the end
  int* const order = (int*)(m.nrm2 + cols);
  for (int e = t; e < cols * pitch; e += THREADS) {    // row by row of L: coalesced reads
    const int r = e / cols, c = e - r * cols;
    m.G[c * pitch + r] = ej_factor_entry(g.L, g.Dinv, g.kp, l, r, c);
  }
  __syncthreads();
  for (int sweep = 0; sweep < EJ_MAX_SWEEPS; ++sweep) {
    m.norms(cols, THREADS / EJ_ONE_LPP);                       // afresh once per sweep
    if (t == 0) rotated = 0;
    __syncthreads();
    if (m.all_pairs(cols) && m.li == 0) rotated = 1;
    __syncthreads();
    const int again = rotated;
    __syncthreads();
    if (!again) break;
  }
  m.norms(cols, THREADS / EJ_ONE_LPP);
  __syncthreads();
  ej_rank(lam, order, &k_eff, l, g.k, g.energy, g.k_out != nullptr, THREADS);
  if (t == 0 && g.k_out) *g.k_out = k_eff;
  for (int e = t; e < l * g.k; e += THREADS) {
    const int r = e / g.k, c = e - r * g.k;
    double v = 0.0;
    if (c < k_eff) {
      const double nv = lam[order[c]];
      if (nv > 0.0) v = m.G[order[c] * pitch + r] / sqrt(nv);
    }
    g.Wk[e] = v;
  }
}

// ---------------------------------------------------------------------------------------------
// Orders above 96: blocks of columns in a work buffer.

// The columns of L; the eigenvalues (which workgroups that give up never write) and the shared words cleared.
__global__ __launch_bounds__(256) void jacobi_init_kernel(EjArgs g) {
  const int cols = ej_blocks(g.l) * ej_block_cols(g.l), pitch = ej_pitch(g.l);
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
// at most ten, whatever else runs ends and makes room, and every wait is bounded (then the status
// word says LORACT_STATUS_INTERNAL and the workgroup ends).
template <int NR>
__global__ __launch_bounds__(EJ_BLK_LPP * EJ_BLOCK) void jacobi_blocks_kernel(EjArgs g) {
  constexpr int THREADS = EJ_BLK_LPP * EJ_BLOCK, NWV = THREADS / 64;
  extern __shared__ __attribute__((aligned(16))) double ej_smem[];
  __shared__ int rotated, go_on;
  constexpr int pitch = EjLds<NR, EJ_BLK_LPP>::PITCH;
  const int nb = ej_blocks(g.l), b = ej_block_cols(g.l);
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  int32_t* const version = ej_words(g);
  int32_t* const sweep_rot = version + 64;
  int32_t* const sweep_in = sweep_rot + EJ_MAX_SWEEPS;
  EjLds<NR, EJ_BLK_LPP> m;
  m.G = ej_smem;
  m.nrm2 = ej_smem + 2 * b * pitch;
  m.grp = t / EJ_BLK_LPP; m.li = t % EJ_BLK_LPP;
  const int block_doubles = b * pitch;                 // even, so a block is whole 16-byte pieces

  // thread 0 polls until `word` has reached `want`; false when the wait ran out
  auto wait_for = [&](const int32_t* word, int want) {
    for (int spin = 0; spin < EJ_SPIN_LIMIT; ++spin) {
      if (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want) return true;
      __builtin_amdgcn_s_sleep(1);
    }
    return false;
  };

  int step = 0;
  for (int sweep = 0; sweep < EJ_MAX_SWEEPS; ++sweep) {
    bool any = false;
    for (int round = 0; round < nb - 1; ++round, ++step) {
      int p = round + blockIdx.x;
      if (p >= nb - 1) p -= nb - 1;
      int q = round + nb - 1 - blockIdx.x;
      if (q >= nb - 1) q -= nb - 1;
      if (blockIdx.x == 0) q = nb - 1;
      if (p > q) { const int tmp = p; p = q; q = tmp; }
      if (t == 0) go_on = wait_for(version + p, step) && wait_for(version + q, step);
      __syncthreads();
      if (!go_on) break;                               // (uniform)
      for (int h = 0; h < 2; ++h) {
        const double* src = g.work + (int64_t)(h ? q : p) * block_doubles;
        unsigned char* dst = (unsigned char*)(m.G + h * block_doubles);
        for (int e = wave * 64; 2 * e < block_doubles; e += NWV * 64)      // 64 pieces of 16 bytes per wave
          if (2 * (e + lane) < block_doubles) sb_async16_device(src + 2 * (e + lane), dst + 16 * e);
      }
      SB_WAIT_VMCNT(0);
      __syncthreads();
      m.norms(2 * b, EJ_BLOCK);
      __syncthreads();
      any |= round == 0 ? m.all_pairs(2 * b) : m.cross_pairs(b);
      for (int h = 0; h < 2; ++h) {
        double* dst = g.work + (int64_t)(h ? q : p) * block_doubles;
        for (int e = t; e < block_doubles; e += THREADS)
          __hip_atomic_store(dst + e, m.G[h * block_doubles + e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();                                 // every wave's stores are complete
      if (t == 0) {
        __hip_atomic_store(version + p, step + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(version + q, step + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      if (round == nb - 2) {                           // this sweep's last holder of the blocks: their squared norms
        m.norms(2 * b, EJ_BLOCK);
        __syncthreads();
        for (int c = t; c < 2 * b; c += THREADS) {
          const int col = (c < b ? p : q - 1) * b + c;
          if (col < g.l) ej_lam(g)[col] = m.nrm2[c];
        }
      }
    }
    if (!go_on) break;
    if (t == 0) rotated = 0;
    __syncthreads();
    if (any && m.li == 0) rotated = 1;
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

// Wk from the converged columns: every workgroup ranks the eigenvalues and writes its share.
__global__ __launch_bounds__(256) void jacobi_finish_kernel(EjArgs g) {
  __shared__ double lam[LORACT_MAX_RANK];
  __shared__ int order[LORACT_MAX_RANK];
  __shared__ int k_eff;
  const int l = g.l, pitch = ej_pitch(l);
  for (int i = threadIdx.x; i < l; i += 256) lam[i] = ej_lam(g)[i];
  __syncthreads();
  ej_rank(lam, order, &k_eff, l, g.k, g.energy, g.k_out != nullptr, 256);
  if (threadIdx.x == 0 && blockIdx.x == 0 && g.k_out) *g.k_out = k_eff;
  for (int e = blockIdx.x * 256 + threadIdx.x; e < l * g.k; e += gridDim.x * 256) {
    const int c = e / l, r = e - c * l;                // down the columns: the reads are the chain
    double v = 0.0;
    if (c < k_eff) {
      const double nv = lam[order[c]];
      if (nv > 0.0) v = g.work[(int64_t)order[c] * pitch + r] / sqrt(nv);
    }
    g.Wk[r * g.k + c] = v;
  }
}

template <int NR, int THREADS>
static int launch_jacobi_one(hipStream_t s, const EjArgs& g) {
  const int cols = g.l + (g.l & 1);
  const size_t lds = ((size_t)cols * ej_pitch(g.l) + cols) * sizeof(double) + (size_t)cols * sizeof(int);
  static std::atomic<bool> attr_done{false};
  if (lds > 64 * 1024 && !attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)jacobi_one_kernel<NR, THREADS>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(eigensolver LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("jacobi_eig", s, (jacobi_one_kernel<NR, THREADS>), dim3(1), dim3(THREADS), lds, g);
  return LORACT_OK;
}
template <int NR>
static int launch_jacobi_blocks(hipStream_t s, const EjArgs& g) {
  const int b = ej_block_cols(g.l);
  const size_t lds = (size_t)2 * b * (ej_pitch(g.l) + 1) * sizeof(double);   // two blocks and the squared norms
  static std::atomic<bool> attr_done{false};
  if (lds > 64 * 1024 && !attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)jacobi_blocks_kernel<NR>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(eigensolver LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("jacobi_init", s, jacobi_init_kernel, dim3(64), dim3(256), 0, g);
  LORACT_LAUNCH("jacobi_eig", s, (jacobi_blocks_kernel<NR>), dim3(ej_blocks(g.l) / 2), dim3(EJ_BLK_LPP * EJ_BLOCK), lds, g);
  LORACT_LAUNCH("jacobi_finish", s, jacobi_finish_kernel, dim3(64), dim3(256), 0, g);
  return LORACT_OK;
}

// L, Dinv: the Cholesky factor of the l x l matrix as the kernels of ortho_f64.h leave it.
static int launch_jacobi_eig(hipStream_t s, const EjArgs& g) {
  if (g.l < 1 || g.l > LORACT_MAX_RANK || g.k < 1 || g.k > g.l) return LORACT_ERR_INVALID_ARG;
#define EJ_ONE(LMAX) if (g.l <= LMAX) return launch_jacobi_one<LMAX / EJ_ONE_LPP, LMAX * EJ_ONE_LPP / 2 < 64 ? 64 : LMAX * EJ_ONE_LPP / 2>(s, g);
#define EJ_BLK(LMAX) if (g.l <= LMAX) return launch_jacobi_blocks<LMAX / EJ_BLK_LPP>(s, g);
  EJ_ONE(32) EJ_ONE(64) EJ_ONE(96)
  EJ_BLK(160) EJ_BLK(288)
  return launch_jacobi_blocks<320 / EJ_BLK_LPP>(s, g);
}
