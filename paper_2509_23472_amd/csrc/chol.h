// Cholesky factorisation of a small Gram matrix and inversion of its triangular factor, in
// float64, by one workgroup.
//
// For a tall-skinny Y with Gram matrix G = Y^T Y = L L^T the orthonormal factor of the thin QR
// of Y is Q = Y L^{-T}; this kernel turns G into Rinv = L^{-T} (upper triangular) so that the
// factor can be applied as a plain matrix product.
//
// Two modes, used as the two rounds of a shifted Cholesky QR:
//  * shift_rel > 0 (first round): factor G + s I with s = shift_rel * trace(G).  The shift keeps
//    the factorisation defined when cond(Y)^2 exceeds what float64 resolves; Q1 = Y Rinv still
//    spans range(Y) exactly (Rinv is invertible) and has cond(Q1) ~ cond(Y) * sqrt(shift_rel),
//    small enough for an unshifted second round.
//  * shift_rel == 0 (second round): plain Cholesky.
// Breakdown rule (second round): after the first round the columns of Q1 are scaled to O(1) and
// stored in at most float32, so a pivot not larger than tol * G[j][j] with tol = (k 2^-24)^2 means
// column j depends on the earlier columns to within float32 resolution (exact duplicates among
// the sampled rows, or an all-zero sampled row).  Its reciprocal pivot is set to zero, which
// zeroes column j of L below the diagonal and the whole column j of Rinv: the matching column
// of Q becomes zero, the other columns are exactly what they would be with column j removed,
// and the status word gets LORACT_STATUS_RANK_DEFICIENT.  The shifted first round only clamps
// (and flags) a pivot that is not positive at all.
#pragma once
#include "common.h"
#include "ortho_f64.h"    // readlane_f64, rsqrt_f64, chol_clamp_tol

#define CH_NB 16

__global__ __launch_bounds__(256) void chol_inverse_kernel(double* G, double* Rinv, int k,
                                                           double tol, double shift_rel,
                                                           int32_t* status) {
  __shared__ double Ds[CH_NB][CH_NB + 1];
  __shared__ double Di[CH_NB][CH_NB + 1];
  __shared__ double Ps[LORACT_MAX_RANK * (CH_NB + 1)];  // panel [row][17], later W [16][k+1]
  __shared__ double dinv[LORACT_MAX_RANK];
  __shared__ double gdiag[LORACT_MAX_RANK];
  __shared__ int deficient;
  __shared__ double shift_s;

  const int t = threadIdx.x;
  const int tr = t >> 4, tc = t & 15;
  for (int i = t; i < k; i += 256) gdiag[i] = G[(int64_t)i * k + i];
  if (t == 0) deficient = 0;
  __syncthreads();
  if (t == 0) {
    double tr_sum = 0.0;
    for (int i = 0; i < k; ++i) tr_sum += gdiag[i];
    shift_s = shift_rel * tr_sum;
  }
  __syncthreads();
  const double shift = shift_s;

  // ---- phase A: G = L L^T, L left in the strict lower triangle of G, 1/L[j][j] in dinv.
  for (int jb = 0; jb < k; jb += CH_NB) {
    const int nb = (k - jb < CH_NB) ? (k - jb) : CH_NB;
    if (tr < nb && tc < nb)
      Ds[tr][tc] = G[(int64_t)(jb + tr) * k + jb + tc] + (tr == tc ? shift : 0.0);
    __syncthreads();
    for (int j = 0; j < nb; ++j) {
      const double piv = Ds[j][j];
      const bool usable = shift > 0.0 ? (piv > 0.0) : (piv > tol * gdiag[jb + j]);
      const bool bad = !usable;
      const double di = usable ? 1.0 / sqrt(piv) : 0.0;
      if (t == 0) {
        dinv[jb + j] = di;
        if (bad) deficient = 1;
      }
      if (t > j && t < nb) Ds[t][j] *= di;
      __syncthreads();
      if (tr < nb && tc > j && tc <= tr) Ds[tr][tc] -= Ds[tr][j] * Ds[tc][j];
      __syncthreads();
    }
    if (tr < nb && tc < tr) G[(int64_t)(jb + tr) * k + jb + tc] = Ds[tr][tc];

    // panel below the diagonal block: solve X * Lbb^T = G[i][jb..jb+nb) row by row
    const int below = jb + nb;
    for (int i = below + t; i < k; i += 256) {
      double x[CH_NB];
#pragma unroll
      for (int c = 0; c < CH_NB; ++c) x[c] = (c < nb) ? G[(int64_t)i * k + jb + c] : 0.0;
#pragma unroll
      for (int c = 0; c < CH_NB; ++c) {
        if (c < nb) {
          double s = x[c];
#pragma unroll
          for (int c2 = 0; c2 < CH_NB; ++c2)
            if (c2 < c) s -= x[c2] * Ds[c][c2];
          x[c] = s * dinv[jb + c];
        }
      }
#pragma unroll
      for (int c = 0; c < CH_NB; ++c) {
        if (c < nb) G[(int64_t)i * k + jb + c] = x[c];
        Ps[(i - below) * (CH_NB + 1) + c] = x[c];
      }
    }
    __syncthreads();
    // trailing update of the lower triangle
    const int nrem = k - below;
    for (int e = t; e < nrem * nrem; e += 256) {
      const int ri = e / nrem, ci = e - ri * nrem;
      if (ci <= ri) {
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < CH_NB; ++c) s += Ps[ri * (CH_NB + 1) + c] * Ps[ci * (CH_NB + 1) + c];
        G[(int64_t)(below + ri) * k + below + ci] -= s;
      }
    }
    __syncthreads();
  }

  // ---- phase B: Linv = L^{-1} (lower), written transposed: Rinv[c][i] = Linv[i][c].
  for (int e = t; e < k * k; e += 256) Rinv[e] = 0.0;
  __syncthreads();
  double* Ws = Ps;  // [CH_NB][k + 1]
  const int wld = k + 1;
  for (int ib = 0; ib < k; ib += CH_NB) {
    const int nb = (k - ib < CH_NB) ? (k - ib) : CH_NB;
    if (tr < nb && tc < nb) {
      Ds[tr][tc] = (tc < tr) ? G[(int64_t)(ib + tr) * k + ib + tc] : 0.0;
      Di[tr][tc] = 0.0;
    }
    __syncthreads();
    // inverse of the diagonal block, one thread per column
    if (t < nb) {
      const int c = t;
      double x[CH_NB];
#pragma unroll
      for (int r = 0; r < CH_NB; ++r) x[r] = 0.0;
#pragma unroll
      for (int r = 0; r < CH_NB; ++r) {
        if (r == c) x[r] = dinv[ib + c];
        else if (r > c && r < nb) {
          double s = 0.0;
#pragma unroll
          for (int j = 0; j < CH_NB; ++j)
            if (j >= c && j < r) s += Ds[r][j] * x[j];
          x[r] = -s * dinv[ib + r];
        }
      }
#pragma unroll
      for (int r = 0; r < CH_NB; ++r)
        if (r < nb) Di[r][c] = x[r];
    }
    // W[r][c] = sum_{j=c}^{ib-1} L[ib+r][j] * Linv[j][c]   for c < ib
    for (int e = t; e < CH_NB * ib; e += 256) {
      const int c = e >> 4, r = e & 15;
      double s = 0.0;
      if (r < nb) {
        const double* lrow = G + (int64_t)(ib + r) * k;
        const double* icol = Rinv + (int64_t)c * k;
        for (int j = c; j < ib; ++j) s += lrow[j] * icol[j];
      }
      Ws[r * wld + c] = s;
    }
    __syncthreads();
    // Linv[ib+r][c] = - sum_{r2<=r} Di[r][r2] * W[r2][c]
    for (int e = t; e < CH_NB * ib; e += 256) {
      const int c = e >> 4, r = e & 15;
      if (r < nb) {
        double s = 0.0;
#pragma unroll
        for (int r2 = 0; r2 < CH_NB; ++r2)
          if (r2 <= r) s += Di[r][r2] * Ws[r2 * wld + c];
        Rinv[(int64_t)c * k + ib + r] = -s;
      }
    }
    if (tr < nb && tc <= tr) Rinv[(int64_t)(ib + tc) * k + ib + tr] = Di[tr][tc];
    __syncthreads();
  }
  if (t == 0 && deficient && status) atomicOr(status, LORACT_STATUS_RANK_DEFICIENT);
}

// The same for k <= NC = 16 or 32 by one wave without barriers: lane i holds row i of G + s I in registers,
// lane 32 + i row i of the identity, and both take the k pivot steps (scaling of the pivot column, rank-1
// update of the later ones with multipliers read from the lanes of G), which turns the first into L and
// the second into L^{-T}, i.e. R^{-1}.  A column whose pivot is not usable gets a zero reciprocal and drops
// out of both.  At k = 16 the blocked kernel's barriers and its passes through memory made 11.6 us of what is a
// chain of 16 pivots; this one takes 4.9 us.  (Beyond 32 columns a lane's rows no longer fit its registers.)
template <int NC>
__device__ __forceinline__ void chol_inverse_guarded(const double* G, int ldg, double* Rinv, int ldr, int k, double tol,
                                                     double shift_rel, int32_t* status, int lane) {
  const int r = lane & 31;
  const bool rows = lane < 32, live = r < k;
  double a[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const double v = G[(live ? r : 0) * ldg + (c < k ? c : 0)];            // unconditional loads, masked at use
    a[c] = rows ? (live && c < k ? v : 0.0) : (r == c ? 1.0 : 0.0);
  }
  const double diag = G[(live ? r : 0) * (ldg + 1)];
  double tr = rows && live ? diag : 0.0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
  const double shift = shift_rel * tr;
  const double level = shift > 0.0 ? 0.0 : tol * diag;                     // lane j: what pivot j has to exceed
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (rows && r == c) a[c] += shift;
  bool bad = false;
#pragma unroll
  for (int j = 0; j < NC; ++j) {
    if (j < k) {
      const double piv = readlane_f64(a[j], j);
      const bool usable = piv > readlane_f64(level, j);
      bad = bad || !usable;
      a[j] *= usable ? rsqrt_f64<OF_RSQ_STEPS>(piv) : 0.0;
#pragma unroll
      for (int c = j + 1; c < NC; ++c) a[c] = fma(-a[j], readlane_f64(a[j], c), a[c]);
    }
  }
  if (!rows && live) {
#pragma unroll
    for (int c = 0; c < NC; ++c)
      if (c < k) Rinv[r * ldr + c] = a[c];
  }
  if (lane == 0 && bad && status) atomicOr(status, LORACT_STATUS_RANK_DEFICIENT);
}
// From CHOL_ROWS_MIN to 16 columns (ROWS) the pivot steps are those of the wide factorisation (cr_pivots: multipliers by row broadcast,
// no test on the chain from pivot to pivot), on rows of the matrix in every row of 16 lanes, padded with unit diagonal entries; only
// when a pivot turns out unusable the form above does it over.  All 16 steps are taken, the form above takes k.  Whole float32 compress, us,
// without and with: 64 x 64 rank 11 22.1 and 19.7, rank 16 23.6 and 20.3; 1024 x 256 rank 11 43.0 and 41.3, rank 16 44.9 and 42.3 (rank 9
// the other way round, 41.9 and 42.4); 4096 x 768 rank 16 53.3 and 49.8.  Fewer columns have kernels without this form: with both in
// one, chosen at run time, they took 0.6 us longer (1.3 with eight strips, which had to make room), 64 x 64 rank 8 21.0 and 21.8, 1024 x
// 256 rank 8 41.4 and 42.7.
#define CHOL_ROWS_MIN 11
template <int NC, bool ROWS>
__device__ __forceinline__ void chol_inverse_wave(const double* G, int ldg, double* Rinv, int ldr, int k, double tol,
                                                  double shift_rel, int32_t* status, int lane) {
  if constexpr (ROWS) {
    static_assert(NC == 16, "rows of 16 lanes");
    __builtin_assume(k >= CHOL_ROWS_MIN);                                  // (no masks on the columns up to there)
    const int r = lane & 15;
    const bool live = r < k;
    double a[NC], b[NC];
    const double diag = G[(live ? r : 0) * (ldg + 1)];
    double tr = live ? diag : 0.0;
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
    const double shift = shift_rel * tr;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const double v = G[(live ? r : 0) * ldg + (c < k ? c : 0)];          // unconditional loads, masked at use
      b[c] = r == c ? 1.0 : 0.0;
      a[c] = live && c < k ? v : b[c];
      if (live && r == c) a[c] += shift;
    }
    const double level = shift > 0.0 ? 0.0 : tol * diag;
    double pivs = 0.0, piv = readlane_f64(a[0], 0), y = __builtin_amdgcn_rsq(piv);
    cr_pivots<0>(a, b, piv, y, pivs, r);
    if (!__any(live && !(pivs > level))) {                                 // (true for NaN)
      if (lane < 16 && live) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
          if (c < k) Rinv[r * ldr + c] = b[c];
      }
      return;
    }
    // (nothing of what follows is to be worked out before it is known to be needed: its masks alone cost 0.6 us)
    asm volatile("" : "+v"(lane), "+s"(k));
  }
  chol_inverse_guarded<NC>(G, ldg, Rinv, ldr, k, tol, shift_rel, status, lane);
}
template <int NC, bool ROWS>
__global__ __launch_bounds__(64) void chol_inverse_wave_kernel(const double* G, double* Rinv, int k, double tol,
                                                               double shift_rel, int32_t* status) {
  chol_inverse_wave<NC, ROWS>(G, k, Rinv, k, k, tol, shift_rel, status, (int)threadIdx.x);
}

static int launch_chol_inverse(hipStream_t stream, double* G, double* Rinv, int k,
                               double shift_rel, int32_t* status) {
  if (k < 1 || k > LORACT_MAX_RANK) return LORACT_ERR_UNSUPPORTED;
  const double tol = chol_clamp_tol(k);
  if (k < CHOL_ROWS_MIN)
    LORACT_LAUNCH("chol_inverse", stream, (chol_inverse_wave_kernel<16, false>), dim3(1), dim3(64), 0, (const double*)G, Rinv, k,
                  tol, shift_rel, status);
  else if (k <= 16)
    LORACT_LAUNCH("chol_inverse", stream, (chol_inverse_wave_kernel<16, true>), dim3(1), dim3(64), 0, (const double*)G, Rinv, k,
                  tol, shift_rel, status);
  else if (k <= 32)
    LORACT_LAUNCH("chol_inverse", stream, (chol_inverse_wave_kernel<32, false>), dim3(1), dim3(64), 0, (const double*)G, Rinv, k,
                  tol, shift_rel, status);
  else
    LORACT_LAUNCH("chol_inverse", stream, chol_inverse_kernel, dim3(1), dim3(256), 0, G, Rinv, k,
                  tol, shift_rel, status);
  return LORACT_OK;
}
