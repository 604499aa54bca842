// Both rounds of the Cholesky QR of a small sketch by ONE workgroup in one launch.
//
// What bounds it: nothing but latency.  A sketch of a few hundred rows and up to 48 columns is a few hundred matrix
// instructions and two pivot chains, but as separate launches (Gram matrix, its sum, factor and solve, twice,
// and the conversion: seven on the bf16 path, eight on the float32 path) it paid 2 to 5 us for each and the
// host's 4.5 us to enqueue it.  One workgroup sums its Gram matrix in LDS, and a workgroup barrier replaces the
// end of a launch.
#pragma once
#include "common.h"
#include "ortho_f64.h"
#include "chol.h"

// ---------------------------------------------------------------------------------------------
// bf16 path: float32 sketch Y (m x kp), kp = 16 NJ <= 48.

// Lower 16 x 16 tiles of S^T S (float64) to G and, if given, G_backup; with e2 given, ||S^T S - I||_F^2 of the live
// k x k part to *e2.  512 threads: wave w takes the 16-row trips (w & 3), (w & 3) + 4, ... and every second tile;
// the four shares of a tile are added up in the order of the waves.  red: 3 * tiles * 256 + 8 doubles of LDS.
template <int NJ>
__device__ __forceinline__ void ortho_small_gram(const float* S, int m, int k, double* G, double* G_backup, double* red,
                                                 double* e2) {
  constexpr int KP = 16 * NJ, TILES = NJ * (NJ + 1) / 2;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lc = lane & 15, lr = lane >> 4, rg = wave & 3, half = wave >> 2;
  f64x4 acc[TILES];
#pragma unroll
  for (int i = 0; i < TILES; ++i) acc[i] = (f64x4){0.0, 0.0, 0.0, 0.0};
  float f[2][4][NJ];
  auto load_trip = [&](int r0, float (*d)[NJ]) {       // unconditional loads from clamped rows, masked at use
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int row = r0 + 4 * u + lr;
      const float* src = S + (int64_t)(row < m ? row : m - 1) * KP + lc;
#pragma unroll
      for (int b = 0; b < NJ; ++b) d[u][b] = src[16 * b];
    }
  };
  auto mac_trip = [&](int r0, const float (*d)[NJ]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = r0 + 4 * u + lr < m;
      double v[NJ];
#pragma unroll
      for (int b = 0; b < NJ; ++b) v[b] = on ? (double)d[u][b] : 0.0;
#pragma unroll
      for (int i = 0; i < NJ; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) {
          const int tile = i * (i + 1) / 2 + j;
          if ((tile & 1) == half) acc[tile] = mfma_f64(v[i], v[j], acc[tile]);
        }
    }
  };
  load_trip(16 * rg, f[0]);
  for (int r0 = 16 * rg; r0 < m; r0 += 128) {
    load_trip(r0 + 64, f[1]);
    mac_trip(r0, f[0]);
    load_trip(r0 + 128, f[0]);
    mac_trip(r0 + 64, f[1]);
  }
  // (register r of lane l is element 64 r + l of a row-major tile)
#pragma unroll
  for (int i = 0; i < TILES; ++i)
    if ((i & 1) == half && rg > 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((rg - 1) * TILES + i) * 256 + 64 * r + lane] = acc[i][r];
    }
  __syncthreads();
  double share = 0.0;
  if (rg == 0) {
#pragma unroll
    for (int i = 0; i < NJ; ++i)
#pragma unroll
      for (int j = 0; j <= i; ++j) {
        const int tile = i * (i + 1) / 2 + j;
        if ((tile & 1) != half) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          double s = acc[tile][r];
#pragma unroll
          for (int w = 0; w < 3; ++w) s += red[(w * TILES + tile) * 256 + 64 * r + lane];
          const int row = 16 * i + 4 * r + lr, col = 16 * j + lc;
          G[row * KP + col] = s;
          if (G_backup) G_backup[gram_backup_at(row, col, KP)] = s;
          const double ev = row < k && col < k ? s - (row == col ? 1.0 : 0.0) : 0.0;
          share += (i == j ? 1.0 : 2.0) * ev * ev;
        }
      }
  }
  if (e2) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) share += __shfl_xor(share, off);
    if (rg == 0 && lane == 0) red[3 * TILES * 256 + half] = share;
    __syncthreads();
    *e2 = red[3 * TILES * 256] + red[3 * TILES * 256 + 1];
  }
  __syncthreads();                                     // G is in memory for the whole workgroup, red is free
}

// c: the rounds' common settings (G, G_backup, Dinv, thresholds of round 1, tol of round 2); t: the final output (Y, L
// and Dinv are filled in here).  Round 2 either finds Q1 orthonormal to exact_tol and converts it, or factors again.
template <int NJ>
__global__ __launch_bounds__(CR_THREADS) void ortho_small_kernel(const float* Y, float* Q1, CholArgs c, TrsmArgs t,
                                                                 double exact_tol) {
  extern __shared__ __attribute__((aligned(16))) double small_lds[];
  const int m = (int)t.m;
  ortho_small_gram<NJ>(Y, m, c.k, c.G, const_cast<double*>(c.G_backup), small_lds, nullptr);
  c.round = 1;
  chol_reg_body<NJ, false>(c, small_lds);
  __syncthreads();
  TrsmArgs t1 = t;
  t1.Y = Y; t1.Q = Q1; t1.ldq = c.kp; t1.out_ek = EK_F32; t1.out_cols = c.kp; t1.Qb = nullptr;
  trsm_body<NJ, CR_THREADS / 64>(t1, 0, 1, small_lds);
  __syncthreads();
  double e2;
  ortho_small_gram<NJ>(Q1, m, c.k, c.G, nullptr, small_lds, &e2);
  if (e2 <= exact_tol * exact_tol) {                   // (uniform; false for NaN)
    const int c4 = c.kp >> 2, l = c.k;
    const bool vec_ok = basis_vec_ok(t.Q, t.Qb, l);
    for (int e = threadIdx.x; e < m * c4; e += CR_THREADS) {
      const int r = e / c4, col = (e - r * c4) << 2;
      basis_store(*(const f32x4*)(Q1 + (int64_t)r * c.kp + col), r, col, l, t.Q, t.out_ek, t.Qb, vec_ok);
    }
    return;
  }
  c.round = 2;
  chol_reg_body<NJ, false>(c, small_lds);
  __syncthreads();
  t.Y = Q1;
  trsm_body<NJ, CR_THREADS / 64>(t, 0, 1, small_lds);
}

// Up to 8192 entries of the sketch and 48 columns.  Whole compress of m x 512, one launch against seven, us: rank 16
// 128 rows 27 against 42, 512 34 against 43, 1024 44 against 43; rank 32 128 rows 33 against 45, 256 38 against
// 44, 400 49 against 46; rank 48 170 rows 47 against 50 and, where the spectrum calls for a second factorisation, 59 against
// 63, 400 rows 63 against 50.  At 64 columns the separate launches have the first-order finish instead of a second
// factorisation, which this kernel does not match: rank 64, 128 rows, spectrum i^-1.5 62 against 53 (without a
// second round 48 against 51).
static inline bool ortho_small_fits(int64_t m, int kp) { return kp <= 48 && m * kp <= 8192; }

template <int NJ>
static int launch_ortho_small_nj(hipStream_t s, const float* Y, float* Q1, const CholArgs& c, const TrsmArgs& t, double exact_tol) {
  constexpr int TILES = NJ * (NJ + 1) / 2;
  const size_t lds = std::max({chol_reg_lds_bytes(16 * NJ), trsm_lds_bytes<NJ, CR_THREADS / 64>(),
                               (size_t)(3 * TILES * 256 + 8) * sizeof(double)});
  LORACT_LAUNCH("ortho_small", s, ortho_small_kernel<NJ>, dim3(1), dim3(CR_THREADS), lds, Y, Q1, c, t, exact_tol);
  return LORACT_OK;
}
static int launch_ortho_small(hipStream_t s, const float* Y, float* Q1, const CholArgs& c, const TrsmArgs& t, double exact_tol) {
  switch (c.kp / 16) {
    case 1: return launch_ortho_small_nj<1>(s, Y, Q1, c, t, exact_tol);
    case 2: return launch_ortho_small_nj<2>(s, Y, Q1, c, t, exact_tol);
    case 3: return launch_ortho_small_nj<3>(s, Y, Q1, c, t, exact_tol);
    default: return LORACT_ERR_UNSUPPORTED;
  }
}

// ---------------------------------------------------------------------------------------------
// float32 path: float64 sketch Y (m x l), l <= 16, at most OS_MAX_ROWS rows.  A wave keeps its strips of 16 rows in
// registers through both rounds: as the Gram product takes them (register r of lane q: row 4 r + q / 16, column
// q % 16), turned through LDS for the product with R^{-1} (row q % 16, column 4 r + q / 16, whose result has the same
// layout) and back.  Factor and inverse are chol_inverse_wave's, on the first wave.
#define OS_WAVES 8
#define OS_STRIPS 8
#define OS_MAX_ROWS (16 * OS_WAVES * OS_STRIPS)
#define OS_GROUP 2
#define OS_TP 17
static_assert(4 * OS_STRIPS * 64 <= OS_WAVES * 256, "a wave's strips have to fit the room of the shares");
template <int STRIPS, bool ROWS>
__global__ __launch_bounds__(64 * OS_WAVES) void ortho_small_f64_kernel(const double* Y, int m, int l, double tol, double shift1,
                                                                        double* Q, float* q32, int32_t* status) {
  __shared__ double G[16 * 17], Rinv[16 * 17], tiles[OS_WAVES][OS_GROUP][16 * OS_TP], red[OS_WAVES][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lc = lane & 15, lr = lane >> 4;
  double (*const tile)[16 * OS_TP] = tiles[wave];
  double y[STRIPS][4];
#pragma unroll
  for (int s = 0; s < STRIPS; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (wave + OS_WAVES * s) * 16 + 4 * r + lr;
      const double v = Y[(int64_t)(row < m ? row : m - 1) * l + (lc < l ? lc : l - 1)];
      y[s][r] = row < m && lc < l ? v : 0.0;
    }
#pragma unroll 1
  for (int round = 0; round < 2; ++round) {
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < STRIPS; ++s)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc = mfma_f64(y[s][r], y[s][r], acc);
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][64 * r + lane] = acc[r];
    __syncthreads();
    if (threadIdx.x < 256) {                             // the shares in the order of the waves
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < OS_WAVES; ++w) s += red[w][threadIdx.x];
      G[(threadIdx.x >> 4) * 17 + (threadIdx.x & 15)] = s;
    }
    __syncthreads();
    if (wave == 0) {
      // (eight strips and the pivots' rows do not fit the registers together: the strips wait in the room of the shares)
      double* const save = &red[0][0] + lane;
      if constexpr (ROWS && STRIPS == OS_STRIPS) {
#pragma unroll
        for (int i = 0; i < 4 * STRIPS; ++i) save[64 * i] = y[i >> 2][i & 3];
        asm volatile("" : : : "memory");
      }
      chol_inverse_wave<16, ROWS>(G, 17, Rinv, 17, l, tol, round == 0 ? shift1 : 0.0, status, lane);
      if constexpr (ROWS && STRIPS == OS_STRIPS) {
        asm volatile("" : : : "memory");
#pragma unroll
        for (int i = 0; i < 4 * STRIPS; ++i) y[i >> 2][i & 3] = save[64 * i];
      }
    }
    __syncthreads();
    double ra[4];                                        // rows and columns of R^{-1} past l are not written: masked here
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double v = Rinv[(4 * r + lr) * 17 + lc];
      ra[r] = 4 * r + lr < l && lc < l ? v : 0.0;
    }
#pragma unroll
    for (int s0 = 0; s0 < STRIPS; s0 += OS_GROUP) {      // OS_GROUP strips side by side
      f64x4 yt[OS_GROUP], o[OS_GROUP];
#pragma unroll
      for (int g = 0; g < OS_GROUP; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) tile[g][(4 * r + lr) * OS_TP + lc] = y[s0 + g][r];
      sb_wave_sync();
#pragma unroll
      for (int g = 0; g < OS_GROUP; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) yt[g][r] = tile[g][lc * OS_TP + 4 * r + lr];
      sb_wave_sync();
#pragma unroll
      for (int g = 0; g < OS_GROUP; ++g) o[g] = (f64x4){0.0, 0.0, 0.0, 0.0};   // Q^T: register r is column 4 r + q / 16, row q % 16
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int g = 0; g < OS_GROUP; ++g) o[g] = mfma_f64(ra[r], yt[g][r], o[g]);
#pragma unroll
      for (int g = 0; g < OS_GROUP; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) tile[g][lc * OS_TP + 4 * r + lr] = o[g][r];
      sb_wave_sync();
#pragma unroll
      for (int g = 0; g < OS_GROUP; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[s0 + g][r] = tile[g][(4 * r + lr) * OS_TP + lc];
      sb_wave_sync();
    }
  }
#pragma unroll
  for (int s = 0; s < STRIPS; ++s)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = (wave + OS_WAVES * s) * 16 + 4 * r + lr;
      if (row < m && lc < l) {
        Q[(int64_t)row * l + lc] = y[s][r];
        if (q32) q32[(int64_t)row * l + lc] = (float)y[s][r];
      }
    }
}

// Whole compress at rank 16 without waiting for the host, one launch against eight, us: 256 rows 27 against 39 (256
// wide), 512 35 against 45, 900 45 against 45, 1024 46 against 45; 768 wide 1024 rows 50 against 48 (rank 12 48 against 45):
// from 900 rows on the passes of one CU over the rows take a little more than the launches did.  A program that enqueues
// its steps one by one waits for the host there, and that has seven launches fewer: 1024 x 256, step 80 -> 62 us.
// (Sixteen waves of four strips above 512 rows: 44 us at 1024 x 256, 48 at 1024 x 768, but 54 against 51 at 1024 x 2048.)
// Beyond 16 columns the pivots of the first wave take the gain (24 columns, 128 rows: 61 against 51), beyond 1024 rows the
// registers end.
static inline bool ortho_small_f64_fits(int64_t m, int l) { return l <= 16 && m <= OS_MAX_ROWS; }
static int launch_ortho_small_f64(hipStream_t s, const double* Y, int m, int l, double tol, double shift1, double* Q,
                                  float* q32, int32_t* status) {
  const int strips = (m + 16 * OS_WAVES - 1) / (16 * OS_WAVES);
#define OS_LAUNCH(STRIPS, ROWS)                                                                                                  \
  LORACT_LAUNCH("ortho_small", s, (ortho_small_f64_kernel<STRIPS, ROWS>), dim3(1), dim3(64 * OS_WAVES), 0, Y, m, l, tol, shift1, \
                Q, q32, status)
  if (l < CHOL_ROWS_MIN) {
    if (strips <= 2) OS_LAUNCH(2, false);
    else if (strips <= 4) OS_LAUNCH(4, false);
    else OS_LAUNCH(OS_STRIPS, false);
  } else {
    if (strips <= 2) OS_LAUNCH(2, true);
    else if (strips <= 4) OS_LAUNCH(4, true);
    else OS_LAUNCH(OS_STRIPS, true);
  }
#undef OS_LAUNCH
  return LORACT_OK;
}
