// Tall-skinny orthonormalisation kernels of the bf16 path: Gram matrix, Cholesky factor and
// triangular solve, all accumulated in float64 on the gfx950 matrix cores
// (v_mfma_f64_16x16x4_f64) without LDS staging of the operands.
//
// Layout conventions used below (verified on the device):
//   A operand (16 x 4):  lane l holds A[m = l % 16][kk = l / 16]
//   B operand (4 x 16):  lane l holds B[kk = l / 16][n = l % 16]
//   C/D      (16 x 16):  register r of lane l holds D[m = 4 r + l / 16][n = l % 16]
// so an accumulator can be fed back as the B operand of a later product whose contraction
// index is the accumulator's row index: slice r (kk = 4 r .. 4 r + 3) is register r.
//
// The sketch Y and the intermediate Q1 are stored as m x kp float32 with kp = k rounded up to a
// multiple of 16; columns k..kp-1 are zero.  The Gram matrix / Cholesky factor is kp x kp.
#pragma once
#include "common.h"
#include "gram_plan.h"
#include "progress.h"

#define OF_NB 16
#ifndef OF_RSQ_STEPS
#define OF_RSQ_STEPS 1
#endif


__device__ inline f64x4 mfma_f64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// c - a b (on float64 matrix instructions the last immediate is a set of sign bits, the first for a)
__device__ inline f64x4 mfma_f64_sub(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 1);
}

// ---------------------------------------------------------------------------------------------
// Widest matrix of the register-resident factorisation.
#define CR_MAX_KP 272
// Where entry (i, j) of the Gram matrix lies in its backup for the register-resident factorisation (kp <= CR_MAX_KP): 16 x 16 blocks one
// after the other, a block as the lanes of a wave take it, lane (q, n) entries (n, 4 q .. 4 q + 3), in two pieces of 16
// bytes, so that a load instruction of the one workgroup that reads it all covers a contiguous kilobyte (in rows of G it
// touches sixteen lines half each, four clocks a line: 136 blocks 20000 clocks).
__device__ __host__ inline int64_t gram_backup_at(int i, int j, int kp) {
  const int r = j & 3, q = (j & 15) >> 2;
  return ((int64_t)(i >> 4) * (kp >> 4) + (j >> 4)) * 256 + (r >> 1) * 128 + (16 * q + (i & 15)) * 2 + (r & 1);
}

// ---------------------------------------------------------------------------------------------
// Gram matrix G = Y^T Y of more than 64 columns.  The columns are cut into blocks of two to four 16-column tiles
// (gram_plan.h); a workgroup of eight waves takes pairs of blocks, every wave ALL tiles of the pair over every eighth group of
// four rows, and the eight add up through LDS, so that a share of the rows leaves one set of tiles, as rows and columns lie in G:
// part[(unit part_at + share * qi qj) * 256 + row * 16 qj + column].
//
// What bounds it: the float64 matrix rate, which a loop of nothing else takes to 66 TFLOP/s with one wave per SIMD and 73 with
// two (65536 x 256: 4.6 GFLOP); vector float64 instructions do not run beside it.  So the loop may hold little else.  A block
// of Q tiles interleaves its columns, tile i taking columns Q x + i, so that a lane's operands of all Q tiles are ONE load of Q
// consecutive floats (tile by tile they are Q loads); 16 matrix instructions then need two loads and eight conversions.
// Addresses are a base that moves on and a fixed lane offset, and rows past the end are looked at in the last trip
// only.  Of a diagonal pair the tiles above the diagonal are not formed.  Before, a wave took 2 x 2 tiles: four loads with
// their addresses and masks for four matrix instructions.  Product and sum, us event to event, before and after: 65536 x 256
// 119 -> 84, x 128 48 -> 34, x 80 40 -> 21; 8192 x 256 30 -> 25.5, x 320 39 -> 31, x 128 20.9 -> 19.3.  (Few rows have fewer
// matrix instructions than the sum of eight waves costs: gram_short_kernel, by gram_is_short.)
// All pairs of blocks of a slice of rows run on one XCD (workgroup b on XCD b mod 8), which then fetches its eighth of Y
// into its L2 once.

#define GRAM_RED_TILES 8         // tiles of every wave in LDS at a time
#define GRAM_TILE_PITCH 260      // doubles between two of them
#define GRAM_LDS_BYTES (GRAM_WAVES * GRAM_RED_TILES * GRAM_TILE_PITCH * sizeof(double))

// Tile (i, j) of a pair: columns ci + qi x + i and cj + qj y + j, x and y = 0 .. 15.  Tiles are numbered row by row.
template <int Q> struct GramVec { typedef float t __attribute__((ext_vector_type(Q), aligned(4))); };

template <int QI, int QJ, bool DIAG>
__device__ __forceinline__ void gram_unit(const float* Y, const int kp, const GramUnit& u, int64_t r_begin, int64_t r_end,
                                          double* out, double* red) {
  constexpr int TILES = DIAG ? QI * (QI + 1) / 2 : QI * QJ;
  constexpr int D = 4;                                  // groups of rows in flight per wave
  constexpr int STEP = GRAM_STEP;                       // rows between a wave's groups
  typedef typename GramVec<QI>::t VI;
  typedef typename GramVec<QJ>::t VJ;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lc = lane & 15, lr = lane >> 4;
  const int off_i = lr * kp + u.ci + QI * lc, off_j = lr * kp + u.cj + QJ * lc;
  f64x4 acc[TILES];
#pragma unroll
  for (int t = 0; t < TILES; ++t) acc[t] = (f64x4){0.0, 0.0, 0.0, 0.0};
  auto mac = [&](const VI& fi, const VJ& fj) {
    double a[QI], b[QJ];
#pragma unroll
    for (int i = 0; i < QI; ++i) a[i] = (double)fi[i];
#pragma unroll
    for (int j = 0; j < QJ; ++j) b[j] = DIAG ? a[j < QI ? j : 0] : (double)fj[j];
#pragma unroll
    for (int i = 0; i < QI; ++i)
#pragma unroll
      for (int j = 0; j < (DIAG ? i + 1 : QJ); ++j) {
        const int t = DIAG ? i * (i + 1) / 2 + j : i * QJ + j;
        acc[t] = mfma_f64(a[i], b[j], acc[t]);
      }
  };
  const int64_t first = r_begin + 4 * wave;
  // groups of four rows that lie inside the chunk as a whole; one more may be cut off by its end
  const int full = first + 4 <= r_end ? (int)((r_end - first - 4) / STEP) + 1 : 0;
  VI fi[D];
  VJ fj[D];
  const float* base = Y + first * kp;                 // (uniform; moves on with the group that is fetched)
  const int64_t stride = (int64_t)STEP * kp;
  auto fetch = [&](int slot) {
    fi[slot] = *(const VI*)(base + off_i);
    if (!DIAG) fj[slot] = *(const VJ*)(base + off_j);
  };
  if (full > 0) {
    int ahead = 0;                                      // group that `base` stands at
    auto fetch_next = [&](int slot) {                   // past the last group: fetched again, never multiplied
      fetch(slot);
      if (ahead + 1 < full) { ++ahead; base += stride; }
    };
#pragma unroll
    for (int p = 0; p < D - 1; ++p) fetch_next(p);
    int s = 0;
    for (; s + D <= full; s += D) {
#pragma unroll
      for (int p = 0; p < D; ++p) {
        fetch_next((p + D - 1) % D);
        mac(fi[p], fj[p]);
      }
    }
#pragma unroll
    for (int p = 0; p < D - 1; ++p)
      if (s + p < full) mac(fi[p], fj[p]);
  }
  const int64_t left = first + (int64_t)full * STEP;    // the group that the end cuts off
  if (left < r_end) {
    const bool on = left + lr < r_end;
    const float* row = Y + left * kp - (on ? 0 : (int64_t)lr * kp);      // rows past the end read its first row, as zero
    VI gi = *(const VI*)(row + off_i);
    VJ gj = *(const VJ*)(row + off_j);
#pragma unroll
    for (int i = 0; i < QI; ++i) gi[i] = on ? gi[i] : 0.0f;
#pragma unroll
    for (int j = 0; j < QJ; ++j) gj[j] = on ? gj[j] : 0.0f;
    mac(gi, gj);
  }
  // The eight waves' tiles are added up through LDS, in the order of the waves, half of the tile rows at a time, and leave as
  // rows and columns lie in G.  (Register r of lane l is element 64 r + l of a row-major tile.)  Every wave writes all of its
  // tiles: choosing the ones that it will not add up itself saves an eighth of the traffic and costs 20 KB of code that
  // runs once, from a cold instruction cache.
  constexpr int RH = (QI + 1) / 2;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    constexpr int SIZE = 64 * GRAM_WAVES;
    const int i0 = h * RH, ni = h ? QI - RH : RH;        // rows i0 .. i0 + ni - 1 of the tiles
    const int t0 = DIAG ? i0 * (i0 + 1) / 2 : i0 * QJ, t1 = DIAG ? (i0 + ni) * (i0 + ni + 1) / 2 : (i0 + ni) * QJ;
    if (h) __syncthreads();
#pragma unroll
    for (int t = 0; t < TILES; ++t)
      if (t >= t0 && t < t1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(wave * GRAM_RED_TILES + t - t0) * GRAM_TILE_PITCH + 64 * r + lane] = acc[t][r];
      }
    __syncthreads();
    for (int e = threadIdx.x; e < ni * 256 * QJ; e += SIZE) {
      const int r = e / (16 * QJ), c = e % (16 * QJ);
      const int x = r / ni, i = i0 + r % ni, y = c / QJ, j = c % QJ;
      if (DIAG && j > i) continue;                      // (not formed)
      const double* src = red + ((DIAG ? i * (i + 1) / 2 + j : i * QJ + j) - t0) * GRAM_TILE_PITCH + 16 * x + y;
      double sum = 0.0;
#pragma unroll
      for (int w = 0; w < GRAM_WAVES; ++w) sum += src[w * GRAM_RED_TILES * GRAM_TILE_PITCH];
      out[(QI * x + i) * 16 * QJ + c] = sum;
      if (DIAG && j < i) out[(QI * y + j) * 16 * QJ + QJ * x + i] = sum;
    }
  }
}

__global__ __launch_bounds__(64 * GRAM_WAVES) void gram_mfma_kernel(const float* Y, GramPlan g, double* part) {
  extern __shared__ __attribute__((aligned(16))) double gram_red[];
  double* const red = gram_red;
  const int slice = blockIdx.x % g.slices, w = blockIdx.x / g.slices;
  const int64_t slice_begin = (int64_t)slice * g.steps * GRAM_STEP;
  const GramBound from = g.bound[w], to = g.bound[w + 1];
  for (int n = from.unit; n <= to.unit; ++n) {
    const int first = n == from.unit ? from.step : 0, last = n == to.unit ? to.step : g.steps;
    if (first == last) break;                           // (the share ends with the unit before)
    const GramUnit u = g.unit[n];
    int64_t r_begin = slice_begin + (int64_t)first * GRAM_STEP, r_end = slice_begin + (int64_t)last * GRAM_STEP;
    if (r_end > g.m) r_end = g.m;
    if (r_begin > r_end) r_begin = r_end;               // (no rows: zeros)
    double* const out = part + ((int64_t)u.part_at + ((w - u.wg0) * g.slices + slice) * u.qi * u.qj) * 256;
    if (u.ci == u.cj) {
      if (u.qi == 4) gram_unit<4, 4, true>(Y, g.kp, u, r_begin, r_end, out, red);
      else if (u.qi == 3) gram_unit<3, 3, true>(Y, g.kp, u, r_begin, r_end, out, red);
      else gram_unit<2, 2, true>(Y, g.kp, u, r_begin, r_end, out, red);
    } else if (u.qi == 4) gram_unit<4, 4, false>(Y, g.kp, u, r_begin, r_end, out, red);
    else if (u.qj == 4) gram_unit<3, 4, false>(Y, g.kp, u, r_begin, r_end, out, red);
    else if (u.qi == 3) gram_unit<3, 3, false>(Y, g.kp, u, r_begin, r_end, out, red);
    else gram_unit<2, 3, false>(Y, g.kp, u, r_begin, r_end, out, red);
    __syncthreads();                                    // the next unit's tiles go through the same LDS
  }
}

// G (kp x kp, the lower triangle and all of the diagonal 16 x 16 blocks) = sum over chunks.  Grid (64, units): a workgroup
// per row of a unit, wave w adds the chunks w, w + GRAM_LANES, ... in ascending order, a column per lane, and the waves' sums
// are added in their order: a fixed order whatever the chunk count.
// Optional by-products for the second round (ns_e2 != null): with E = G - I restricted to the
// live k x k part, T = -E/2 as a full symmetric bf16 matrix (pad rows/columns zero; ns_T != null), the other triangle of
// G (mirror), and this workgroup's share of ||E||_F^2 in ns_e2[64 unit + workgroup] (an element of an off-diagonal unit
// counts twice, for its mirror image).  The consumer adds the shares in index order.
#define GRAM_LANES 8
__global__ __launch_bounds__(64 * GRAM_LANES) void gram_reduce_kernel(const double* part, GramPlan g, int k, double* G,
                                                                      double* G_copy, bf16_t* ns_T, double* ns_e2, int mirror,
                                                                      int32_t* clear_word) {
  __shared__ double sums[GRAM_LANES][64];
  // (the progress word of a fused factor-and-solve launch that follows starts at zero)
  if (clear_word && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear_word = 0;
  const GramUnit u = g.unit[blockIdx.y];
  const int chunks = u.wgs * g.slices, kp = g.kp, row = blockIdx.x, c = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool diag = u.ci == u.cj, on = row < 16 * u.qi && c < 16 * u.qj;
  const int stride = 256 * u.qi * u.qj;
  const double* const src = part + (int64_t)u.part_at * 256 + (on ? row * 16 * u.qj + c : 0);
  double s = 0.0;
  for (int c0 = wave; c0 < chunks; c0 += 8 * GRAM_LANES) {      // eight loads in flight, masked at use
    double v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = src[(int64_t)(c0 + GRAM_LANES * q < chunks ? c0 + GRAM_LANES * q : c0) * stride];
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (c0 + GRAM_LANES * q < chunks) s += v[q];
  }
  sums[wave][c] = s;
  __syncthreads();
  if (wave > 0) return;
  s = sums[0][c];
#pragma unroll
  for (int w = 1; w < GRAM_LANES; ++w) s += sums[w][c];
  const int i = u.ci + row, j = u.cj + c;
  const int64_t row_at = (int64_t)i * kp + j, mirror_at = (int64_t)j * kp + i;
  if (on) {
    G[row_at] = s;
    if (G_copy) G_copy[kp <= CR_MAX_KP ? gram_backup_at(i, j, kp) : row_at] = s;
  }
  if (!ns_e2) return;
  const double ev = on && i < k && j < k ? s - (i == j ? 1.0 : 0.0) : 0.0;
  if (on) {
    if (mirror && !diag) G[mirror_at] = s;
    if (ns_T) {
      const bf16_t tv = (bf16_t)(float)(-0.5 * ev);
      ns_T[row_at] = tv;
      if (!diag) ns_T[mirror_at] = tv;
    }
  }
  double share = diag ? ev * ev : 2.0 * ev * ev;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) share += __shfl_xor(share, off);
  if (c == 0) ns_e2[blockIdx.y * 64 + row] = share;
}

// ---------------------------------------------------------------------------------------------
// Gram matrix of up to 64 columns (NB = kp / 16 blocks).  There the product is a few hundred clocks of
// matrix instructions and all the rest is latency and partial tiles, of which 64 x 64 blocks
// write full squares whatever kp is.  Here every wave takes all lower 16 x 16 tiles over rows of its
// own, the four waves of a workgroup add up through LDS, and a chunk leaves only those tiles; in the
// sum (gram_tiles_reduce_kernel) every wave takes some of the chunks.  Product and sum together, 13.2 -> 7.2 us at 12608 x 32 and 16.6 -> 11.2 us at
// 12608 x 64, against blocks of 64 x 64; up to 2048 rows, where those are as short, no difference (one trip per
// wave and a sum spread over the four waves: with two trips and the sum by one wave 64 columns took 3.8 us longer).
// part[(chunk * tiles + tile) * 256 + 16 i + j], tile = I (I + 1) / 2 + J for columns 16 I + i, 16 J + j.

template <int NB>
__global__ __launch_bounds__(256) void gram_narrow_kernel(const float* Y, int64_t m, int rows_per_chunk, double* part) {
  constexpr int KP = 16 * NB, TILES = NB * (NB + 1) / 2;
  __shared__ double red[3 * TILES * 256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lc = lane & 15, lr = lane >> 4;
  const int rows_per_wave = rows_per_chunk >> 2;        // multiple of 16
  const int64_t r_begin = (int64_t)blockIdx.x * rows_per_chunk + wave * rows_per_wave;
  const int64_t r_end = r_begin + rows_per_wave < m ? r_begin + rows_per_wave : m;
  f64x4 acc[TILES];
#pragma unroll
  for (int i = 0; i < TILES; ++i) acc[i] = (f64x4){0.0, 0.0, 0.0, 0.0};
  // 16 rows per trip, one trip ahead; unconditional loads from clamped rows, masked at use
  float f[2][4][NB];
  auto load_trip = [&](int64_t r0, float (*d)[NB]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t row = r0 + 4 * u + lr;
      const float* yr = Y + (row < r_end ? row : m - 1) * KP + lc;
#pragma unroll
      for (int b = 0; b < NB; ++b) d[u][b] = yr[16 * b];
    }
  };
  auto mac_trip = [&](int64_t r0, const float (*d)[NB]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = r0 + 4 * u + lr < r_end;
      double v[NB];
#pragma unroll
      for (int b = 0; b < NB; ++b) v[b] = on ? (double)d[u][b] : 0.0;
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j <= i; ++j) acc[i * (i + 1) / 2 + j] = mfma_f64(v[i], v[j], acc[i * (i + 1) / 2 + j]);
    }
  };
  load_trip(r_begin, f[0]);
  if (rows_per_wave == 16) {                            // one trip (short matrices)
    if (r_begin < r_end) mac_trip(r_begin, f[0]);
  } else {
    for (int64_t r0 = r_begin; r0 < r_end; r0 += 32) {
      load_trip(r0 + 16, f[1]);
      mac_trip(r0, f[0]);
      load_trip(r0 + 32, f[0]);
      mac_trip(r0 + 16, f[1]);
    }
  }
  // (register r of lane l is element 64 r + l of a row-major tile)  Tile i is added up and written by wave i % 4;
  // the others leave theirs in LDS
#pragma unroll
  for (int i = 0; i < TILES; ++i)
    if (wave != (i & 3)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((wave - (wave > (i & 3))) * TILES + i) * 256 + 64 * r + lane] = acc[i][r];
    }
  __syncthreads();
  double* const out = part + (int64_t)blockIdx.x * TILES * 256;
#pragma unroll
  for (int i = 0; i < TILES; ++i)
    if (wave == (i & 3)) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        double v[4];                                    // added in the order of the waves
#pragma unroll
        for (int w = 0; w < 4; ++w)
          v[w] = w == (i & 3) ? acc[i][r] : red[((w - (w > (i & 3))) * TILES + i) * 256 + 64 * r + lane];
        out[i * 256 + 64 * r + lane] = ((v[0] + v[1]) + v[2]) + v[3];
      }
    }
}

__device__ inline void gram_block_of(int b, int* bi, int* bj) {
  int i = 0;
  while ((i + 1) * (i + 2) / 2 <= b) ++i;
  *bi = i;
  *bj = b - i * (i + 1) / 2;
}

// ---------------------------------------------------------------------------------------------
// Gram matrix of more than 64 columns and few rows (gram_is_short, with the times of both kernels): one WAVE per (chunk of rows,
// 32 x 32 block on or below the diagonal), 2 x 2 tiles each, and no sum before the one over the chunks.
// Bound by latency: a wave has two trips of loads and a few dozen matrix instructions.  The kernel for tall matrices pays there for the
// sum of eight waves through LDS and for the epilogue of 4 x 4 tiles, to save partial tiles that are few anyway.
// part as gram_narrow_kernel leaves it.

__global__ __launch_bounds__(256) void gram_short_kernel(const float* Y, int64_t m, int kp, int rows_per_chunk, int chunks, double* part) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nj = kp >> 4, nb32 = (nj + 1) >> 1, nblocks = nb32 * (nb32 + 1) / 2;
  const int unit = blockIdx.x * 4 + wave;
  if (unit >= chunks * nblocks) return;                 // (no barrier below)
  const int chunk = unit / nblocks;
  int bi, bj;
  gram_block_of(unit - chunk * nblocks, &bi, &bj);
  const int64_t r_begin = (int64_t)chunk * rows_per_chunk;
  const int64_t r_end = r_begin + rows_per_chunk < m ? r_begin + rows_per_chunk : m;
  const int lc = lane & 15, lr = lane >> 4;
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};
  // (a last block of one tile takes it twice)
  const int ca[2] = {32 * bi + lc, 16 * (2 * bi + 1 < nj ? 2 * bi + 1 : 2 * bi) + lc};
  const int cb[2] = {32 * bj + lc, 16 * (2 * bj + 1 < nj ? 2 * bj + 1 : 2 * bj) + lc};
  // 16 rows per trip, a ring of 4 trips: the loads run 3 trips ahead.  They are unconditional, from clamped rows, and masked at use.
  float fa[4][4][2], fb[4][4][2];
  auto load_trip = [&](int64_t r0, float (*a)[2], float (*b)[2]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t row = r0 + 4 * u + lr;
      const float* yr = Y + (row < r_end ? row : r_begin) * kp;
#pragma unroll
      for (int i = 0; i < 2; ++i) { a[u][i] = yr[ca[i]]; b[u][i] = yr[cb[i]]; }
    }
  };
  auto mac_trip = [&](int64_t r0, const float (*a)[2], const float (*b)[2]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool on = r0 + 4 * u + lr < r_end;
      double va[2], vb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) { va[i] = on ? (double)a[u][i] : 0.0; vb[i] = on ? (double)b[u][i] : 0.0; }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = mfma_f64(va[i], vb[j], acc[i][j]);
    }
  };
#pragma unroll
  for (int p = 0; p < 3; ++p) load_trip(r_begin + 16 * p, fa[p], fb[p]);
  for (int64_t r0 = r_begin; r0 < r_end; r0 += 64) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      load_trip(r0 + 16 * (q + 3), fa[(q + 3) & 3], fb[(q + 3) & 3]);
      if (r0 + 16 * q < r_end) mac_trip(r0 + 16 * q, fa[q], fb[q]);
    }
  }
  // (register r of lane l is element 64 r + l of a row-major tile)
  double* const out = part + (int64_t)chunk * (nj * (nj + 1) / 2) * 256 + lane;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int I = 2 * bi + i, J = 2 * bj + j;
      if (I >= nj || J > I) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(int64_t)(I * (I + 1) / 2 + J) * 256 + 64 * r] = acc[i][j][r];
    }
}

// What gram_reduce_kernel does, for chunks of lower 16 x 16 tiles (gram_narrow_kernel, solve_body, gram_short_kernel).  Grid
// (4, tiles): a workgroup takes 64 elements of a tile, a lane each; wave w adds the chunks w, w + GT_WAVES, ... in ascending
// order and the waves' sums are added in their order: a fixed order.  One share of ||E||_F^2 per workgroup, four per tile.
template <int GT_WAVES>
__global__ __launch_bounds__(64 * GT_WAVES) void gram_tiles_reduce_kernel(const double* part, int chunks, int tiles, int kp, int k,
                                                                          double* G, double* G_copy, bf16_t* ns_T, double* ns_e2,
                                                                          int32_t* clear_word) {
  __shared__ double sums[GT_WAVES][64];
  if (clear_word && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *clear_word = 0;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int e = blockIdx.x * 64 + lane;
  const double* src = part + (int64_t)blockIdx.y * 256 + e;
  double s = 0.0;
  for (int c0 = wave; c0 < chunks; c0 += 8 * GT_WAVES) {        // eight loads in flight, masked at use
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = src[(int64_t)(c0 + GT_WAVES * u < chunks ? c0 + GT_WAVES * u : c0) * tiles * 256];
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (c0 + GT_WAVES * u < chunks) s += v[u];
  }
  sums[wave][lane] = s;
  __syncthreads();
  if (wave > 0) return;
  s = sums[0][lane];
#pragma unroll
  for (int w = 1; w < GT_WAVES; ++w) s += sums[w][lane];
  int bi, bj;
  gram_block_of(blockIdx.y, &bi, &bj);
  const int i = 16 * bi + (e >> 4), j = 16 * bj + (e & 15);
  G[(int64_t)i * kp + j] = s;
  if (G_copy) G_copy[kp <= CR_MAX_KP ? gram_backup_at(i, j, kp) : (int64_t)i * kp + j] = s;
  if (!ns_e2) return;
  if (bi != bj) G[(int64_t)j * kp + i] = s;              // round 2 leaves the whole symmetric matrix
  const double ev = (i < k && j < k) ? s - (i == j ? 1.0 : 0.0) : 0.0;
  if (ns_T) {
    const bf16_t tv = (bf16_t)(float)(-0.5 * ev);
    ns_T[(int64_t)i * kp + j] = tv;
    if (bi != bj) ns_T[(int64_t)j * kp + i] = tv;
  }
  double share = (bi == bj) ? ev * ev : 2.0 * ev * ev;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) share += __shfl_xor(share, off);
  if (lane == 0) ns_e2[blockIdx.y * 4 + blockIdx.x] = share;
}

// ---------------------------------------------------------------------------------------------
// Blocked Cholesky factorisation G (+ shift) = L L^T of the kp x kp Gram matrix by one workgroup.
// Two kernels: chol_reg_kernel (further down: kp <= CR_MAX_KP, matrix in registers, what the benchmark
// shapes use) and chol_blocked_kernel (any kp, matrix updated in place in global memory).
//
// chol_blocked_kernel, per 16-column panel: every wave holds the 16 diagonal-block rows
// redundantly in lanes 0..15 and up to 48 rows below in lanes 16..63, one row per lane with its 16
// panel entries in registers; the 16 pivot steps then need no workgroup barrier, only wave-wide
// lane reads.  The trailing lower triangle is updated per 16 x 16 block on the matrix cores.
//
// Outputs: L in the strict lower triangle of G (global), and Dinv[b] = inverse of the b-th
// 16 x 16 diagonal block of L (row-major, lower triangular), which is what the triangular solve
// in trsm_apply_kernel consumes.
//
// Pivot rule: see chol.h.  Columns k..kp-1 are padding: their reciprocal pivot is whatever the
// rule gives (zero without a shift) and they never raise the status flag.

__device__ inline double readlane_f64(double v, int src_lane) {
  union { double d; int i[2]; } u;
  u.d = v;
  u.i[0] = __builtin_amdgcn_readlane(u.i[0], src_lane);
  u.i[1] = __builtin_amdgcn_readlane(u.i[1], src_lane);
  return u.d;
}

// 1 / sqrt(x) to float64 accuracy: the hardware estimate (relative error below ~2^-22) refined by
// third-order steps y <- y (1 + e/2 + 3 e^2/8), e = 1 - x y^2, each of which cubes the error.
template <int STEPS>
__device__ inline double rsqrt_f64(double x) {
  double y = __builtin_amdgcn_rsq(x);
#pragma unroll
  for (int it = 0; it < STEPS; ++it) {
    const double e = fma(-x * y, y, 1.0);
    y = fma(y * fma(0.375, e, 0.5), e, y);
  }
  return y;
}


// chol_blocked_kernel runs 8 waves to overlap the memory latency of the trailing-block updates.
//
// round == 1 (Gram matrix of the sketch): the factorisation is first attempted WITHOUT a shift;
//   a pivot that is not above unshifted_thresh * G[j][j] (a small multiple of the rounding level
//   k u) abandons the attempt and the matrix is factored again as G + s I, s = shift_rel * trace
//   (the matrix is restored from G_backup).  Unshifted factors leave
//   Q1 = Y R^{-1} orthonormal to ~u cond(G); shifted ones only well conditioned (see chol.h).
// round == 2 (Gram matrix of Q1): if ns_flag is given, E = G - I is measured first.  When
//   ||E||_F <= ns_tol the factorisation is skipped (T = -E/2 was already written by
//   gram_reduce_kernel) and *ns_flag = 1, so that the caller finishes with the first-order Newton-Schulz correction
//   Q = Q1 (I - E/2), whose defect is ~ (3/4) ||E||^2.  When ||E||_F <= ns_exact_tol, Q1 is taken as
//   it is (*ns_flag = 2: no second round at all).  Otherwise *ns_flag = 0 and the matrix is
//   factored unshifted with the clamping rule of chol.h.
struct CholArgs {
  double* G;
  const double* G_backup;
  double* Dinv;
  int k, kp;
  int round;
  double tol;               // round 2 clamping level
  double shift_rel;         // round 1 shift (second attempt)
  double unshifted_thresh;  // round 1 breakdown level of the unshifted attempt (0 = always shift)
  int32_t* status;
  const double* ns_e2;      // round 2: shares of ||E||_F^2 from gram_reduce_kernel
  int ns_e2_count;
  int32_t* ns_flag;
  double ns_tol;            // Newton-Schulz finish up to this ||E||_F (0 = not available)
  double ns_exact_tol;      // Q1 accepted unchanged up to this ||E||_F
  const double* poly_p4;    // optional: shares of ||E^4||_F^2 from ns_poly_finish_kernel
  int poly_count;
  double poly_hi_tol;       // the polynomial finish was attempted for ||E||_F in (ns_tol, poly_hi_tol]
  double poly_b4_tol;       // ... and is accepted when ||E^4||_F^(1/4) (>= ||E||_2) is at most this
  int32_t* ready;           // fused factor-and-solve launch only: progress word read by the solving workgroups
};

// Progress word of the fused factor-and-solve launch (progress.h).  The producer writes L, Dinv and the word with
// device-scope write-through stores and waits for their completion before it advances the word; consumers read with
// device-scope loads.  No read-modify-write and no cache write-back is involved.
__device__ inline void cf_store(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// (two doubles that lie together; whoever reads them waits for the progress word, so that they need not arrive as one)
typedef double f64x2 __attribute__((ext_vector_type(2)));
__device__ inline void cf_store2(double* p, f64x2 v) {
  // (the wait: data of a store this wide may be overwritten one state later at the earliest)
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" : : "v"(p), "v"(v) : "memory");
}
__device__ inline void cf_publish(int32_t* ready, int attempt, int panels) {
  __hip_atomic_store(ready, cf_word(attempt, panels), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int cf_poll(const int32_t* ready) {
  return __hip_atomic_load(ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Round 2 decision, taken by the whole workgroup before any factorisation work: E = G - I has been
// measured by gram_reduce_kernel (||E||_F^2 in pieces, T = -E/2 already written).  Returns true,
// with *ns_flag set, when no second factorisation is needed; misc is an LDS scratch of 4 doubles.
__device__ inline bool chol_round2_exit(const CholArgs& g, double* misc, const bool write_flag = true) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  // wave 0 adds the shares (lane i takes shares i, i + 64, ...; butterfly sum, so every lane
  // ends with the same value) and hands the total to the other waves through LDS
  if (wave == 0) {
    double part_sum = 0.0;
    for (int w0 = lane; w0 < g.ns_e2_count; w0 += 256) {      // four loads in flight, no branch around them
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int w = w0 + 64 * u;
        v[u] = g.ns_e2[w < g.ns_e2_count ? w : g.ns_e2_count - 1] * (w < g.ns_e2_count ? 1.0 : 0.0);
      }
      part_sum += (v[0] + v[1]) + (v[2] + v[3]);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part_sum += __shfl_xor(part_sum, off);
    if (lane == 0) misc[1] = part_sum;
  }
  __syncthreads();
  const double tot = misc[1];
  if (tot <= g.ns_exact_tol * g.ns_exact_tol) {     // Q1 is orthonormal as it stands
    if (t == 0 && write_flag) *g.ns_flag = 2;
    return true;
  }
  if (g.ns_tol > 0.0 && tot <= g.ns_tol * g.ns_tol) {       // comparisons are false for NaN
    if (t == 0 && write_flag) *g.ns_flag = 1;
    return true;
  }
  if (g.ns_tol > 0.0 && g.poly_count > 0 && tot <= g.poly_hi_tol * g.poly_hi_tol) {
    // the degree-4 correction was prepared (T holds it): accept it if the spectral norm of E,
    // bounded by ||E^4||_F^(1/4), keeps the truncated series accurate
    if (wave == 0) {
      double part_sum = 0.0;
      for (int w = lane; w < g.poly_count; w += 64) part_sum += g.poly_p4[w];
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) part_sum += __shfl_xor(part_sum, off);
      if (lane == 0) misc[2] = part_sum;
    }
    __syncthreads();
    const double b4 = sqrt(sqrt(sqrt(misc[2])));
    if (b4 <= g.poly_b4_tol) {
      if (t == 0 && write_flag) *g.ns_flag = 1;
      return true;
    }
  }
  if (t == 0 && write_flag) *g.ns_flag = 0;
  return false;
}

__global__ __launch_bounds__(512) void chol_blocked_kernel(CholArgs g) {
  constexpr int CHOL_THREADS = 512;
  double* const G = g.G;
  double* const Dinv = g.Dinv;
  const int k = g.k, kp = g.kp;
  const double tol = g.tol;
  int32_t* const status = g.status;
  extern __shared__ double smem[];
  // layout: gdiag[kp] | dinv[kp] | misc[8] | Pt[16][kp - 16]
  double* gdiag = smem;            // original diagonal
  double* dinv = smem + kp;        // reciprocal pivots
  double* misc = smem + 2 * kp;    // [0] = shift
  const int ptld = kp > OF_NB ? kp - OF_NB : 2;
  double* Pt = smem + 2 * kp + 8;  // panel below the diagonal block, transposed: Pt[p][row - below]
  double* Am = G;
  const int lda = kp;
  __shared__ int deficient, restart;

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  if (t == 0) { deficient = 0; restart = 0; }
  __syncthreads();

  // ---- round 2: is Q1 already orthonormal enough for a Newton-Schulz finish?  On that branch
  // the kernel ends here.
  if (g.round == 2 && g.ns_flag && chol_round2_exit(g, misc)) return;

  for (int i = t; i < kp; i += CHOL_THREADS) gdiag[i] = G[(int64_t)i * kp + i];
  __syncthreads();

  double trace_sum = 0.0;
  if (wave == 0) {
    double tr = 0.0;
    for (int i = lane; i < kp; i += 64) tr += gdiag[i];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
    if (lane == 0) misc[0] = tr;
  }
  __syncthreads();
  trace_sum = misc[0];

  const bool try_unshifted = g.round == 1 && g.unshifted_thresh > 0.0;
  for (int attempt = try_unshifted ? 0 : 1; attempt < 2; ++attempt) {
  const bool unshifted_attempt = g.round == 1 && attempt == 0;
  const double shift = (g.round == 1 && attempt == 1) ? g.shift_rel * trace_sum : 0.0;
  if (attempt == 1 && try_unshifted) {
    // the unshifted attempt broke down: restore the matrix and start over with the shift
      for (int e = t; e < kp * kp; e += CHOL_THREADS) G[e] = g.G_backup[e];
    
    if (t == 0) restart = 0;
    __syncthreads();
  }

  for (int jb = 0; jb < kp; jb += OF_NB) {
    const int below = jb + OF_NB;
    const int nrows_below = kp - below;

    // ---- panel: one row per lane, its 16 panel entries in registers.  Lanes 0..15 of every
    // wave hold the diagonal block (redundantly), lanes 16..63 hold 48 of the rows below.
    // 4 waves x 48 rows per pass; a second pass (kp > 208) reuses the saved diagonal block
    constexpr int NWAVES = CHOL_THREADS / 64;
    const int npass = nrows_below > 0 ? (nrows_below + 48 * NWAVES - 1) / (48 * NWAVES) : 1;
    double dsave[OF_NB];
    double thr[OF_NB], gdiag_reg[OF_NB];
#pragma unroll
    for (int c = 0; c < OF_NB; ++c) {
      double v = 0.0;
      if (lane < 16 && c <= lane) v = Am[(jb + lane) * lda + jb + c];
      if (lane < 16 && c == lane) v += shift;
      dsave[c] = v;
      gdiag_reg[c] = gdiag[jb + c];
      thr[c] = tol * gdiag_reg[c];
    }
    // the first pass's rows below are fetched together with the diagonal block, before the barrier:
    // one memory round trip per panel instead of two (they are written only after it)
    double afirst[OF_NB];
    {
      const int row = below + wave * 48 + lane - 16;
      const bool on = lane >= 16 && row < kp;
#pragma unroll
      for (int c = 0; c < OF_NB; ++c) afirst[c] = on ? Am[row * lda + jb + c] : 0.0;
    }
    __syncthreads();   // every wave has read the unfactored diagonal block
    for (int pass = 0; pass < npass; ++pass) {
    const int row = (lane < 16) ? (jb + lane) : (below + (pass * NWAVES + wave) * 48 + lane - 16);
    const bool row_ok = row < kp;
    double a[OF_NB];
    if (pass == 0) {
#pragma unroll
      for (int c = 0; c < OF_NB; ++c) a[c] = (lane < 16) ? dsave[c] : afirst[c];
    } else {
#pragma unroll
      for (int c = 0; c < OF_NB; ++c)
        a[c] = (lane < 16) ? dsave[c] : (row_ok ? Am[row * lda + jb + c] : 0.0);
    }
    double dval[OF_NB];
    bool any_bad = false;
#pragma unroll
    for (int j = 0; j < OF_NB; ++j) {
      const double piv = readlane_f64(a[j], j);
      const bool live = jb + j < k;                      // padding columns never count
      bool usable;
      if (unshifted_attempt) usable = piv > g.unshifted_thresh * gdiag_reg[j];
      else if (g.round == 1) usable = piv > 0.0;
      else usable = piv > thr[j];
      const double d = (usable && live) ? rsqrt_f64<OF_RSQ_STEPS>(piv) : 0.0;
      dval[j] = d;
      any_bad = any_bad || (!usable && live);
      a[j] *= d;
#pragma unroll
      for (int c = j + 1; c < OF_NB; ++c) {
        const double lcj = readlane_f64(a[j], c);
        a[c] = fma(-a[j], lcj, a[c]);
      }
    }
    if (lane >= 16) {
      if (row_ok) {
#pragma unroll
        for (int c = 0; c < OF_NB; ++c) {
          Am[row * lda + jb + c] = a[c];
          Pt[c * ptld + row - below] = a[c];
        }
      }
    } else if (wave == 0 && pass == 0) {   // wave 0 owns the diagonal block
#pragma unroll
      for (int c = 0; c < OF_NB; ++c)
        if (c < lane) Am[row * lda + jb + c] = a[c];
      if (lane == 0) {
#pragma unroll
        for (int j = 0; j < OF_NB; ++j) dinv[jb + j] = dval[j];
        if (any_bad) {
          if (unshifted_attempt) restart = 1; else deficient = 1;
        }
      }
    }
    }
    __syncthreads();
    if (restart) break;          // uniform: written before the barrier

    // ---- trailing update of the lower triangle: A[I][C] -= P_I P_C^T per 16 x 16 block (C <= I),
    // on the float64 matrix cores, the panel read from Pt.
    {
      const int nb16 = nrows_below / OF_NB;
      const int nblocks = nb16 * (nb16 + 1) / 2;
      const int lc = lane & 15, lr = lane >> 4;
      // Several blocks per wave and trip: the loads of all their accumulators are issued before
      // the first matrix instruction, so that their latency (LDS, or L2 when the matrix lives in
      // global memory) is paid once per trip.  The panel operands come from LDS at the point of use.
      constexpr int NWV = CHOL_THREADS / 64, TB = 4;
      for (int e0 = wave; e0 < nblocks; e0 += NWV * TB) {
        double* ablk[TB];
        int ta[TB], tb[TB];
        f64x4 acc[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b) {
          const int e = e0 + b * NWV;
          const int ee = e < nblocks ? e : e0;            // idle slots redo the first block's loads
          int ti = (int)((sqrtf(8.0f * (float)ee + 1.0f) - 1.0f) * 0.5f);
          while (ti * (ti + 1) / 2 > ee) --ti;
          while ((ti + 1) * (ti + 2) / 2 <= ee) ++ti;
          const int tc = ee - ti * (ti + 1) / 2;
          ta[b] = OF_NB * ti + lc;
          tb[b] = OF_NB * tc + lc;
          ablk[b] = Am + (below + OF_NB * ti + lr) * lda + below + OF_NB * tc + lc;
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[b][r] = ablk[b][4 * r * lda];
        }
#pragma unroll
        for (int b = 0; b < TB; ++b) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[b] = mfma_f64(-Pt[(4 * r + lr) * ptld + ta[b]], Pt[(4 * r + lr) * ptld + tb[b]], acc[b]);
        }
#pragma unroll
        for (int b = 0; b < TB; ++b) {
          if (e0 + b * NWV < nblocks) {
#pragma unroll
            for (int r = 0; r < 4; ++r) ablk[b][4 * r * lda] = acc[b][r];
          }
        }
      }
    }
    __syncthreads();
  }
  if (!restart) break;
  __syncthreads();
  }

  // ---- inverses of the 16 x 16 diagonal blocks, one thread per (block, column c):
  // column c of L_bb^{-1} by forward substitution in update form (x_j is final after step j and
  // is then subtracted from all later rows at once, so the 15 steps carry a two-operation chain).
  const int nblk = kp / OF_NB;
  for (int e = t; e < nblk * OF_NB; e += CHOL_THREADS) {
    const int b = e >> 4, c = e & 15;
    const int base = b * OF_NB;
    double acc[OF_NB], x[OF_NB];
#pragma unroll
    for (int r = 0; r < OF_NB; ++r) acc[r] = (r == c) ? 1.0 : 0.0;
#pragma unroll
    for (int j = 0; j < OF_NB; ++j) {
      const double xj = (j >= c) ? acc[j] * dinv[base + j] : 0.0;
      x[j] = xj;
#pragma unroll
      for (int r = j + 1; r < OF_NB; ++r) acc[r] = fma(-Am[(base + r) * lda + base + j], xj, acc[r]);
    }
#pragma unroll
    for (int r = 0; r < OF_NB; ++r) Dinv[((int64_t)b * OF_NB + r) * OF_NB + c] = x[r];
  }
  if (t == 0 && deficient && status) atomicOr(status, LORACT_STATUS_RANK_DEFICIENT);
}

// ---------------------------------------------------------------------------------------------
// Register-resident blocked Cholesky for kp <= CR_MAX_KP: one workgroup of 8 waves, the matrix never
// touches LDS or global memory between panels.
//
// Storage.  The symmetric matrix is kept as its UPPER 16 x 16 blocks U(C, I) = G[C rows][I cols],
// C <= I, each in the accumulator layout of the float64 matrix instruction, dealt round-robin in
// row-major order to the worker waves (so every suffix C > j, the trailing matrix of panel j, and
// every block row C == j, the panel itself, are spread evenly).  In that layout register r of a
// block is at once slice r of the B operand of a product contracting over the block's rows, so
//   panel j:     P_I^T = Linv_j U(j, I)            (P_I = L[I rows][j cols], 4 matrix instructions)
//   trailing:    U(C, I) -= P_C P_I^T              (operands from LDS, accumulated in place)
// need no layout change at all.  P^T goes to LDS (Pt) for the trailing update, and from there to global
// memory as rows of L.  Within a block the rows are permuted: register r of lane group q holds row 4 q + r
// (the hardware's natural order would be q + 4 r), so that a lane's four registers are 32
// contiguous bytes of a row of G; the permutation
// is undone where it matters, in the row index of the A operand of the trailing update.
//
// Look-ahead.  Wave 0 owns the serial part.  While the workers form panel j and apply it to the trailing
// matrix, wave 0 takes the next diagonal block and the block above it (staged in LDS by their owners one
// iteration earlier), applies panel j to it, factors it one row per lane (cr_pivots), and leaves L_bb and Linv_bb in
// LDS, from where the helper copies them out.  The rows of the identity go through the same 16 pivot steps, which
// turns them into the rows of L^{-T}.
// Two workgroup barriers per panel, which order LDS only; wave 0's pivot steps (2600 of some 4700 clocks per panel once
// the trailing matrix is small) are the critical path, and what bounds the first panels of a wide matrix is the trailing
// update: its matrix instructions at 64 clocks each on three SIMDs, and the LDS reads before them.
// While a float64 matrix instruction runs no vector instruction of any wave of its SIMD does (measured: 8 vector instructions per
// matrix instruction, in the same wave or in another one, take their own time in full), so wave 0's SIMD is kept free of them: its
// other wave, the helper, has trailing blocks only as long as the trailing update is the longer part.
// Factor and solve in one launch at 8192 rows, us, with seven workers of which one ran beside wave 0, scattered stores of the panel in
// phase A and G read row by row: 64 columns 24.8 -> 23.7, 128 36.5 -> 34.0, 160 51.9 -> 43.0,
// 192 62.5 -> 52.0, 256 89.7 -> 82.4 (event to event, with the second round's launch, which returns at once).
//
// In round 1 the original matrix is read from G_backup (required: the unshifted attempt may have
// to start over with the shift after L has begun to overwrite G), in round 2 from G.
// Pivot rules, outputs (L in the strict lower triangle of G, Dinv) and the round-2 early exits are
// those of chol_blocked_kernel, except that padding columns get a unit diagonal (their rows and
// columns of L are zero either way).
#define CR_THREADS 512
#define CR_WORKERS 6
#define CR_HELPER 4              // wave beside wave 0 on its SIMD

// Doubles per row of the panel in LDS, a constant of the instantiation (kpm: the largest kp it is used for), so that the rows
// of an operand are immediate offsets.  (Consecutive rows start 128 bytes apart, mod 256.)
static constexpr int chol_reg_ptld(int kpm) {
  const int w = kpm > OF_NB ? kpm - OF_NB : OF_NB;
  return (w % 32 == 16) ? w : w + 16;
}
static constexpr int chol_reg_slots(int nbm) {           // blocks a worker has registers for
  const int s = (nbm * (nbm + 1) / 2 - 1 + CR_WORKERS - 1) / CR_WORKERS;
  return s > 20 ? 20 : (s > 0 ? s : 1);
}
// Whether the blocks of block row 0 wait in LDS for the first panel, the only one that they are needed for, instead of in registers: 17 block
// rows have as many other blocks as 16 have in all (264 columns: 79 us, as chol_blocked_kernel 183).  "In registers" but for 56 values that the compiler
// spills at 17 block rows, 29 to 31 at 13 to 16.
static constexpr bool chol_reg_parks(int nbm) { return nbm > 16; }
// LDS doubles: misc[8] | LinvT[2][16][CR_TP] | Ltile[2][16][CR_TP] | Dstage[2][256] | Ustage[2][256] |
//              Dtile[16][17] | gdiag[kpm] | Pt[16][chol_reg_ptld(kpm)] | (chol_reg_parks) Park[nbm - 1][256]
#define CR_TP 18              // (even: rows are written in 16-byte pieces)
static constexpr size_t chol_reg_lds_bytes(int kpm) {
  return sizeof(double) * (size_t)(8 + 64 * CR_TP + 1024 + 272 + kpm + OF_NB * chol_reg_ptld(kpm) +
                                   (chol_reg_parks(kpm / OF_NB) ? (kpm / OF_NB - 1) * 256 : 0));
}

// Value of src in lane C of each row of 16 lanes.
template <int C>
__device__ __forceinline__ double cr_bcast(double src) {
  const long long v = __builtin_bit_cast(long long, src);
  const long long r = __builtin_amdgcn_update_dpp(v, v, 0x150 + C, 0xf, 0xf, false);       // row_newbcast:C
  return __builtin_bit_cast(double, r);
}
// a[c] -= (a[J] in lane c of each row of 16 lanes) a[J] and the same for b with b[J], columns c = C .. C + N - 1: one
// instruction per column and array, because the double precision FMA takes its first operand through a row
// broadcast.  A vector instruction's result may be read that way two wait states later at the earliest, which assembly has
// to see to itself; the wait is part of the statement, so that no copy of a[J] can come between.  Statements of several
// columns, because each pays the wait, and not one for all, so that the chain of the next pivot is scheduled between
// them (kernel alone at 128 columns: two columns each 21.5 us, four 21.1, half the columns 20.8; the compiler's own
// broadcasts, which it does not fold into the FMA, 23.7).
#define CR_SUB(I)                                                                                              \
  "\n\tv_fmac_f64_dpp %[a" #I "], -%[s], %[s] row_newbcast:%c[c" #I "] row_mask:0xf bank_mask:0xf"             \
  "\n\tv_fmac_f64_dpp %[b" #I "], -%[s], %[m] row_newbcast:%c[c" #I "] row_mask:0xf bank_mask:0xf"
#define CR_OUT(I) [a##I] "+&v"(a[C + I]), [b##I] "+&v"(b[C + I])
#define CR_IN [s] "v"(a[J]), [m] "v"(b[J])
#define CR_NUM(I) [c##I] "n"(C + I)
template <int J, int C, int N>
__device__ __forceinline__ void cr_columns(double* a, double* b) {
  if constexpr (N == 1)
    asm("s_nop 1" CR_SUB(0) : CR_OUT(0) : CR_IN, CR_NUM(0));
  else if constexpr (N == 2)
    asm("s_nop 1" CR_SUB(0) CR_SUB(1) : CR_OUT(0), CR_OUT(1) : CR_IN, CR_NUM(0), CR_NUM(1));
  else if constexpr (N == 3)
    asm("s_nop 1" CR_SUB(0) CR_SUB(1) CR_SUB(2)
        : CR_OUT(0), CR_OUT(1), CR_OUT(2) : CR_IN, CR_NUM(0), CR_NUM(1), CR_NUM(2));
  else if constexpr (N == 4)
    asm("s_nop 1" CR_SUB(0) CR_SUB(1) CR_SUB(2) CR_SUB(3)
        : CR_OUT(0), CR_OUT(1), CR_OUT(2), CR_OUT(3) : CR_IN, CR_NUM(0), CR_NUM(1), CR_NUM(2), CR_NUM(3));
  else if constexpr (N == 5)
    asm("s_nop 1" CR_SUB(0) CR_SUB(1) CR_SUB(2) CR_SUB(3) CR_SUB(4)
        : CR_OUT(0), CR_OUT(1), CR_OUT(2), CR_OUT(3), CR_OUT(4)
        : CR_IN, CR_NUM(0), CR_NUM(1), CR_NUM(2), CR_NUM(3), CR_NUM(4));
  else if constexpr (N == 6)
    asm("s_nop 1" CR_SUB(0) CR_SUB(1) CR_SUB(2) CR_SUB(3) CR_SUB(4) CR_SUB(5)
        : CR_OUT(0), CR_OUT(1), CR_OUT(2), CR_OUT(3), CR_OUT(4), CR_OUT(5)
        : CR_IN, CR_NUM(0), CR_NUM(1), CR_NUM(2), CR_NUM(3), CR_NUM(4), CR_NUM(5));
  else
    asm("s_nop 1" CR_SUB(0) CR_SUB(1) CR_SUB(2) CR_SUB(3) CR_SUB(4) CR_SUB(5) CR_SUB(6)
        : CR_OUT(0), CR_OUT(1), CR_OUT(2), CR_OUT(3), CR_OUT(4), CR_OUT(5), CR_OUT(6)
        : CR_IN, CR_NUM(0), CR_NUM(1), CR_NUM(2), CR_NUM(3), CR_NUM(4), CR_NUM(5), CR_NUM(6));
}
#undef CR_SUB
#undef CR_OUT
#undef CR_IN
#undef CR_NUM

// The 16 pivot steps on a 16 x 16 block, lane i of every row of 16 lanes holding row i: a becomes the rows of the factor
// L, b (the identity before) those of L^{-T}.  pivs: lane j gets pivot j.
//
// One wave issues in order, so what counts is the number of instructions and the chain from one pivot to the next.
// The chain is seven operations long and runs on values that every lane holds:
//   y = rsq(piv);  e = 1 - piv y^2;  q = e (1/2 + 3e/8)     (1/sqrt(piv) = y (1 + q))
//   l = l0 y (1 + q)        l0 = entry (j+1, j), broadcast BEFORE the step
//   piv' = p0 - l^2         p0 = entry (j+1, j+1), likewise
// The lanes scale their own row entry the same way (bitwise the same arithmetic as l); the rank-1 update takes one
// instruction per column, whose multiplier is the broadcast operand (read back from LDS one step late, as it was
// before, a panel took 4000 to 5400 clocks).  No operation on the chain tests the pivot.
template <int J>
__device__ __forceinline__ void cr_pivots(double* a, double* b, double& piv, double& y, double& pivs, int lc) {
  pivs = lc == J ? piv : pivs;
  double l0 = 0.0, p0 = 0.0;
  if constexpr (J + 1 < OF_NB) {
    l0 = cr_bcast<J + 1>(a[J]);
    p0 = cr_bcast<J + 1>(a[J + 1]);
  }
  const double s0 = a[J] * y, b0 = b[J] * y, ls0 = l0 * y;
  const double tq = piv * y;
  const double eq = fma(-tq, y, 1.0);
  const double q = eq * fma(0.375, eq, 0.5);
  if constexpr (J + 1 < OF_NB) {
    const double l = fma(ls0, q, ls0);
    piv = fma(-l, l, p0);
    y = __builtin_amdgcn_rsq(piv);
    a[J] = fma(s0, q, s0);
    b[J] = fma(b0, q, b0);
    a[J + 1] = fma(-a[J], l, a[J + 1]);
    b[J + 1] = fma(-b[J], l, b[J + 1]);
    if constexpr (J + 2 < OF_NB) {
      constexpr int N = OF_NB - (J + 2), N0 = N <= 7 ? N : (N + 1) / 2;
      cr_columns<J, J + 2, N0>(a, b);
      if constexpr (N0 < N) cr_columns<J, J + 2 + N0, N - N0>(a, b);
    }
    cr_pivots<J + 1>(a, b, piv, y, pivs, lc);
  } else {
    a[J] = fma(s0, q, s0);
    b[J] = fma(b0, q, b0);
  }
}

typedef __attribute__((address_space(3))) const double* LdsDouble;
// NBM: most 16-column blocks there can be.  PUB: the factor is published panel by panel for the solving workgroups of the same launch
// (chol_trsm_fused_kernel): write-through stores and the progress word g.ready.
template <int NBM, bool PUB>
__device__ inline void chol_reg_body(const CholArgs& g, double* smem) {
  constexpr int SLOTS = chol_reg_slots(NBM), ptld = chol_reg_ptld(OF_NB * NBM);
  double* const G = g.G;
  // (round 2 never starts over, and its caller's backup, if any, is round 1's matrix)
  const bool backup = g.round == 1 && g.G_backup;
  const double* const src = backup ? g.G_backup : g.G;
  const int k = g.k, kp = g.kp, nb = kp / OF_NB;
  // (the fixed-size pieces come first, so that their addresses are compile-time constants)
  double* misc = smem;                 // [0] trace, [1], [2] round-2 decision
  double* LinvT = smem + 8;            // [b & 1][c * CR_TP + i] = Linv_bb[i][c]
  double* Ltile = LinvT + 32 * CR_TP;  // [b & 1][r * CR_TP + c] = L_bb[r][c]
  double* Dstage = Ltile + 32 * CR_TP; // next diagonal blocks, accumulator layout, two buffers
  double* Ustage = Dstage + 512;       // the blocks left of them (above them in U), likewise
  double* Dtile = Ustage + 512;        // wave 0: blocks turned from one lane to another
  double* gdiag = Dtile + 272;         // original diagonal (read by wave 0 only)
  double* Pt = gdiag + OF_NB * NBM;    // Pt[p * ptld + x] = L[below + x][16 j + p]
  constexpr bool PARKS = chol_reg_parks(NBM);
  double* Park = Pt + OF_NB * ptld;    // block (0, I) at 256 (I - 1), accumulator layout
  __shared__ int deficient, restart;

  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lc = lane & 15, lr = lane >> 4;
  const int pm = 4 * (lc & 3) + (lc >> 2);   // accumulator row of logical row lc, and back
  if (t == 0) { deficient = 0; restart = 0; }
  __syncthreads();
  // (in the fused launch every workgroup has taken the round-2 decision before it got here)
  if (!PUB && g.round == 2 && g.ns_flag && chol_round2_exit(g, misc)) return;

  // ---- block ownership: the row-major upper triangle without block (0, 0), which wave 0 reads itself, is dealt to workers 0 .. 5
  // (waves 1 to 3 and 5 to 7) and, `both` rounds long, to the helper (wave 4) as well.  The helper runs beside wave 0, whose
  // vector instructions stand still while one of its matrix instructions runs (factoring a block 4400 to 4800 clocks
  // against 3500), so it only takes blocks of the first block rows: they are done with after a few panels, in which the trailing
  // update takes longer than the pivots anyway, and what remains of nine block rows does not.
  // (packed as C | I << 8, in order of C; the unused ones at the end name block (0, 0), which no condition below selects)
  const int worker = wave == CR_HELPER ? CR_WORKERS : wave - 1 - (wave > CR_HELPER);
  int ci[SLOTS];
  {
    const int first = PARKS ? nb : 1;      // (row-major number of the first block to deal)
    const int total = nb * (nb + 1) / 2 - first;
    const int early = nb > 9 ? total - 45 : 0;
    const int most = total - CR_WORKERS * SLOTS;       // (what the six have no room for)
    const int both = most > early / (CR_WORKERS + 1) ? most : early / (CR_WORKERS + 1);
    int c = 0, rem = worker + first;       // block e + first = rem-th of block row c, carried from slot to slot
#pragma unroll
    for (int s = 0; s < SLOTS; ++s) {
      const int e = s < both ? s * (CR_WORKERS + 1) + worker : both + s * CR_WORKERS + worker;
      while (c < nb && rem >= nb - c) { rem -= nb - c; ++c; }
      ci[s] = (wave > 0 && e < total && (s < both || worker < CR_WORKERS)) ? (c | ((c + rem) << 8)) : 0;
      rem += s < both ? CR_WORKERS + 1 : CR_WORKERS;
    }
  }
  // Unpacking goes through an empty volatile asm so that nothing derived from a slot's block
  // coordinates is hoisted out of the panel loop (20 slots' worth of addresses would spill).
#define CR_SLOT(s, C, I)                       \
  int ci_ = ci[s];                             \
  asm volatile("" : "+s"(ci_));                \
  const int C = ci_ & 255, I = ci_ >> 8
  // block row of slot s (or of the last one)
#define CR_ROW(s) (ci[(s) < SLOTS ? (s) : SLOTS - 1] & 255)
  // Row p of the panel has its two halves of every 16 entries exchanged where bit 1 of p is set: the rows that a store reads
  // side by side, p = 0, 2, 4, .., lie a multiple of 256 bytes apart.
#define CR_SWZ(p) (((p) & 2) << 2)
  // Block (C, I): lane (q, n) takes G[16 I + n][16 C + 4 q .. + 3], from rows of G or from the backup's blocks
  const int step_c = backup ? 256 : OF_NB;
  const unsigned lane_at = 8u * (backup ? 2 * lane : lc * kp + 4 * lr), lane_at2 = lane_at + 8u * (backup ? 128 : 2);
#define CR_LOAD_BLOCK(dst, C, I)                                                              \
  {                                                                                           \
    const char* p_ = (const char*)(src + OF_NB * kp * (I) + step_c * (C));                      \
    const double2 v0_ = *(const double2*)(p_ + lane_at), v1_ = *(const double2*)(p_ + lane_at2); \
    dst[0] = v0_.x; dst[1] = v0_.y; dst[2] = v1_.x; dst[3] = v1_.y;                            \
  }
  // Diagonal entries of a diagonal block: the shift, and 1 on the padding columns
#define CR_FIX_DIAG(dst, C)                                                                   \
  _Pragma("unroll") for (int r_ = 0; r_ < 4; ++r_)                                            \
    if (4 * lr + r_ == lc) dst[r_] = (OF_NB * (C) + lc < k) ? dst[r_] + shift : 1.0;

  // Round 1 starts with the unshifted attempt (the launcher sends anything else to
  // chol_blocked_kernel), so the shift is needed on a second attempt only, long after the helper has
  // left the trace in LDS.
  const bool try_unshifted = g.round == 1;
  int attempt_pub = 0;                 // attempt number as the solving workgroups count it
  for (int attempt = try_unshifted ? 0 : 1; attempt < 2; ++attempt) {
    attempt_pub = (try_unshifted && attempt == 1) ? 1 : 0;
    const bool unshifted_attempt = g.round == 1 && attempt == 0;
    const double shift = (g.round == 1 && attempt == 1) ? g.shift_rel * misc[0] : 0.0;
    if (PUB && attempt_pub == 1 && t == 64 * CR_HELPER) cf_publish(g.ready, 1, 0);   // the solvers start over

    // The two roles run separate loops with the same sequence of barriers, so that the workers'
    // blocks and wave 0's pivot rows never compete for registers.
    if (wave == 0) {
      // ---- wave 0: factor diagonal block b, given in the accumulator layout
      auto factor_diag = [&](const int b, const f64x4 dacc) {
#pragma unroll
        for (int r = 0; r < 4; ++r) Dtile[(4 * lr + r) * 17 + lc] = dacc[r];
        __builtin_amdgcn_wave_barrier();      // LDS operations of one wave complete in order
        double a[OF_NB], binv[OF_NB];
#define CR_LOAD_ROWS()                                                           \
  _Pragma("unroll") for (int c = 0; c < OF_NB; ++c) {                            \
    a[c] = Dtile[lc * 17 + c];                                                   \
    binv[c] = lc == c ? 1.0 : 0.0;                                               \
  }
        CR_LOAD_ROWS();
        // lane c: the level pivot c has to exceed (one rule for the three cases)
        const double level = unshifted_attempt ? g.unshifted_thresh : (g.round == 1 ? 0.0 : g.tol);
        const double thl = level * gdiag[OF_NB * b + lc];
        double pivs = 0.0;
        {
          double piv = readlane_f64(a[0], 0);
          double y = __builtin_amdgcn_rsq(piv);
          cr_pivots<0>(a, binv, piv, y, pivs, lc);
        }
        // (padding columns carry a unit diagonal and never fail; false for NaN)
        const bool any_bad = __any(OF_NB * b + lc < k && !(pivs > thl));
        // ---- guarded form, only after a pivot failed its test (and the factorisation goes on:
        // an unshifted attempt is abandoned anyway): unusable and padding columns get a zero
        // reciprocal, so that they drop out of L and of Linv instead of spreading NaN.
        if (any_bad && !unshifted_attempt) {
          CR_LOAD_ROWS();
#pragma unroll
          for (int jj = 0; jj < OF_NB; ++jj) {
            const double piv = readlane_f64(a[jj], jj);
            const bool live = OF_NB * b + jj < k;
            const bool usable = piv > readlane_f64(thl, jj);
            const double y = __builtin_amdgcn_rsq(piv);
            const double tq = piv * y;
            const double eq = fma(-tq, y, 1.0);
            const double hq = y * fma(0.375, eq, 0.5);
            const double d = (usable && live) ? fma(hq, eq, y) : 0.0;
            a[jj] *= d;
            binv[jj] *= d;
#pragma unroll
            for (int c = jj + 1; c < OF_NB; ++c) {
              const double lcj = readlane_f64(a[jj], c);
              a[c] = fma(-a[jj], lcj, a[c]);
              binv[c] = fma(-binv[jj], lcj, binv[c]);
            }
          }
        }
#undef CR_LOAD_ROWS
        // the rows of L_bb and of L_bb^{-T} to LDS (the helper copies them to global memory later)
        if (lane < 16) {
          double* const lrow = Ltile + ((b & 1) * 16 + lc) * CR_TP;
          double* const irow = LinvT + ((b & 1) * 16 + lc) * CR_TP;
#pragma unroll
          for (int c = 0; c < OF_NB; c += 2) {
            *(double2*)(irow + c) = double2{binv[c], binv[c + 1]};
            *(double2*)(lrow + c) = double2{a[c], a[c + 1]};
          }
        }
        if (lane == 0 && any_bad) {
          if (unshifted_attempt) restart = 1; else deficient = 1;
        }
      };

      __builtin_amdgcn_s_setprio(3);
      {
        // block (0, 0), whose diagonal is all that its own thresholds need
        f64x4 first;
        CR_LOAD_BLOCK(first, 0, 0);
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (4 * lr + r == lc) gdiag[lc] = first[r];
        CR_FIX_DIAG(first, 0);
        factor_diag(0, first);
      }
      __syncthreads();
      // (the flag is made wave-uniform for the compiler)
      for (int j = 0; j < nb - 1 && !__builtin_amdgcn_readfirstlane(restart); ++j) {
        const int b = j + 1;
        // Panel j applied to diagonal block b.  The one block of the panel that this takes, P = L[b][j], is formed here
        // as well, from the staged U(j, b), instead of waiting for the workers' phase A to leave it in Pt (at 128 columns
        // that wait was 2000 of a panel's 8000 clocks).
        f64x4 p = {0.0, 0.0, 0.0, 0.0}, dacc;
#pragma unroll
        for (int r = 0; r < 4; ++r) dacc[r] = Dstage[(b & 1) * 256 + r * 64 + lane];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
          p = mfma_f64(LinvT[((j & 1) * 16 + 4 * lr + kk) * CR_TP + lc], Ustage[(b & 1) * 256 + kk * 64 + lane], p);
#pragma unroll
        for (int r = 0; r < 4; ++r) Dtile[(lr + 4 * r) * 17 + lc] = p[r];       // P^T, register r: row lr + 4 r
        __builtin_amdgcn_wave_barrier();      // LDS operations of one wave complete in order
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) dacc = mfma_f64_sub(Dtile[(4 * kk + lr) * 17 + pm], p[kk], dacc);
        __builtin_amdgcn_wave_barrier();
        sb_barrier_lds();                     // (the workers' panel j is in Pt)
        factor_diag(b, dacc);
        sb_barrier_lds();                     // restart, if set, was written before this barrier
      }
      __builtin_amdgcn_s_setprio(0);
    } else {
      if constexpr (PARKS) {                  // (block 0, which is unused, where there are none left)
        constexpr int PER = (NBM - 1 + CR_WORKERS) / (CR_WORKERS + 1);
        f64x4 row0[PER];
#pragma unroll
        for (int q = 0; q < PER; ++q) {
          const int I = 1 + worker + q * (CR_WORKERS + 1);
          CR_LOAD_BLOCK(row0[q], 0, I < nb ? I : 0);
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
          const int I = 1 + worker + q * (CR_WORKERS + 1);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            if (I < nb) Park[256 * (I - 1) + r * 64 + lane] = row0[q][r];
            if (I == 1) Ustage[256 + r * 64 + lane] = row0[q][r];
          }
        }
      }
      // ---- workers load their blocks (all loads are issued before the first use)
      f64x4 acc[SLOTS];
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        CR_SLOT(s, C, I);
        CR_LOAD_BLOCK(acc[s], C, I);
      }
      // the helper also the diagonal (pivot thresholds), whose sum is the shift of a second attempt
      constexpr int DIAGS = (OF_NB * NBM + 63) / 64;
      const bool diagonal = wave == CR_HELPER && (attempt == 0 || !try_unshifted);
      double dg[DIAGS];
      if (diagonal) {
#pragma unroll
        for (int q = 0; q < DIAGS; ++q) {
          const int i = lane + 64 * q, ic = i < kp ? i : kp - 1;
          dg[q] = src[backup ? gram_backup_at(ic, ic, kp) : (int64_t)ic * kp + ic];
        }
      }
#pragma unroll
      for (int s = 0; s < SLOTS; ++s) {
        CR_SLOT(s, C, I);
        if (C == I) {
          CR_FIX_DIAG(acc[s], C);
          if (C == 1) {                       // wave 0 takes it after block (0, 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) Dstage[256 + r * 64 + lane] = acc[s][r];
          }
        } else if (C == 0 && I == 1) {
#pragma unroll
          for (int r = 0; r < 4; ++r) Ustage[256 + r * 64 + lane] = acc[s][r];
        }
      }
      // Block b's factors, left in LDS by wave 0, to global memory: the inverse, and L itself
      auto copy_out = [&](const int b, const bool inverse, const bool block) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int e = lane + 64 * q, r = e >> 4, c = e & 15;
          const double dv = LinvT[((b & 1) * 16 + c) * CR_TP + r];      // Dinv[b][r][c] = Linv[r][c] = LinvT[c][r]
          const double lv = Ltile[((b & 1) * 16 + r) * CR_TP + c];
          double* const at = G + (int64_t)(OF_NB * b + r) * kp + OF_NB * b + c;
          if (inverse) {
            if (PUB) cf_store(g.Dinv + (int64_t)b * 256 + e, dv); else g.Dinv[(int64_t)b * 256 + e] = dv;
          }
          if (block && c < r) {
            if (PUB) cf_store(at, lv); else *at = lv;
          }
        }
      };
      // Said to the compiler as well (an assembly statement would not): while it takes a block for possibly under way it waits
      // for it at its first use in the loop below, each time round, and with it for every store of the factor in flight.
      SB_WAIT_VMCNT(0);
      __syncthreads();
      if (diagonal) {
        // (read by wave 0 after the loop's first barrier, those of block 0 are its own)
        double tr = 0.0;
#pragma unroll
        for (int q = 0; q < DIAGS; ++q) {
          const int i = lane + 64 * q;
          if (i >= OF_NB && i < kp) gdiag[i] = dg[q];
          tr += dg[q] * (i < kp ? 1.0 : 0.0);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) tr += __shfl_xor(tr, off);
        if (lane == 0) misc[0] = tr;
      }
      int jdone = -1;                         // last panel whose factors were copied out
      for (int j = 0; j < nb - 1 && !__builtin_amdgcn_readfirstlane(restart); ++j) {
        // ---- phase A: the rows of panel j, P_I^T = Linv_j U(j, I), to LDS
        // (slots are looked at four at a time)
        bool skip = false;
        double la[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) la[kk] = LinvT[((j & 1) * 16 + 4 * lr + kk) * CR_TP + lc];
        if constexpr (PARKS) if (j == 0) {
          for (int I = 1 + worker; I < nb; I += CR_WORKERS + 1) {     // (each parked by the wave that reads it)
            f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) d = mfma_f64(la[kk], Park[256 * (I - 1) + kk * 64 + lane], d);
            double* const at = Pt + lr * ptld + OF_NB * (I - 1) + (lc ^ CR_SWZ(lr));
#pragma unroll
            for (int r = 0; r < 4; ++r) at[4 * r * ptld] = d[r];
          }
        }
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          if (s % 4 == 0) skip = CR_ROW(s) != j && CR_ROW(s + 1) != j && CR_ROW(s + 2) != j && CR_ROW(s + 3) != j;
          if (skip) continue;
          CR_SLOT(s, C, I);
          if (C == j && I > j) {
            f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) d = mfma_f64(la[kk], acc[s][kk], d);
            double* const at = Pt + lr * ptld + OF_NB * (I - j - 1) + (lc ^ CR_SWZ(lr));
#pragma unroll
            for (int r = 0; r < 4; ++r) at[4 * r * ptld] = d[r];
          }
        }
        // The barriers of this loop order LDS only: a store takes about a microsecond to complete, and wave 0 would
        // wait for it at either of them.  The stores of panel j - 1 are a phase B old here.
        if (PUB) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        sb_barrier_lds();

        // ---- phase B: panel j to L, and applied to the trailing matrix (wave 0 factors block j + 1).
        jdone = j;
        if (wave == CR_HELPER) {
          // block row j of L (its last piece was panel j - 1) and Dinv up to block j - 1 are in memory
          if (PUB && lane == 0 && j > 0) cf_publish(g.ready, attempt_pub, j);
          copy_out(j, true, true);            // its LDS copy is overwritten two panels later
        } else {
          // Whole rows of the panel, eight of them a store instruction: element by element as the matrix instructions leave
          // it, a store touches sixteen lines, and 15 blocks of them took 4000 clocks of phase A.
          for (int x0 = 8 * worker; x0 < OF_NB * (nb - 1 - j); x0 += 8 * CR_WORKERS) {
            const int x = x0 + (lane >> 3), p = 2 * (lane & 7);
            const double* const from = Pt + p * ptld + (x ^ CR_SWZ(p));
            const f64x2 v = {from[0], from[ptld]};
            double* const at = G + (OF_NB * (j + 1) + x) * kp + OF_NB * j + p;
            if (PUB) cf_store2(at, v); else *(f64x2*)at = v;
          }
        }
        // Vector instructions do not run beside a float64 matrix instruction of the same SIMD, so addresses are kept to two a
        // block: row offsets are immediate.
        const int b = j + 1;
        LdsDouble pa = (LdsDouble)(Pt + lr * ptld + (pm ^ CR_SWZ(lr))), pb = (LdsDouble)(Pt + lr * ptld + (lc ^ CR_SWZ(lr)));
        asm volatile("" : "+v"(pa), "+v"(pb));  // (or the constant part of the address is added again for every block)
#pragma unroll
        for (int s = 0; s < SLOTS; ++s) {
          if (s % 4 == 0) skip = CR_ROW(s) <= j && CR_ROW(s + 1) <= j && CR_ROW(s + 2) <= j && CR_ROW(s + 3) <= j;
          if (skip) continue;
          CR_SLOT(s, C, I);
          if (C > j && I > b) {
            LdsDouble xc = pa + OF_NB * (C - b), xi = pb + OF_NB * (I - b);
            double a[4], x[4];
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) { a[kk] = xc[4 * kk * ptld]; x[kk] = xi[4 * kk * ptld]; }
            __builtin_amdgcn_sched_barrier(0);  // (one wait for LDS a block)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) acc[s] = mfma_f64_sub(a[kk], x[kk], acc[s]);
            if (I == b + 1 && C >= b) {       // the diagonal block wave 0 takes next, and the one above it
              double* const st = (C == I ? Dstage : Ustage) + (I & 1) * 256;
#pragma unroll
              for (int r = 0; r < 4; ++r) st[r * 64 + lane] = acc[s][r];
            }
          }
        }
        sb_barrier_lds();
      }
      // the blocks not copied yet: the last one factored, and the one before it if the loop did not run for it (their LDS buffers
      // differ).  Of few columns two waves take a factor each (one-launch QR of 150 x 29, us, by the helper alone 20.7, by two
      // 20.1); the registers that this takes are missed by the wide ones (in one launch with the solve 8192 x 256 163 and 168, compress).
      constexpr bool TWO = NBM <= 4 && !PUB;
      if ((TWO || wave == CR_HELPER) && !__builtin_amdgcn_readfirstlane(restart)) {
        for (int b = jdone + 1; b < nb; ++b) {
          if (!TWO) copy_out(b, true, true);
          else if (wave == CR_HELPER) copy_out(b, true, false);
          else if (wave == 1) copy_out(b, false, true);
        }
      }
    }
    if (!__builtin_amdgcn_readfirstlane(restart)) break;
    __syncthreads();                          // everyone has seen the flag
    if (t == 0) restart = 0;
    __syncthreads();
  }
#undef CR_SLOT
#undef CR_ROW
#undef CR_SWZ
#undef CR_LOAD_BLOCK
#undef CR_FIX_DIAG
  if (PUB) {
    // the last factors were copied out after the loop: once every wave's stores are complete the
    // whole of L and Dinv is published (attempt 1 if the unshifted one was abandoned)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (t == 64 * CR_HELPER) cf_publish(g.ready, attempt_pub, nb);
  }
  if (t == 0 && deficient && g.status) atomicOr(g.status, LORACT_STATUS_RANK_DEFICIENT);
}

// What the factorising workgroup 0 reads first, the backup's blocks on and below the diagonal, touched by the workgroups that run on its
// XCD (8, 16, ...: workgroup b runs on XCD b mod 8): one CU has room for some 28 GB/s of misses of its L2, and finds there what others
// fetched side by side.
#define CR_PREFETCH_WGS 16
__device__ inline void chol_prefetch(const CholArgs& g) {
  const int n = ((int)gridDim.x - 1) / 8, h = (int)blockIdx.x / 8 - 1, nb = g.kp / OF_NB;
  if (g.round != 1 || !g.G_backup || (blockIdx.x & 7) != 0 || blockIdx.x == 0) return;
  for (int e = h * CR_THREADS + threadIdx.x; e < nb * nb * 16; e += n * CR_THREADS) {       // 16 lines of 128 bytes a block
    const int block = e >> 4, row = block / nb;
    if (block - row * nb > row) continue;
    const double v = g.G_backup[(int64_t)e * 16];
    asm volatile("" : : "v"(v));
  }
}

template <int NBM>
__global__ __launch_bounds__(CR_THREADS) void chol_reg_kernel(CholArgs g) {
  extern __shared__ double smem[];
  if (blockIdx.x == 0) chol_reg_body<NBM, false>(g, smem);
  else chol_prefetch(g);
}

// ---------------------------------------------------------------------------------------------
// Q = Y R^{-1} with R = L^T, as a blocked triangular solve per 16-row strip (one wave each):
//   for J = 0 .. NJ-1:   T = Y[:, J] - sum_{I < J} Q[:, I] R[I, J];   Q[:, J] = T R[J, J]^{-1}
// evaluated transposed (Q_J^T = Linv_JJ (Y_J^T - sum_I L[J, I] Q_I^T)) so that each finished
// 16 x 16 block of Q^T stays in the accumulator layout and is reused directly as the B operand.

struct TrsmArgs {
  const float* Y;       // m x kp, ld = ldy
  int64_t ldy;
  const double* L;      // kp x kp, strict lower triangle valid
  const double* Dinv;   // NJ blocks of 16 x 16
  int64_t m;
  int kp;
  int k;
  void* Q;              // output
  int64_t ldq;
  int out_ek;           // EK_F32 (all kp columns written) or EK_BF16 / EK_F32 final (k columns)
  int out_cols;         // number of columns to write (kp or k)
  bf16_t* Qb;           // optional second bf16 copy (ld = ldqb, out_cols columns), may be null
  int64_t ldqb;
  const int32_t* skip_flag;   // optional: the launch does nothing when *skip_flag != 0
  double* gram_part;          // optional (solve_body, half of whose waves own rows): partial tiles of Q^T Q, Q as float32
};

// Workgroup = WAVES waves = 16 WAVES rows of Y.  The operands every wave needs -- block row J of
// L left of the diagonal and the inverted diagonal block, together "panel J", 16 x 16 (J + 1)
// doubles -- are staged in LDS once per workgroup by asynchronous global -> LDS copies instead of
// being fetched by every wave:
//   panels 0 .. J0-1 (J0 = min(NJ, 8), 6 for the widest) are copied up front, side by side in one 16-row array;
//   panel J + 1 >= J0 is copied into the other half of a double buffer while step J runs.
// The LDS row pitches are 2 modulo 32 doubles (or 18), which spreads the 16 rows that one matrix
// instruction operand touches over distinct banks.
#define TRSM_J0(NJ) ((NJ) < 8 ? (NJ) : ((NJ) > 16 ? 6 : 8))
#define TRSM_TILE_FLOATS (16 * 20)     // per-wave staging tile for the stores: 16 rows, pitch 20 floats
#define TRSM_SPIN_LIMIT (1 << 22)      // polls of the progress word before a solving workgroup gives up

// Stores Q_J (o: register r of lane (lr, lc) is column 16 J + 4 r + lr of row `row`) to Q and, if given, Qb.  With
// vec_ok the 16 x 16 block is turned through a wave-private LDS tile (LDS operations of one wave execute in
// order) so that every lane stores 4 consecutive columns at once.
__device__ __forceinline__ void trsm_store_block(const TrsmArgs& g, const f64x4 o, int J, int64_t row, bool rok, bool vec_ok,
                                                 float* tile, int lc, int lr) {
  if (vec_ok && 16 * J + 16 <= g.out_cols) {
#pragma unroll
    for (int r = 0; r < 4; ++r) tile[lc * 20 + 4 * r + lr] = (float)o[r];
    const f32x4 v = *(const f32x4*)(tile + lc * 20 + 4 * lr);
    bf16x4 vh;
#pragma unroll
    for (int u = 0; u < 4; ++u) vh[u] = (bf16_t)v[u];
    if (rok) {
      const int col = 16 * J + 4 * lr;
      if (g.out_ek == EK_F32) *(f32x4*)((float*)g.Q + row * g.ldq + col) = v;
      else *(bf16x4*)((bf16_t*)g.Q + row * g.ldq + col) = vh;
      if (g.Qb) *(bf16x4*)(g.Qb + row * g.ldqb + col) = vh;
    }
  } else if (rok) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int col = 16 * J + 4 * r + lr;
      if (col < g.out_cols) {
        if (g.out_ek == EK_F32) ((float*)g.Q)[row * g.ldq + col] = (float)o[r];
        else ((bf16_t*)g.Q)[row * g.ldq + col] = (bf16_t)(float)o[r];
        if (g.Qb) g.Qb[row * g.ldqb + col] = (bf16_t)(float)o[r];
      }
    }
  }
}
// Columns c .. c + 3 (c a multiple of 4; those below l) of row r of the basis, to Q and, if given, its bf16 copy, both with
// row pitch l; vec_ok: pitch and base addresses keep such groups aligned.
__device__ __forceinline__ bool basis_vec_ok(const void* Q, const bf16_t* Qb, int64_t l) {
  return (l & 3) == 0 && ((uintptr_t)Q & 15) == 0 && ((uintptr_t)Qb & 7) == 0;
}
__device__ __forceinline__ void basis_store(const f32x4 q, int64_t r, int c, int l, void* Q, int q_ek, bf16_t* Qb, bool vec_ok) {
  const int64_t at = r * l + c;
  if (vec_ok) {
    if (c >= l) return;
    bf16x4 qh;
#pragma unroll
    for (int u = 0; u < 4; ++u) qh[u] = (bf16_t)q[u];
    if (q_ek == EK_F32) *(f32x4*)((float*)Q + at) = q;
    else *(bf16x4*)((bf16_t*)Q + at) = qh;
    if (Qb) *(bf16x4*)(Qb + at) = qh;
    return;
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (c + u < l) {
      if (q_ek == EK_F32) ((float*)Q)[at + u] = q[u];
      else ((bf16_t*)Q)[at + u] = (bf16_t)q[u];
      if (Qb) Qb[at + u] = (bf16_t)q[u];
    }
  }
}
// 4 consecutive output columns per lane can be stored as one vector
__device__ __forceinline__ bool trsm_vec_ok(const TrsmArgs& g) {
  return (g.ldq & 3) == 0 && ((uintptr_t)g.Q & 15) == 0 && (!g.Qb || ((g.ldqb & 3) == 0 && ((uintptr_t)g.Qb & 7) == 0));
}

// L and Dinv are complete when the kernel starts.  A workgroup takes the strips first_strip, first_strip +
// strip_stride, ... of 16 WAVES rows one after the other (several only with NJ <= J0: the double buffer is not
// ordered between strips).
template <int NJ, int WAVES>
__device__ inline void trsm_body(const TrsmArgs& g, const int first_strip, const int strip_stride, double* trsm_lds) {
  constexpr int J0 = TRSM_J0(NJ);
  constexpr int PK = 8 * J0 * (J0 + 1) + 2;           // pitch of the side-by-side array, in doubles
  constexpr int PR = 16 * NJ + 2;                     // pitch of a double-buffer half
  double* const ring = trsm_lds + 16 * PK;
  float* const tile = (float*)(ring + (NJ > J0 ? 32 * PR : 0)) + (threadIdx.x >> 6) * TRSM_TILE_FLOATS;
  if (g.skip_flag && *g.skip_flag != 0) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int lc = lane & 15, lr = lane >> 4;
  const int nstrips = (int)((g.m + 16 * WAVES - 1) / (16 * WAVES));
  const bool vec_ok = trsm_vec_ok(g);

  // Copy of panel J to `dst` (pitch in doubles): one wave-wide instruction per (panel row, 64
  // pieces of 16 bytes), dealt round-robin to the waves; lanes past the row end stay idle.
  auto copy_panel = [&](int J, double* dst, int pitch) {
    const int pieces = 8 * (J + 1);
    const int nq = (pieces + 63) / 64;
    for (int e = wave; e < 16 * nq; e += WAVES) {
      const int r = e / nq, q = e - r * nq;
      const int c = 2 * (64 * q + lane);
      if (c < 16 * (J + 1)) {
        const double* src = c < 16 * J ? g.L + (int64_t)(16 * J + r) * g.kp + c
                                        : g.Dinv + ((int64_t)J * 16 + r) * 16 + (c - 16 * J);
        sb_async16(src, (unsigned char*)(dst + r * pitch) + q * 1024);
      }
    }
  };
#pragma unroll
  for (int J = 0; J < J0; ++J) copy_panel(J, trsm_lds + 8 * J * (J + 1), PK);
  SB_WAIT_VMCNT(0);
  __syncthreads();

  f64x4 qb[NJ];
  float ycur[4], ynext[4];
  for (int strip = first_strip; strip < nstrips; strip += strip_stride) {
    const int64_t row = (int64_t)strip * (16 * WAVES) + wave * 16 + lc;
    const bool rok = row < g.m;
    // every row of the wave exists: its store instructions per step can be counted
    const bool full_wave = (int64_t)strip * (16 * WAVES) + wave * 16 + 15 < g.m;
    const float* yrow = g.Y + (rok ? row : 0) * g.ldy;   // rows past m read row 0 and are never stored
#pragma unroll
    for (int r = 0; r < 4; ++r) ycur[r] = yrow[4 * r + lr];
#pragma unroll
    for (int J = 0; J < NJ; ++J) {
      const bool ring_next = J + 1 >= J0 && J + 1 < NJ;
      if (ring_next) copy_panel(J + 1, ring + ((J + 1) & 1) * 16 * PR, PR);
      if (J + 1 < NJ) {
#pragma unroll
        for (int r = 0; r < 4; ++r) ynext[r] = yrow[16 * (J + 1) + 4 * r + lr];
      }
      const double* pan = J < J0 ? trsm_lds + lc * PK + 8 * J * (J + 1) : ring + (J & 1) * 16 * PR + lc * PR;
      f64x4 s = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int I = 0; I < J; ++I) {
#pragma unroll
        for (int r = 0; r < 4; ++r) s = mfma_f64(pan[16 * I + 4 * r + lr], qb[I][r], s);
      }
      f64x4 tt;
#pragma unroll
      for (int r = 0; r < 4; ++r) tt[r] = (double)ycur[r] - s[r];
      f64x4 o = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int r = 0; r < 4; ++r) o = mfma_f64(pan[16 * J + 4 * r + lr], tt[r], o);
      qb[J] = o;
      trsm_store_block(g, o, J, row, rok, vec_ok, tile, lc, lr);
      if (J + 1 < NJ) {
#pragma unroll
        for (int r = 0; r < 4; ++r) ycur[r] = ynext[r];
      }
      if (J + 1 >= J0 && J + 1 < NJ) {
        // The copies of panel J + 1 are older than this step's stores (1 per wave on the vector
        // path, 2 with the second output; every column of a step that is not the last lies inside
        // out_cols), so they have landed once at most that many operations are pending.  The barrier also orders this step's
        // reads of its buffer half before the copy that the next step issues into it.
        if (!full_wave || !vec_ok) SB_WAIT_VMCNT(0);
        else if (g.Qb) SB_WAIT_VMCNT(2);
        else SB_WAIT_VMCNT(1);
        sb_barrier_lds();
      }
    }
  }
}

template <int NJ, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void trsm_apply_kernel(TrsmArgs g) {
  extern __shared__ __attribute__((aligned(16))) double trsm_lds[];
  trsm_body<NJ, WAVES>(g, blockIdx.x, gridDim.x, trsm_lds);
}

template <int NJ, int WAVES>
static constexpr size_t trsm_lds_bytes() {
  constexpr int J0 = TRSM_J0(NJ);
  return ((size_t)16 * (8 * J0 * (J0 + 1) + 2) + (NJ > J0 ? (size_t)32 * (16 * NJ + 2) : 0)) * sizeof(double) +
         (size_t)WAVES * TRSM_TILE_FLOATS * sizeof(float) + 16;
}

// The solve beside the factorisation (chol_trsm_fused_kernel), in the other order: as soon as panel J -- the
// inverted diagonal block and block COLUMN J of L below it -- is complete, Q_J = T_J Linv_JJ^T is formed, and then taken
// out of all later blocks, T_J' -= Q_J L[J', J]^T.  After the last panel only one 16 x 16 product remains, and
// the rest of a step's work runs while the next panel is factored.  (Left-looking, block row J at step J, a strip
// of 256 columns had 64 matrix instructions to go after the last panel and fell behind by three panels: 8192 rows,
// 128 columns 35.4 us, 256 columns 108.)  Only the first `row_waves` waves own rows, 16 each: with half of
// them, one per SIMD, a step takes half the time, and there are CUs enough for the twice as many workgroups up to
// 16320 rows (8192 rows: 28.6 us against 29.9 at 128 columns, 88.7 against 90.2 at 256).
//
// Panel J in LDS: rows of 16 doubles in 16-byte pieces, piece p of row r at position p ^ (r & 7) (the 16 rows of an
// operand then fall into different banks); rows 0 .. 15 are Linv_JJ, row 16 + i is row 16 (J + 1) + i of L.  It goes to
// half J & 1 of a double buffer, and panel J + 1 is copied ahead if it is complete already.  A change of the attempt
// number sends the workgroup back to its first strip: everything it wrote so far belongs to the abandoned attempt.
//
// Up to 64 columns the waves without rows form the Gram matrix of the result (g.gram_part) from float32 copies of the finished
// blocks in LDS, block row J while the next panel is awaited or taken out: the second round's product then needs no launch of its own
// and Q1 is not read again; what remains after the last panel is one block row for all eight waves.  Gram products and factor and
// solve, both rounds, us event to event: 12608 x 32 12.8 + 19.9 -> 6.5 + 20.2, 8192 x 64 17.3 + 25.1 -> 9.0 + 26.4.  With more
// columns the block rows no longer fit between two panels and the launch grows by what the other one cost: 8192 x 128
// 23.8 + 34.0 -> 11.6 + 43.0, 1000 x 96 15.8 + 27.8 -> 8.0 + 32.3, 8192 x 256 37 + 82 -> 19 + 98 and four times the partial tiles.
#define SOLVE_GRAM_MAX 4                 // columns / 16
#define SOLVE_GRAM_ROWS (16 * CR_THREADS / 128)
static constexpr int solve_gram_pitch(int nj) { return (16 * nj + 63) / 64 * 64 + 16; }  // (four rows of an operand in distinct banks)
template <int NJ>
static constexpr size_t solve_lds_bytes() {
  return (size_t)2 * 256 * (NJ + 1) * sizeof(double) + (size_t)(CR_THREADS / 64) * TRSM_TILE_FLOATS * sizeof(float) +
         (NJ <= SOLVE_GRAM_MAX ? (size_t)SOLVE_GRAM_ROWS * solve_gram_pitch(NJ) * sizeof(float) : 0) + 16;
}
template <int NJ>
__device__ inline void solve_body(const TrsmArgs& g, const int first_strip, const int strip_stride, const int row_waves,
                                  double* lds, const int32_t* ready, int32_t* status) {
  constexpr int WAVES = CR_THREADS / 64, HALF = 256 * (NJ + 1);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int lc = lane & 15, lr = lane >> 4;
  float* const tile = (float*)(lds + 2 * HALF) + wave * TRSM_TILE_FLOATS;
  constexpr int GP = solve_gram_pitch(NJ);
  float* const rows_f32 = (float*)(lds + 2 * HALF) + WAVES * TRSM_TILE_FLOATS;     // [SOLVE_GRAM_ROWS][GP], for the Gram matrix
  constexpr bool GRAM = NJ <= SOLVE_GRAM_MAX;
  int* const word = (int*)(rows_f32 + (GRAM ? SOLVE_GRAM_ROWS * GP : 0));          // the progress word as the workgroup saw it
  const bool solves = wave < row_waves;
  const int strip_rows = 16 * row_waves;
  const int nstrips = (int)((g.m + strip_rows - 1) / strip_rows);
  const bool vec_ok = trsm_vec_ok(g);

  // (device-scope loads: the panel was written by another workgroup of this launch)
  auto copy_panel = [&](int J) {
    unsigned char* const dst = (unsigned char*)(lds + (J & 1) * HALF);
    for (int e = wave; e < 2 * (NJ - J); e += WAVES) {               // 8 rows per instruction
      const int row = 8 * e + (lane >> 3), piece = (lane & 7) ^ (row & 7);
      const double* src = row < 16 ? g.Dinv + ((int64_t)J * 16 + row) * 16 : g.L + (int64_t)(16 * J + row) * g.kp + 16 * J;
      sb_async16_device(src + 2 * piece, dst + e * 1024);
    }
  };
  // The whole workgroup learns the progress word: one poll per trip, shared through LDS.  The first one was sent off while
  // the step before was computed, so it may be older than what a later poll of the last wait returned.
  int polled = 0;
  auto poll = [&](int spin) -> int {
    if (spin > 1) __builtin_amdgcn_s_sleep(2);
    if (t == 0) *word = spin == 0 ? polled : cf_poll(ready);
    sb_barrier_lds();
    const int f = *word;
    sb_barrier_lds();                    // everyone has read the word before the next poll rewrites it
    return f;
  };
  int off[4];                            // slice r of a block's operand: entry (lc, 4 r + lr)
#pragma unroll
  for (int r = 0; r < 4; ++r) off[r] = lc * 16 + (((2 * r + (lr >> 1)) ^ (lc & 7)) << 1) + (lr & 1);

  // tiles (J, I), I = first, first + step, ... <= J, of the Gram matrix of this workgroup's rows
  auto gram_tiles = [&](const int J, const int first, const int step) {
    const float* const from = rows_f32 + lr * GP + lc;
    double a[SOLVE_GRAM_ROWS / 4];
#pragma unroll
    for (int q = 0; q < SOLVE_GRAM_ROWS / 4; ++q) a[q] = (double)from[4 * q * GP + 16 * J];
#pragma nounroll
    for (int I = first; I <= J; I += step) {
      f64x4 d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < SOLVE_GRAM_ROWS / 4; ++q) d = mfma_f64(a[q], (double)from[4 * q * GP + 16 * I], d);
      double* const out = g.gram_part + ((int64_t)first_strip * (NJ * (NJ + 1) / 2) + J * (J + 1) / 2 + I) * 256 + lane;
#pragma unroll
      for (int r = 0; r < 4; ++r) out[64 * r] = d[r];
    }
  };
  const bool gram = GRAM && g.gram_part != nullptr;     // (then one strip, and waves without rows)

  CfProgress at;                         // (uniform in the workgroup)
  // A workgroup takes the strips first_strip, first_strip + strip_stride, ... one after the other (fewer workgroups than
  // strips when the matrix is tall; once the progress word has been seen complete no strip polls again).
  for (int strip = first_strip; strip < nstrips; strip += strip_stride) {
    const int64_t row = (int64_t)strip * strip_rows + wave * 16 + lc;
    const bool rok = solves && row < g.m;
    const float* yrow = g.Y + (rok ? row : 0) * g.ldy;   // rows past m read row 0 and are never stored
    f64x4 T[NJ];
    {
      float y[NJ][4];
#pragma unroll
      for (int J = 0; J < NJ; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) y[J][r] = yrow[16 * J + 4 * r + lr];
#pragma unroll
      for (int J = 0; J < NJ; ++J)
#pragma unroll
        for (int r = 0; r < 4; ++r) T[J][r] = (double)y[J][r];
    }
    bool next_copied = false;
    // Step J up to where panel J lies in LDS; the same for every wave.
    auto step = [&](const int J) -> int {
      const int go = cf_wait_panel(at, J, TRSM_SPIN_LIMIT, poll);
      if (go != CF_TAKE) return go;
      if (!next_copied) copy_panel(J);
      SB_WAIT_VMCNT(0);
      sb_barrier_lds();                                  // everyone's share of panel J landed; panel J - 1 has been read
      next_copied = J + 1 < NJ && at.known > cf_word(at.attempt, J + 1);  // the next panel is complete as well: copy it ahead
      if (next_copied) copy_panel(J + 1);
      if (t == 0) polled = cf_poll(ready);
      return go;
    };
    int go = CF_TAKE;
    if (solves) {
#pragma unroll
      for (int J = 0; J < NJ; ++J) {
        if (go != CF_TAKE) continue;                     // (uniform) drain the unrolled loop
        go = step(J);
        if (go != CF_TAKE) continue;
        const double* const pan = lds + (J & 1) * HALF;
        f64x4 o = (f64x4){0.0, 0.0, 0.0, 0.0}, q;
#pragma unroll
        for (int r = 0; r < 4; ++r) o = mfma_f64(pan[off[r]], T[J][r], o);
        trsm_store_block(g, o, J, row, rok, vec_ok, tile, lc, lr);
        if (gram) {
#pragma unroll
          for (int r = 0; r < 4; ++r) rows_f32[(wave * 16 + lc) * GP + 16 * J + 4 * r + lr] = rok ? (float)o[r] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) q[r] = -o[r];
#pragma unroll
        for (int I = J + 1; I < NJ; ++I)
#pragma unroll
          for (int r = 0; r < 4; ++r) T[I] = mfma_f64(pan[256 * (I - J) + off[r]], q[r], T[I]);
      }
    } else {
      // (not unrolled: what runs once or twice runs from a cold instruction cache)
#pragma nounroll
      for (int J = 0; J < NJ; ++J) {
        go = step(J);
        if (go != CF_TAKE) break;
        if (gram && J > 0) gram_tiles(J - 1, wave - row_waves, WAVES - row_waves);
      }
    }
    if (go == CF_GIVE_UP) {                              // the factorisation never got here: flagged
      if (t == 0 && status) atomicOr(status, LORACT_STATUS_INTERNAL);
      return;
    }
    const bool restart_solve = go == CF_RESTART;         // the attempt changed
    if (gram && !restart_solve) {
      sb_barrier_lds();
      gram_tiles(NJ - 1, wave, WAVES);
    }
    sb_barrier_lds();                    // this strip's last reads of the buffer halves precede the next strip's copies
    if (restart_solve) strip = first_strip - strip_stride;        // (uniform) back to the first strip
  }
}

template <int NJ, int WAVES>
static int launch_trsm_nj_waves(hipStream_t s, const TrsmArgs& g) {
  constexpr size_t lds = trsm_lds_bytes<NJ, WAVES>();
  static std::atomic<bool> attr_done{false};
  if (lds > 64 * 1024 && !attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)trsm_apply_kernel<NJ, WAVES>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(trsm LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("trsm_apply", s, (trsm_apply_kernel<NJ, WAVES>),
                dim3((unsigned)ceil_div64(g.m, 16 * WAVES)), dim3(64 * WAVES), lds, g);
  return LORACT_OK;
}

// ---------------------------------------------------------------------------------------------
// Factorisation and triangular solve of round 1 in ONE launch: workgroup 0 factors the Gram
// matrix (chol_reg_body, publishing), workgroups 1 .. solve their 64 or 128 rows of Y panel by panel
// as the factor appears (solve_body), so that one 16 x 16 product and its stores remain after the factorisation ends
// instead of a launch of their own.  Workgroup 0 waits for nobody, and is dispatched
// first, so the others' bounded waits cannot starve it.  The progress word must be zero when the
// launch starts (an earlier kernel of the same call clears it).
//
// Where round 2 has no Newton-Schulz finish, which would write the factors, the launch that accepts Q1 converts it as well (12608 x 32: 3.9 us, as two
// launches 2.7 and 3.4).  Whole compress of flat spectra, us less than with a launch of its own: 16 to 48 columns 1 to 2.5, 80 0.3 to 0.8, 112 0 to 0.8, but 144 to
// 240 columns 0.5 to 1.6 more, because the kernel of the factorisation grows by the code for it.  Its 256 workgroups convert at 3 TB/s, a
// launch of as many as are useful at 4.8: from 4M values on that is what counts (262144 x 16 0.3 less, x 112 6.8 more, x 176 50 more).
static constexpr bool round2_width_converts(int kp) { return kp % 64 != 0 && kp < 128; }
__host__ __device__ static inline bool round2_converts(int64_t m, int kp) { return round2_width_converts(kp) && m * kp <= 4 << 20; }
template <int NBM, int NJ>
__global__ __launch_bounds__(CR_THREADS) void chol_trsm_fused_kernel(CholArgs c, TrsmArgs g, int row_waves) {
  extern __shared__ __attribute__((aligned(16))) double fused_lds[];
  // Round 2: whether Q1 needs a second factorisation at all is decided from the shares of
  // ||E||_F^2 that the Gram reduction left -- by every workgroup for itself, with the same
  // arithmetic in the same order, so that on the usual exits (Newton-Schulz finish, or Q1 accepted
  // as it is) the whole launch ends after one look at those few hundred numbers and nobody waits
  // for anybody.  Workgroup 0 records the decision in *ns_flag.
  if (c.round == 2 && c.ns_flag) {
    if constexpr (round2_width_converts(OF_NB * NJ)) {
      // (the thread's first piece of Q1 is under way meanwhile)
      const int c4 = g.kp >> 2;
      const int64_t total = round2_converts(g.m, OF_NB * NJ) ? g.m * c4 : 0, step = (int64_t)gridDim.x * CR_THREADS;
      int64_t e = (int64_t)blockIdx.x * CR_THREADS + threadIdx.x;
      f32x4 q = *(const f32x4*)(g.Y + (e < total ? e : 0) * 4);
      if (chol_round2_exit(c, fused_lds, blockIdx.x == 0)) {
        const bool vec_ok = basis_vec_ok(g.Q, g.Qb, g.ldq);
        while (e < total) {
          const int64_t r = total < (1ll << 31) ? (int64_t)((unsigned)e / (unsigned)c4) : e / c4;
          basis_store(q, r, (int)(e - r * c4) << 2, g.out_cols, g.Q, g.out_ek, g.Qb, vec_ok);
          e += step;
          if (e < total) q = *(const f32x4*)(g.Y + e * 4);
        }
        return;
      }
    } else if (chol_round2_exit(c, fused_lds, blockIdx.x == 0)) return;
    __syncthreads();
  }
  if (blockIdx.x == 0) chol_reg_body<NBM, true>(c, fused_lds);
  else {
    chol_prefetch(c);
    solve_body<NJ>(g, (int)blockIdx.x - 1, (int)gridDim.x - 1, row_waves, fused_lds, c.ready, c.status);
  }
}

// Few rows: 64 per workgroup so that more CUs take part; many rows: 128, which halves the panel
// traffic per row.
template <int NJ>
static int launch_trsm_nj(hipStream_t s, const TrsmArgs& g) {
  return g.m >= 32768 ? launch_trsm_nj_waves<NJ, 8>(s, g) : launch_trsm_nj_waves<NJ, 4>(s, g);
}

// ---------------------------------------------------------------------------------------------
// Higher-order finish of round 2.  With E = Q1^T Q1 - I symmetric and ||E||_2 < 1,
//   (I + E)^(-1/2) = I - E/2 + 3 E^2/8 - 5 E^3/16 + 35 E^4/128 - ...,
// so Q = Q1 (I + T) with T = -E/2 + 3 E^2/8 - 5 E^3/16 + 35 E^4/128 is orthonormal up to
// ~ (63/128) ||E||_2^5: 1.6e-4 at ||E||_2 = 0.2.  The first-order step T = -E/2 only serves
// ||E|| <= 0.015; with this one a sketch whose Gram matrix loses 14 digits (the long-context
// sites) still needs no second factorisation and no second triangular solve over the m rows.
// Two small launches on k x k matrices in float64: E^2, then E^3, E^4, T (bf16) and the shares of
// ||E^4||_F^2, from which the factorisation kernel bounds ||E||_2 before it accepts T.
// By 16 x 16 tiles.  The contraction index is dealt to the lanes in runs of four
// (lane group q of an operand holds columns 16 kb + 4 q .. + 3), the same way for both operands,
// so that every lane reads 32 contiguous bytes and a tile row is one 128-byte line; the second
// operand is read by rows too, all matrices involved being symmetric.

struct NsPolyArgs {
  const double* G;          // Q1^T Q1, full symmetric kp x kp
  double* P2;               // E^2 (kp x kp)
  bf16_t* T;                // out: the correction, kp x kp bf16
  const double* e2;         // shares of ||E||_F^2
  int e2_count;
  double* p4;               // out: one share of ||E^4||_F^2 per workgroup
  int k, kp;
  double lo_tol, hi_tol;    // active for ||E||_F in (lo_tol, hi_tol]
};

__device__ inline bool ns_poly_active(const NsPolyArgs& g, int lane) {
  // lane i adds shares i, i + 64, ... in that order; eight loads at a time are in flight (from
  // clamped indices, masked at use), or the loop is a chain of as many memory latencies
  double part_sum = 0.0;
  for (int w0 = lane; w0 < g.e2_count; w0 += 512) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int w = w0 + 64 * u;
      v[u] = g.e2[w < g.e2_count ? w : g.e2_count - 1];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (w0 + 64 * u < g.e2_count) part_sum += v[u];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) part_sum += __shfl_xor(part_sum, off);
  return part_sum > g.lo_tol * g.lo_tol && part_sum <= g.hi_tol * g.hi_tol;
}

// rows [16 t .. +15], four consecutive columns from c0 of E = G - I (live k x k part, else 0)
__device__ inline f64x4 ns_poly_e4(const NsPolyArgs& g, int row, int c0) {
  f64x4 v = *(const f64x4*)(g.G + (int64_t)row * g.kp + c0);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    if (c0 + u == row) v[u] -= 1.0;
    if (row >= g.k || c0 + u >= g.k) v[u] = 0.0;
  }
  return v;
}

// Four waves share a tile, every fourth block of the contraction each, and add up through LDS, two
// tiles per workgroup: a wave on its own walked through 16 blocks of loads one after the other (at 256 columns 14 and 16 us for the two
// launches, now 7.9 and 10.6).  All loads are written before the first product; the compiler leaves them so in the second launch, in the first it has
// seven or eight of the 16 at 256 columns in flight.  PER: blocks per wave, kp / 64.
#define NS_POLY_TILES 2
template <int PER>
__global__ __launch_bounds__(256 * NS_POLY_TILES) void ns_poly_square_kernel(NsPolyArgs g) {
  __shared__ double sums[4 * NS_POLY_TILES][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (!ns_poly_active(g, lane)) return;          // (uniform over the grid)
  constexpr int nj = 4 * PER;
  const int tile = blockIdx.x * NS_POLY_TILES + (wave >> 2), part = wave & 3;
  const int ti = tile / nj, tj = tile - ti * nj;
  const int lc = lane & 15, lr = lane >> 4;
  f64x4 a[PER], b[PER], acc = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    a[u] = ns_poly_e4(g, 16 * ti + lc, 16 * (part + 4 * u) + 4 * lr);
    b[u] = ns_poly_e4(g, 16 * tj + lc, 16 * (part + 4 * u) + 4 * lr);
  }
#pragma unroll
  for (int u = 0; u < PER; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc = mfma_f64(a[u][r], b[u][r], acc);
#pragma unroll
  for (int r = 0; r < 4; ++r) sums[wave][64 * r + lane] = acc[r];
  __syncthreads();
  // (wave `part` of a tile adds register `part` of the four)
  const int r = part, w0 = wave & ~3, e = 64 * r + lane;
  g.P2[(int64_t)(16 * ti + 4 * r + lr) * g.kp + 16 * tj + lc] = (sums[w0][e] + sums[w0 + 1][e]) + (sums[w0 + 2][e] + sums[w0 + 3][e]);
}

template <int PER>
__global__ __launch_bounds__(256 * NS_POLY_TILES) void ns_poly_finish_kernel(NsPolyArgs g) {
  __shared__ double sums[4 * NS_POLY_TILES][2][256];
  __shared__ double red[4 * NS_POLY_TILES];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (!ns_poly_active(g, lane)) {                // uniform over the grid: every wave sums the same shares
    // Not prepared: say so in the share itself.  The factorisation kernel adds the shares of
    // ||E||_F^2 in another order and may land on the other side of a threshold by a rounding;
    // an infinite share makes it reject the series instead of reading a stale value.
    if (threadIdx.x == 0) g.p4[blockIdx.x] = __builtin_huge_val();
    return;
  }
  constexpr int nj = 4 * PER;
  const int tile = blockIdx.x * NS_POLY_TILES + (wave >> 2), part = wave & 3;
  const int ti = tile / nj, tj = tile - ti * nj;
  const int lc = lane & 15, lr = lane >> 4;
  f64x4 a[PER], be[PER], bp[PER], p3 = (f64x4){0.0, 0.0, 0.0, 0.0}, p4 = (f64x4){0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int c0 = 16 * (part + 4 * u) + 4 * lr;
    a[u] = *(const f64x4*)(g.P2 + (int64_t)(16 * ti + lc) * g.kp + c0);
    be[u] = ns_poly_e4(g, 16 * tj + lc, c0);
    bp[u] = *(const f64x4*)(g.P2 + (int64_t)(16 * tj + lc) * g.kp + c0);
  }
  // the entries of E and E^2 that this lane finishes: register `part` of the tile
  const int row = 16 * ti + 4 * part + lr, col = 16 * tj + lc;
  double e = g.G[(int64_t)row * g.kp + col] - (row == col ? 1.0 : 0.0);
  const double p2 = g.P2[(int64_t)row * g.kp + col];
  if (row >= g.k || col >= g.k) e = 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      p3 = mfma_f64(a[u][r], be[u][r], p3);
      p4 = mfma_f64(a[u][r], bp[u][r], p4);
    }
#pragma unroll
  for (int r = 0; r < 4; ++r) { sums[wave][0][64 * r + lane] = p3[r]; sums[wave][1][64 * r + lane] = p4[r]; }
  __syncthreads();
  const int w0 = wave & ~3, at = 64 * part + lane;
  const double e3 = (sums[w0][0][at] + sums[w0 + 1][0][at]) + (sums[w0 + 2][0][at] + sums[w0 + 3][0][at]);
  const double e4 = (sums[w0][1][at] + sums[w0 + 1][1][at]) + (sums[w0 + 2][1][at] + sums[w0 + 3][1][at]);
  g.T[(int64_t)row * g.kp + col] = (bf16_t)(float)(-0.5 * e + 0.375 * p2 - 0.3125 * e3 + 0.2734375 * e4);
  double share = e4 * e4;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) share += __shfl_xor(share, off);
  if (lane == 0) red[wave] = share;
  __syncthreads();
  if (threadIdx.x == 0) {
    double total = red[0];
#pragma unroll
    for (int w = 1; w < 4 * NS_POLY_TILES; ++w) total += red[w];
    g.p4[blockIdx.x] = total;
  }
}

// kp a multiple of 64, up to 320.
static inline int ns_poly_blocks(int kp) { return (kp / 16) * (kp / 16) / NS_POLY_TILES; }
#define NS_POLY_MAX_BLOCKS 200
static int launch_ns_poly(hipStream_t s, const NsPolyArgs& g) {
  const dim3 grid((unsigned)ns_poly_blocks(g.kp)), block(256 * NS_POLY_TILES);
  switch (g.kp) {
#define NP_CASE(PER)                                                                                 \
  case 64 * PER:                                                                                     \
    LORACT_LAUNCH("ns_poly_square", s, ns_poly_square_kernel<PER>, grid, block, 0, g);               \
    LORACT_LAUNCH("ns_poly_finish", s, ns_poly_finish_kernel<PER>, grid, block, 0, g);               \
    return LORACT_OK;
    NP_CASE(1) NP_CASE(2) NP_CASE(3) NP_CASE(4) NP_CASE(5)
#undef NP_CASE
    default: return LORACT_ERR_UNSUPPORTED;
  }
}

// ---------------------------------------------------------------------------------------------
// Newton-Schulz finish: Q = Q1 + C with C = Q1 (-E/2) (computed by the bf16 matrix-core product
// of the sketch kernel from the bf16 copy of Q1; the correction is O(||E||) small, so bf16 inputs
// cost nothing at the accuracy required).  Runs only when *flag != 0.
__global__ __launch_bounds__(256) void ns_finalize_kernel(const float* Q1, const float* C,
                                                          int64_t m, int kp, int l, void* Q,
                                                          int q_ek, bf16_t* Qb,
                                                          const int32_t* flag) {
  const int mode = *flag;            // 0: the second factorisation ran; 1: Q = Q1 + C; 2: Q = Q1
  if (mode == 0) return;
  const bool add_c = mode == 1;
  const int c4 = kp >> 2;
  const int64_t total = m * c4;
  const bool vec_ok = basis_vec_ok(Q, Qb, l);
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < total; e += (int64_t)gridDim.x * 256) {
    const int64_t r = e / c4;
    const int c = (int)(e - r * c4) << 2;
    f32x4 q = *(const f32x4*)(Q1 + r * kp + c);
    if (add_c) q += *(const f32x4*)(C + r * kp + c);
    basis_store(q, r, c, l, Q, q_ek, Qb, vec_ok);
  }
}

// ---------------------------------------------------------------------------------------------
// Host-side launchers.

// gram_narrow_kernel: 16, 32 or 64 rows per wave, so that a chunk is one or two memory
// latencies long and the sum meets 256 chunks at most.
static int gram_narrow_rows(int64_t m) {
  const int64_t rows = m <= 4096 ? 64 : (m <= 16384 ? 128 : 256);
  return (int)std::max<int64_t>(rows, ceil_div64(ceil_div64(m, 256), 64) * 64);
}
static inline int gram_narrow_tiles(int kp) { return (kp / 16) * (kp / 16 + 1) / 2; }
// Solving workgroups of round 1 that also form the Gram matrix of their result, 64 rows each; 0: not they (too many columns, or
// more rows than 255 of them take with half of their waves).
static int solve_gram_chunks(int64_t m, int kp) {
  const int64_t n = ceil_div64(m, SOLVE_GRAM_ROWS);
  return kp <= 16 * SOLVE_GRAM_MAX && n <= 255 ? (int)n : 0;
}
// Shares of ||E||_F^2 that the Gram reduction leaves, at most NS_E2_MAX (320 columns).
#define NS_E2_MAX (64 * 15)
static int gram_e2_count(int64_t m, int kp) {
  const int nblk = (kp / 16 + 3) / 4;                    // (blocks of gram_plan)
  return gram_is_narrow(kp) || gram_is_short(m, kp) ? 4 * gram_narrow_tiles(kp) : 64 * (nblk * (nblk + 1) / 2);
}
// (plan: gram_plan of the same m and kp, worked out once a call where gram_is_planned)
static size_t gram_partial_bytes(int64_t m, int kp, const GramPlan& plan) {
  if (gram_is_narrow(kp)) {
    const int64_t chunks = std::max<int64_t>(solve_gram_chunks(m, kp), ceil_div64(m, gram_narrow_rows(m)));
    return (size_t)chunks * gram_narrow_tiles(kp) * 256 * sizeof(double);
  }
  if (gram_is_short(m, kp))
    return (size_t)ceil_div64(m, gram_short_rows(m, kp)) * gram_narrow_tiles(kp) * 256 * sizeof(double);
  return (size_t)plan.part_tiles * 256 * sizeof(double);
}

// Sum of `chunks` sets of lower 16 x 16 tiles.
static int launch_gram_tiles_reduce(hipStream_t s, const double* part, int chunks, int kp, int k, double* G, double* G_copy,
                                    bf16_t* ns_T, double* ns_e2, int32_t* clear_word) {
  const int tiles = gram_narrow_tiles(kp);
  if (gram_is_narrow(kp))
    LORACT_LAUNCH("gram_reduce", s, gram_tiles_reduce_kernel<16>, dim3(4, tiles), dim3(64 * 16), 0, part, chunks, tiles, kp, k, G,
                  G_copy, ns_T, ns_e2, clear_word);
  else
    LORACT_LAUNCH("gram_reduce", s, gram_tiles_reduce_kernel<8>, dim3(4, tiles), dim3(64 * 8), 0, part, chunks, tiles, kp, k, G,
                  G_copy, ns_T, ns_e2, clear_word);
  return LORACT_OK;
}
// Y: m x kp.  g: gram_plan above 64 columns.  ns_e2 needs gram_e2_count(kp) doubles.  mirror: with ns_e2, the whole symmetric G.
static int launch_gram_mfma(hipStream_t s, const float* Y, int64_t m, int kp, int k, const GramPlan& g,
                            double* part, double* G, double* G_copy = nullptr,
                            bf16_t* ns_T = nullptr, double* ns_e2 = nullptr, bool mirror = false, int32_t* clear_word = nullptr) {
  if (gram_is_narrow(kp)) {
    const int rows = gram_narrow_rows(m), chunks = (int)ceil_div64(m, rows);
    switch (kp / 16) {
#define GN_CASE(N) \
  case N: LORACT_LAUNCH("gram", s, gram_narrow_kernel<N>, dim3(chunks), dim3(256), 0, Y, m, rows, part); break;
      GN_CASE(1) GN_CASE(2) GN_CASE(3) GN_CASE(4)
#undef GN_CASE
      default: return LORACT_ERR_UNSUPPORTED;
    }
    return launch_gram_tiles_reduce(s, part, chunks, kp, k, G, G_copy, ns_T, ns_e2, clear_word);
  }
  if (gram_is_short(m, kp)) {
    const int rows = gram_short_rows(m, kp), chunks = (int)ceil_div64(m, rows), waves = chunks * gram_short_blocks(kp);
    LORACT_LAUNCH("gram", s, gram_short_kernel, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, Y, m, kp, rows, chunks, part);
    return launch_gram_tiles_reduce(s, part, chunks, kp, k, G, G_copy, ns_T, ns_e2, clear_word);
  }
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)gram_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)GRAM_LDS_BYTES);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(Gram LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("gram", s, gram_mfma_kernel, dim3((unsigned)(g.slices * g.wgs)), dim3(64 * GRAM_WAVES), GRAM_LDS_BYTES, Y, g, part);
  LORACT_LAUNCH("gram_reduce", s, gram_reduce_kernel, dim3(64, (unsigned)g.units), dim3(64 * GRAM_LANES), 0, (const double*)part, g, k,
                G, G_copy, ns_T, ns_e2, mirror ? 1 : 0, clear_word);
  return LORACT_OK;
}

static size_t chol_lds_bytes(int kp) {
  const int ptld = kp > OF_NB ? kp - OF_NB : 2;
  return sizeof(double) * ((size_t)2 * kp + 8 + (size_t)OF_NB * ptld);
}

// Breakdown level of the unshifted first-round attempt: 16 k u (pivots below it are within a
// couple of digits of the rounding noise of the factorisation).
static inline double chol_unshifted_thresh(int k) { return 16.0 * (double)k * 1.1102230246251565e-16; }

// Clamping level of round 2 (see chol.h): columns of Q1 are stored in float32.
static inline double chol_clamp_tol(int k) {
  return ((double)k * 5.9604644775390625e-08) * ((double)k * 5.9604644775390625e-08);
}

static int launch_chol_reg_272(hipStream_t s, dim3 grid, const CholArgs& a, const char* name) {
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)chol_reg_kernel<17>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)chol_reg_lds_bytes(272));
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(factorisation LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH(name, s, chol_reg_kernel<17>, grid, dim3(CR_THREADS), chol_reg_lds_bytes(272), a);
  return LORACT_OK;
}
static int launch_chol_blocked(hipStream_t s, const CholArgs& a, const char* name = "chol") {
  if (a.round == 1 && a.unshifted_thresh > 0.0 && !a.G_backup) return LORACT_ERR_INVALID_ARG;
  if (a.kp <= CR_MAX_KP && (a.round == 2 || a.unshifted_thresh > 0.0)) {
    const dim3 grid(a.round == 1 ? 1 + 8 * CR_PREFETCH_WGS : 1);
    // By what an instantiation has registers and code for.  The trailing matrix of 192 columns fits the registers, that of 256 spills 31:
    // through 16 blocks and through 12, event to event, 144 columns 35.4 and 29.7 us, 176 43.7 and 37.3, 192 50.6 and 41.9.
    // Few columns (a truncation's) are bound by the code that is fetched: through 8 blocks and through 4 or 1, 12 columns
    // 5.8 and 4.8, 32 columns 8.1 and 6.6.
    if (a.kp <= 16)
      LORACT_LAUNCH(name, s, chol_reg_kernel<1>, grid, dim3(CR_THREADS), chol_reg_lds_bytes(16), a);
    else if (a.kp <= 64)
      LORACT_LAUNCH(name, s, chol_reg_kernel<4>, grid, dim3(CR_THREADS), chol_reg_lds_bytes(64), a);
    else if (a.kp <= 128)
      LORACT_LAUNCH(name, s, chol_reg_kernel<8>, grid, dim3(CR_THREADS), chol_reg_lds_bytes(128), a);
    else if (a.kp <= 192)
      LORACT_LAUNCH(name, s, chol_reg_kernel<12>, grid, dim3(CR_THREADS), chol_reg_lds_bytes(192), a);
    else if (a.kp <= 256)
      LORACT_LAUNCH(name, s, chol_reg_kernel<16>, grid, dim3(CR_THREADS), chol_reg_lds_bytes(256), a);
    else
      LORACT_TRY(launch_chol_reg_272(s, grid, a, name));
    return LORACT_OK;
  }
  LORACT_LAUNCH(name, s, chol_blocked_kernel, dim3(1), dim3(512), chol_lds_bytes(a.kp), a);
  return LORACT_OK;
}

template <int NBM, int NJ>
static int launch_chol_trsm_fused_nj(hipStream_t s, const CholArgs& c, const TrsmArgs& g) {
  // At least 81 KB: one workgroup per CU, so that the factorising workgroup -- whose first wave is
  // the critical path of the whole launch -- never shares its CU's issue slots with solving
  // workgroups.  (On an idle card 256 workgroups at most find a CU each without it: 2048 to 32768 rows, 72 to 256 columns,
  // the same within 0.3 %.  It matters where another stream's kernels hold CUs.)
  const size_t lds = std::max<size_t>(std::max(chol_reg_lds_bytes(OF_NB * NBM), solve_lds_bytes<NJ>()),
                                      81 * 1024);
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)chol_trsm_fused_kernel<NBM, NJ>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(fused factor-and-solve LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  // one solving workgroup per CU beside the factorising one; a tall matrix gives each several strips
  const int row_waves = ceil_div64(g.m, SOLVE_GRAM_ROWS) <= 255 ? CR_THREADS / 128 : CR_THREADS / 64;
  const unsigned solvers = (unsigned)std::min<int64_t>(ceil_div64(g.m, 16 * row_waves), 255);
  LORACT_LAUNCH("chol_trsm", s, (chol_trsm_fused_kernel<NBM, NJ>), dim3(1 + solvers), dim3(CR_THREADS), lds,
                c, g, row_waves);
  return LORACT_OK;
}

// One launch per round when the register-resident factorisation applies (kp <= 256; round 1:
// unshifted first attempt); c.ready must have been cleared by an earlier kernel.
// A solving workgroup works strip by strip and a strip needs every panel, so only its first strip
// overlaps the factorisation.  With one strip of 128 rows per workgroup, up to 32640 rows, the one launch is the faster by
// the whole solve; with more, what it saves is close to what its solver, one workgroup per CU, loses against the plain one
// (whole compress of m x 512, us, one launch and two, with an earlier Gram matrix and factorisation, which both share: 8192 rows, 128 columns 93 and 100, 256 columns 183 and 214; 24576
// x 256 261 and 321; 32768 x 128 160 and 150, x 256 345 and 334; 40000 x 128 178 and 182, x 256 373 and 405; 65536 x 128
// 232 and 217, x 256 540 and 520).  Round 2 normally has nothing to factor, and there the single launch that decides
// for itself always wins.
static bool chol_trsm_fusable(const CholArgs& c, int64_t m) {
  if (c.kp > 256 || !c.ready) return false;
  if (c.round == 2) return true;
  return m <= 32768 && c.unshifted_thresh > 0.0 && c.G_backup;
}
static int launch_chol_trsm_fused(hipStream_t s, const CholArgs& c, const TrsmArgs& g) {
  switch (c.kp / 16) {
// (registers, slots to look at and code for blocks in steps of four)
#define CF_CASE(N) case N: return launch_chol_trsm_fused_nj<(N + 3) / 4 * 4, N>(s, c, g);
    CF_CASE(1) CF_CASE(2) CF_CASE(3) CF_CASE(4) CF_CASE(5) CF_CASE(6) CF_CASE(7) CF_CASE(8)
    CF_CASE(9) CF_CASE(10) CF_CASE(11) CF_CASE(12) CF_CASE(13) CF_CASE(14) CF_CASE(15) CF_CASE(16)
#undef CF_CASE
    default: return LORACT_ERR_UNSUPPORTED;
  }
}

static int launch_trsm_apply(hipStream_t s, const TrsmArgs& g) {
  switch (g.kp / 16) {
#define TRSM_CASE(N) case N: return launch_trsm_nj<N>(s, g);
    TRSM_CASE(1) TRSM_CASE(2) TRSM_CASE(3) TRSM_CASE(4) TRSM_CASE(5) TRSM_CASE(6) TRSM_CASE(7)
    TRSM_CASE(8) TRSM_CASE(9) TRSM_CASE(10) TRSM_CASE(11) TRSM_CASE(12) TRSM_CASE(13)
    TRSM_CASE(14) TRSM_CASE(15) TRSM_CASE(16) TRSM_CASE(17) TRSM_CASE(18) TRSM_CASE(19)
    TRSM_CASE(20)
#undef TRSM_CASE
    default: return LORACT_ERR_UNSUPPORTED;
  }
}
