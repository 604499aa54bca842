// General matrix product with float64 accumulation on the float64 matrix cores
// (v_mfma_f64_16x16x4_f64), for the float32 input path, for float32 factors, for the truncation of
// an l-column factor, and for the thin contractions of the LoRA gradient.
//
//   C[i][j] = alpha * sum_kk opA(i, kk) * opB(j, kk)
//
// Operand addressing as in gemm_bf16.h (K-contiguous with optional row indirection for B, or
// K-strided); operand types and addressing are compiled in, the output type is chosen at run time.
//
// What bounds it.  The sizes met here are small (K from 16 to a few thousand, a side of 16 to 320),
// so a launch is one or two memory latencies plus the matrix instructions of its longest wave; only
// the float32 reconstruction is a bandwidth-sized write.  Hence: operands go from global memory
// straight to registers (no LDS, no barrier in the loop), 16 values of K per trip, several trips ahead; the
// contraction index is dealt to the lane groups in runs of four (group q takes 4 q .. 4 q + 3, the
// same way for both operands), so that a K-contiguous operand is one 16-byte load per lane and
// trip; and the wave layout follows the output:
//   T64  64 x 64 per workgroup, 2 x 2 waves of 32 x 32: large outputs, operands re-read least
//   T32  32 x 32 per workgroup, the four waves take a quarter of K each and add up through LDS in
//        wave order: outputs too small to fill the CUs with T64, four times shorter chains
//   T16  16 x 16 likewise: a side of at most 16 (rank 16, LoRA ranks), where wider tiles are padding; with
//        sixteen waves where K would be split two to four ways, which then needs no partial tiles and no
//        launch that sums them (launches are what bounds a 1024 x 256 rank-16 float32 step:
//        18 -> 15 of them with the float32 copy of Q made here too, kernels together 65.5 -> 62.5 us)
// Splitting K over workgroups (float64 partial tiles, summed in a fixed order by
// reduce_partials_f64) is what is left when even those tiles are too few.
// Measured against the previous form (64 x 64 tiles staged through LDS, vector-unit FMAs): the ten
// products of a 1024 x 256 rank-16 float32 site 136 -> 43 us (T16 and T32), the float32
// reconstruction 12608 x 768 of rank 32 43 -> 27 us (9 us of matrix instructions at the 66 to 73 TFLOP/s
// that a loop of nothing else takes them to), B B^T of a 264 x 11008 factor 134 -> 39 us, Q W 8192 x 256 x 264 102 -> 30 us,
// W^T B 256 x 11008 x 264 71 -> 41 us.
#pragma once
#include "common.h"

struct GemmF64Args {
  const void* A;
  int64_t lda;
  const void* B;
  int64_t ldb;
  const int32_t* b_rows;
  void* C;
  int64_t ldc;
  float* C32;            // optional float32 copy of C, same pitch (unsplit K only)
  double* Cpart;
  int64_t M, N, K;
  int64_t Mv, Nv;        // operand rows that exist: C is zero from there up to M, N
  int64_t k_per_split;   // multiple of 16
  double alpha;
  int out_ek;
  int rows_f32;          // C is float32, K unsplit and no C32: whole wave tiles leave as rows
};

__device__ inline f64x4 gd_mfma(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

// Widening that is exact: bf16 goes through float32.
template <int EK, typename T>
__device__ inline double gd_wide(T v) {
  if (EK == EK_BF16) return (double)(float)v;
  return (double)v;
}

template <int EK> struct gd_elem;
template <> struct gd_elem<EK_F32> { typedef float t; };
template <> struct gd_elem<EK_F64> { typedef double t; };
template <> struct gd_elem<EK_BF16> { typedef bf16_t t; };

// Four consecutive values of K of one operand row, as they come from memory.
template <int EK> struct GdFrag { typename gd_elem<EK>::t v[4]; };

// `base`: first element of the operand row (K-contiguous) or column (K-strided); kk = first of the
// four values, all of them inside the matrix.
template <int EK, bool KC>
__device__ inline void gd_fetch(GdFrag<EK>& f, const typename gd_elem<EK>::t* base, int64_t ld, int64_t kk) {
  typedef typename gd_elem<EK>::t T;
  if (KC) {
    typedef T vec __attribute__((ext_vector_type(4), aligned(sizeof(T))));
    const vec w = *(const vec*)(base + kk);
#pragma unroll
    for (int s = 0; s < 4; ++s) f.v[s] = w[s];
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) f.v[s] = base[(kk + s) * ld];
  }
}

// AEK / AKC, BEK / BKC: element kind and addressing of the operands.  MT x NT: 16 x 16 tiles per
// wave.  WK: 1 = 2 x 2 waves side by side, 4 or 16 = that many waves split K.
template <int AEK, bool AKC, int BEK, bool BKC, int MT, int NT, int WK>
__global__ __launch_bounds__(WK == 16 ? 1024 : 256) void gemm_f64_kernel(GemmF64Args g) {
  // trips in flight: one is 4 MT NT matrix instructions (sixteen waves share a CU and have few trips each)
  constexpr int D = WK == 16 ? 4 : (MT * NT == 1 ? 6 : 3);
  constexpr int BM = WK == 1 ? 32 * MT : 16 * MT, BN = WK == 1 ? 32 * NT : 16 * NT;
  __shared__ double red[WK == 1 ? 1 : WK * MT * NT * 256];
  __shared__ __attribute__((aligned(16))) float turn[WK == 1 ? 4 : 1][WK == 1 ? 16 * MT * (16 * NT + 4) : 1];
  typedef typename gd_elem<AEK>::t TA;
  typedef typename gd_elem<BEK>::t TB;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int lc = lane & 15, lq = lane >> 4;
  const int64_t row0 = (int64_t)blockIdx.x * BM + (WK == 1 ? (wave >> 1) * 16 * MT : 0);
  const int64_t col0 = (int64_t)blockIdx.y * BN + (WK == 1 ? (wave & 1) * 16 * NT : 0);
  int64_t kbeg = (int64_t)blockIdx.z * g.k_per_split;
  int64_t kend = (kbeg + g.k_per_split < g.K) ? kbeg + g.k_per_split : g.K;
  if (WK > 1) {
    const int64_t per = (kend - kbeg + 16 * WK - 1) / (16 * WK) * 16;   // a quarter or a sixteenth, in whole trips
    kbeg += wave * per;
    if (kbeg > kend) kbeg = kend;
    if (kbeg + per < kend) kend = kbeg + per;
  }
  // rows and columns past the end repeat the last one; they are never stored
  const TA* a_base[MT];
  const TB* b_base[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    int64_t r = row0 + 16 * i + lc;
    if (r > g.Mv - 1) r = g.Mv - 1;
    a_base[i] = (const TA*)g.A + (AKC ? r * g.lda : r);
  }
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    int64_t r = col0 + 16 * j + lc;
    if (r > g.Nv - 1) r = g.Nv - 1;
    if (BKC && g.b_rows) r = g.b_rows[r];
    b_base[j] = (const TB*)g.B + (BKC ? r * g.ldb : r);
  }
  f64x4 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j) acc[i][j] = (f64x4){0.0, 0.0, 0.0, 0.0};

  const int ntrip = (int)((kend - kbeg) >> 4);
  GdFrag<AEK> fa[D][MT];
  GdFrag<BEK> fb[D][NT];
  auto load_trip = [&](int p, int trip) {
    const int64_t kk = kbeg + 16 * (int64_t)trip + 4 * lq;
#pragma unroll
    for (int i = 0; i < MT; ++i) gd_fetch<AEK, AKC>(fa[p][i], a_base[i], g.lda, kk);
#pragma unroll
    for (int j = 0; j < NT; ++j) gd_fetch<BEK, BKC>(fb[p][j], b_base[j], g.ldb, kk);
  };
  auto mac_trip = [&](int p) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = gd_mfma(gd_wide<AEK>(fa[p][i].v[s]), gd_wide<BEK>(fb[p][j].v[s]), acc[i][j]);
  };
  if (ntrip > 0) {
    // ring of D trips, D - 1 ahead; loads past the last trip repeat it and are not multiplied
#pragma unroll
    for (int p = 0; p < D - 1; ++p) load_trip(p, p < ntrip ? p : ntrip - 1);
    for (int t0 = 0; t0 < ntrip; t0 += D) {
#pragma unroll
      for (int p = 0; p < D; ++p) {
        const int nxt = t0 + p + D - 1;
        load_trip((p + D - 1) % D, nxt < ntrip ? nxt : ntrip - 1);
        if (t0 + p < ntrip) mac_trip(p);
      }
    }
  }
  if (kbeg + 16 * (int64_t)ntrip < kend) {
    // fewer than 16 values of K are left: element by element, what lies past the end is zero
    const int64_t k0 = kbeg + 16 * (int64_t)ntrip + 4 * lq;
    double a[MT][4], b[NT][4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool on = k0 + s < kend;
      const int64_t kk = on ? k0 + s : kend - 1;
#pragma unroll
      for (int i = 0; i < MT; ++i) {
        const double v = gd_wide<AEK>(a_base[i][AKC ? kk : kk * g.lda]);
        a[i][s] = on ? v : 0.0;
      }
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        const double v = gd_wide<BEK>(b_base[j][BKC ? kk : kk * g.ldb]);
        b[j][s] = on ? v : 0.0;
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = gd_mfma(a[i][s], b[j][s], acc[i][j]);
  }

  const bool split = gridDim.z > 1;
  auto store = [&](int64_t row, int64_t col, double v) {
    if (row >= g.M || col >= g.N) return;
    if (row >= g.Mv || col >= g.Nv) v = 0.0;
    if (split) g.Cpart[((int64_t)blockIdx.z * g.M + row) * g.N + col] = v;
    else {
      store_f64(g.C, row * g.ldc + col, g.out_ek, g.alpha * v);
      if (g.C32) g.C32[row * g.ldc + col] = (float)(g.alpha * v);
    }
  };
  // accumulator register r of lane l: row 4 r + l / 16, column l % 16 of its tile
  if (WK == 1 && g.rows_f32 && row0 + 16 * MT <= g.Mv && col0 + 16 * NT <= g.Nv) {
    // A whole wave tile of float32 output leaves as whole rows, turned through LDS of the wave's own: written element by element
    // every value has its own address and bounds, which cost as much as the matrix instructions beside which no vector instruction
    // runs (12608 x 768 of rank 32 29.2 -> 23.6 us, 8192 x 2048 of rank 16 33.5 -> 25.3, 16384 x 3072 of rank 64 165 -> 147).
    constexpr int LD = 16 * NT + 4, PER_ROW = 4 * NT, ROWS = 64 / PER_ROW;     // lanes per row of 16-byte pieces, rows per store
    typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));   // (rows of C begin anywhere)
    float* const mine = turn[wave];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) mine[(16 * i + 4 * r + lq) * LD + 16 * j + lc] = (float)(g.alpha * acc[i][j][r]);
    sb_wave_sync();
    float* out = (float*)g.C + (row0 + lane / PER_ROW) * g.ldc + col0 + 4 * (lane % PER_ROW);
    const float* from = mine + (lane / PER_ROW) * LD + 4 * (lane % PER_ROW);
#pragma unroll
    for (int q = 0; q < 16 * MT / ROWS; ++q) {
      *(f32x4_any*)out = *(const f32x4*)(from + q * ROWS * LD);
      out += ROWS * g.ldc;
    }
    return;
  }
  if (WK == 1) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) store(row0 + 16 * i + 4 * r + lq, col0 + 16 * j + lc, acc[i][j][r]);
  } else {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) red[(((wave * MT + i) * NT + j) * 4 + r) * 64 + lane] = acc[i][j][r];
    __syncthreads();
    constexpr int SLICE = MT * NT * 256;
    if (WK == 16 && t >= 256) return;
#pragma unroll
    for (int e = 0; e < MT * NT; ++e) {
      const int at = e * 256 + t;                  // tile e, register t / 64, lane t % 64
      double v = red[at];
#pragma unroll
      for (int w = 1; w < WK; ++w) v += red[w * SLICE + at];
      store(row0 + 16 * (e / NT) + 4 * wave + lq, col0 + 16 * (e % NT) + lc, v);
    }
  }
}

// out = alpha * sum over splits (ascending), eight loads in flight.
__global__ __launch_bounds__(256) void reduce_partials_f64(const double* part, int splits,
                                                           int64_t M, int64_t N, double alpha,
                                                           void* out, int64_t ldc, int out_ek) {
  const int64_t total = M * N;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    double s = 0.0;
    for (int z = 0; z < splits; z += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(z + u < splits ? z + u : splits - 1) * total + i];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (z + u < splits) s += v[u];
    }
    const int64_t row = i / N, col = i - row * N;
    store_f64(out, row * ldc + col, out_ek, alpha * s);
  }
}

// Tile of an M x N output: 16, 32 or 64 (see the top of the file).  64-wide tiles once they alone
// make two workgroups per CU; 16-wide ones where a side has no more.
static inline int gd_tile_for(int64_t M, int64_t N) {
  if (N > 16 * 65535) return 64;                     // (the grid's second dimension)
  if (M >= 1ll << 28) return 64;                     // (a launch has fewer than 2^32 threads in its first dimension)
  if (M <= 16 || N <= 16) return 16;
  return ceil_div64(M, 64) * ceil_div64(N, 64) >= 512 ? 64 : 32;
}
// K splits over workgroups: two workgroups per CU, at least 256 values of K each (four trips per
// wave of a WK = 4 tile), at most 32 partial tiles.
static inline int gemm_f64_splits(int64_t M, int64_t N, int64_t K) {
  const int tile = gd_tile_for(M, N);
  const int64_t tiles = ceil_div64(M, tile) * ceil_div64(N, tile);
  const int64_t s = std::min<int64_t>(std::max<int64_t>(1, 512 / tiles), K / 256);
  return (int)std::max<int64_t>(1, std::min<int64_t>(s, 32));
}
static inline size_t gemm_f64_part_bytes(int64_t M, int64_t N, int64_t K) {
  const int s = gemm_f64_splits(M, N, K);
  return s > 1 ? (size_t)s * M * N * 8 : 0;
}

template <int AEK, bool AKC, int BEK, bool BKC>
static void launch_gemm_f64_kinds(hipStream_t s, const char* name, const GemmF64Args& g, int tile, bool wk16, dim3 grid) {
  KernelScope scope(name, s);
  if (tile == 64)
    hipLaunchKernelGGL((gemm_f64_kernel<AEK, AKC, BEK, BKC, 2, 2, 1>), grid, dim3(256), 0, s, g);
  else if (tile == 32)
    hipLaunchKernelGGL((gemm_f64_kernel<AEK, AKC, BEK, BKC, 2, 2, 4>), grid, dim3(256), 0, s, g);
  else if (wk16)
    hipLaunchKernelGGL((gemm_f64_kernel<AEK, AKC, BEK, BKC, 1, 1, 16>), grid, dim3(1024), 0, s, g);
  else
    hipLaunchKernelGGL((gemm_f64_kernel<AEK, AKC, BEK, BKC, 1, 1, 4>), grid, dim3(256), 0, s, g);
}

// Enqueue C = alpha opA opB^T.  Cpart: gemm_f64_part_bytes(M, N, K) bytes of partial tiles, or null for
// a single pass over K.  C32: optional float32 copy of C (single pass only).  pad: C gets that many rows and columns of zeros more (M and N do not count them).
static int launch_gemm_f64(const char* name, hipStream_t stream, const void* A, int64_t lda,
                           int a_kc, int a_ek, const void* B, int64_t ldb, int b_kc, int b_ek,
                           const int32_t* b_rows, int64_t M, int64_t N, int64_t K, double alpha,
                           void* C, int64_t ldc, int out_ek, double* Cpart, int pad = 0, float* C32 = nullptr) {
  if (M <= 0 || N <= 0 || K <= 0) return LORACT_OK;
  GemmF64Args g;
  g.Mv = M; g.Nv = N;
  M += pad; N += pad;
  g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.b_rows = b_rows;
  g.C = C; g.ldc = ldc; g.Cpart = Cpart; g.M = M; g.N = N; g.K = K; g.alpha = alpha;
  g.out_ek = out_ek;
  g.C32 = C32;
  int splits = Cpart ? gemm_f64_splits(M, N, K) : 1;
  if (C32 && splits > 1) return LORACT_ERR_INVALID_ARG;
  const int tile = gd_tile_for(M, N);
  // (a Gram matrix, with two float64 operands, is too much for one CU's loads: 12.1 us at 1024 x 16 against 6.3 us
  // for four workgroups and their sum; U^T G 6.6 against 5.8 us, the projection 9.8 against 7.7 us, less a launch)
  const bool wk16 = tile == 16 && splits > 1 && splits <= 4 && !(a_ek == EK_F64 && b_ek == EK_F64);
  if (wk16) splits = 1;
  g.k_per_split = ceil_div64(ceil_div64(K, splits), 16) * 16;
  splits = (int)ceil_div64(K, g.k_per_split);
  dim3 grid((unsigned)ceil_div64(M, tile), (unsigned)ceil_div64(N, tile), (unsigned)splits);
  if (grid.y > 65535 || grid.z > 65535) return LORACT_ERR_UNSUPPORTED;
  if ((int64_t)grid.x * (wk16 ? 1024 : 256) >= 1ll << 32) return LORACT_ERR_UNSUPPORTED;   // (would be cut off silently)
  g.rows_f32 = out_ek == EK_F32 && splits == 1 && !C32;
  // one instantiation per pair of operand kinds and addressings that a caller uses
#define GD_CASE(AE, AK, BE, BK) \
  if (a_ek == AE && (a_kc != 0) == AK && b_ek == BE && (b_kc != 0) == BK) \
    launch_gemm_f64_kinds<AE, AK, BE, BK>(stream, name, g, tile, wk16, grid); \
  else
  GD_CASE(EK_F32, true, EK_F32, true)        // sketch, dY B^T, B B^T
  GD_CASE(EK_F32, true, EK_F64, true)        // sketch of a power round
  GD_CASE(EK_F64, true, EK_F64, true)        // B B^T of the float32 path
  GD_CASE(EK_F64, false, EK_F64, false)      // Gram matrix, W^T B
  GD_CASE(EK_F64, true, EK_F64, false)       // Q1 = Y R^-1, Q W
  GD_CASE(EK_F32, true, EK_F64, false)       // Q W
  GD_CASE(EK_F64, false, EK_F32, false)      // projection, W^T B
  GD_CASE(EK_F32, true, EK_F32, false)       // reconstruction
  GD_CASE(EK_F32, false, EK_F32, false)      // U^T G, V^T T
  GD_CASE(EK_BF16, false, EK_F32, false)     // the same with bf16 factors
  return LORACT_ERR_INVALID_ARG;
#undef GD_CASE
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, name);
  if (splits > 1) {
    const int64_t total = M * N;
    int blocks = (int)(ceil_div64(total, 256) < 2048 ? ceil_div64(total, 256) : 2048);
    LORACT_LAUNCH("reduce_partials_f64", stream, reduce_partials_f64, dim3(blocks), dim3(256), 0,
                  (const double*)Cpart, splits, M, N, alpha, C, ldc, out_ek);
  }
  return LORACT_OK;
}
