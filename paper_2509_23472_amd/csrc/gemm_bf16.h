// General bf16 x bf16 -> fp32 matrix product on the gfx950 matrix cores, for operands that the
// streaming kernels of stream_bf16.h do not take (rows that are not 16-byte aligned, sizes that are
// no multiples of their tiles).
//
//   C[i][j] = sum_kk opA(i, kk) * opB(j, kk),   0 <= i < M, 0 <= j < N, 0 <= kk < K
//
// Each operand is addressed either "K-contiguous" (element (i, kk) at P[row(i) * ld + kk],
// i.e. a row-major M x K matrix, with an optional row indirection for B) or "K-strided"
// (element (i, kk) at P[kk * ld + i], i.e. the transpose of a row-major K x M matrix).
// This covers the sketch Y = X X_S^T (both K-contiguous, B rows gathered through the sample
// indices), the projection V = U^T X (both K-strided, long reduction over the tokens, split
// across workgroups) and the reconstruction Xhat = U V (A K-contiguous, B K-strided).
//
// What bounds it: like the streaming kernels, the bytes in flight per CU; their asynchronous copies
// need aligned pieces, so here the slabs (64 of K) pass through registers: 16-byte loads at whatever
// alignment the rows have (2 bytes; the hardware splits a piece that straddles two lines), two slabs ahead of
// the one that is multiplied, then into a double-buffered LDS tile in the layouts of the streaming
// kernels -- K-contiguous as [row][64 K] with the 16-byte chunks permuted by the row, K-strided as it lies in
// memory, read with the transposing LDS read.  A piece that crosses the end of a row is loaded from
// the last 16 bytes of that row and shifted, which also fills in the zeros past the end of K.
// Tiles of 128 x 128 or, where a side has at most 64, 64 in that direction; four waves, two workgroups per CU
// (64 x 64 for one or two slabs, see gb_few_slabs, and for projections with few tiles, see launch_gemm_bf16).
// K is split over workgroups while the tiles alone leave CUs idle.
// Measured at 3001 x 2050, rank 100 (previous form: 64 x 64 tiles, element loads, no slab ahead, no split of the
// sketch): sketch 190 -> 21 us with its sum, projection 70 -> 22, reconstruction 31 -> 11, dY B^T
// (n_out 1030) 50 -> 17.
#pragma once
#include "common.h"

typedef unsigned int gb_u32x4 __attribute__((ext_vector_type(4)));
typedef gb_u32x4 gb_u32x4_any __attribute__((aligned(2)));     // a 16-byte piece at any element's address
typedef short gb_s16x4 __attribute__((ext_vector_type(4)));
typedef short gb_s16x8 __attribute__((ext_vector_type(8)));

struct GemmBf16Args {
  const bf16_t* A;
  int64_t lda;
  const bf16_t* B;
  int64_t ldb;
  const int32_t* b_rows;  // optional row indirection for a K-contiguous B
  void* C;                // final output (out_kind) when gridDim.z == 1
  int64_t ldc;
  float* Cpart;           // [splits][M][N] partial sums when gridDim.z > 1
  int64_t M, N, K;
  int64_t n_pad;          // columns N..n_pad-1 of C are written as zero
  int64_t k_per_split;    // multiple of 64
  int out_kind;           // EK_F32 or EK_BF16
};

#define GB_BK 64

// The 16-byte piece of a row that starts at element `at`, of a row with `len` elements: elements past
// the end come out zero.  len >= 8: one load from the last whole piece at the latest, to be shifted down
// by gb_shift; shorter rows element by element.
__device__ inline gb_u32x4 gb_load(const bf16_t* row, int64_t at, int64_t len) {
  if (len >= 8) return *(const gb_u32x4_any*)(row + (at + 8 <= len ? at : len - 8));
  union { bf16_t h[8]; gb_u32x4 v; } u;
  for (int e = 0; e < 8; ++e) u.h[e] = at + e < len ? row[at + e] : (bf16_t)0.0f;
  return u.v;
}
__device__ inline gb_u32x4 gb_shift(gb_u32x4 v, int64_t at, int64_t len) {
  if (len < 8 || at + 8 <= len) return v;
  const int64_t over = at + 8 - len;
  if (over >= 8) return (gb_u32x4){0u, 0u, 0u, 0u};
  return __builtin_bit_cast(gb_u32x4, __builtin_bit_cast(unsigned __int128, v) >> (16 * (int)over));
}

// One operand's share of a slab: R rows (or columns) of the output x 64 of K, R / 32 pieces per thread.
template <bool KC, int R>
struct GbOperand {
  static constexpr int NCH = R / 32;
  static constexpr int CPR = R / 8;                // K-strided: pieces per row of the slab
  static constexpr int BYTES = R * 128;
  const bf16_t* row[KC ? NCH : 1];
  int64_t ld, k_len, col, n_len;
  int lds_off[NCH], kr0;

  __device__ void init(const bf16_t* P, int64_t ld_, const int32_t* rows, int64_t first, int64_t count, int64_t K, int t) {
    ld = ld_;
    k_len = K;
    n_len = count;
    if (KC) {
      col = (t & 7) * 8;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int r = (t >> 3) + 32 * i;
        int64_t g = first + r;
        if (g > count - 1) g = count - 1;          // rows past the end are never stored
        row[i] = P + (rows ? (int64_t)rows[g] : g) * ld;
        lds_off[i] = r * 128 + (((t & 7) ^ (r & 7)) << 4);
      }
    } else {
      const int c = t % CPR;
      kr0 = t / CPR;
      col = first + c * 8;
      row[0] = P;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int kr = kr0 + (256 / CPR) * i;
        lds_off[i] = kr * (R * 2) + ((c ^ (2 * (kr & 3))) << 4);
      }
    }
  }
  // few: the second half of a K-strided slab is left out where it lies past K (uniform; put() and the products too)
  __device__ void load(gb_u32x4* v, int64_t k0, bool few) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      if (KC) {
        v[i] = gb_load(row[i], k0 + col, k_len);
      } else {
        int64_t k = k0 + kr0 + (256 / CPR) * i;
        if (few && i > 0 && k0 + (256 / CPR) * i >= k_len) continue;
        if (k > k_len - 1) k = k_len - 1;
        v[i] = gb_load(row[0] + k * ld, col < n_len ? col : n_len, n_len);
      }
    }
  }
  // `edge`: the slab or the tile touches the end of the matrix (uniform)
  __device__ void put(const gb_u32x4* v, unsigned char* lds, int64_t k0, bool edge, bool few) const {
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      if (!KC && few && i > 0 && k0 + (256 / CPR) * i >= k_len) continue;
      gb_u32x4 w = v[i];
      if (edge) {
        if (KC) {
          w = gb_shift(w, k0 + col, k_len);
        } else {
          w = gb_shift(w, col < n_len ? col : n_len, n_len);
          if (k0 + kr0 + (256 / CPR) * i >= k_len) w = (gb_u32x4){0u, 0u, 0u, 0u};
        }
      }
      *(gb_u32x4*)(lds + lds_off[i]) = w;
    }
  }
  // fragment address of a 32-wide group that starts at row (or column) `base` of the tile
  __device__ static int frag_off(int base, int lane) {
    if (KC) return (base + (lane & 31)) * 128;
    const int s16 = lane & 15, c = base + 16 * ((lane >> 4) & 1) + 4 * (s16 & 3);
    return (8 * (lane >> 5) + (s16 >> 2)) * (R * 2) + (((c >> 3) ^ (2 * (s16 >> 2))) << 4) + (c & 7) * 2;
  }
  __device__ static bf16x8 frag(const unsigned char* lds, int off, int ks, int lane) {
    if (KC) return *(const bf16x8*)(lds + off + (((2 * ks + (lane >> 5)) ^ (lane & 7)) << 4));
    typedef __attribute__((address_space(3))) gb_s16x4* lds_ptr;
    const gb_s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lds + off + 16 * ks * (R * 2)));
    const gb_s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(lds + off + (16 * ks + 4) * (R * 2)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// BM x BN tile, four waves of BM/2 x BN/2.  FEW: K is one or two slabs, which are all fetched at the start (0: any
// number, two slabs ahead); 16-wide steps past K are left out.  TURN: bf16 output of a single split, turned through LDS
// and stored as 16-byte pieces (the products are formed transposed for it, so that a lane holds four
// consecutive columns).
template <bool AKC, bool BKC, int BM, int BN, bool TURN, int FEW = 0>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(GemmBf16Args g) {
  constexpr int MT = BM / 64, NT = BN / 64;
  typedef GbOperand<AKC, BM> OpA;
  typedef GbOperand<BKC, BN> OpB;
  constexpr int STAGE = OpA::BYTES + OpB::BYTES;
  constexpr int LDC = BN + 8;                      // elements per row of the output staging tile
  constexpr int STAGES = FEW == 1 ? 1 : 2;
  constexpr int LDS = TURN && BM * LDC * 2 > STAGES * STAGE ? BM * LDC * 2 : STAGES * STAGE;
  __shared__ __attribute__((aligned(16))) unsigned char smem[LDS];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t row0 = (int64_t)blockIdx.x * BM, col0 = (int64_t)blockIdx.y * BN;
  const int64_t kbeg = (int64_t)blockIdx.z * g.k_per_split;
  const int64_t kend = (kbeg + g.k_per_split < g.K) ? kbeg + g.k_per_split : g.K;
  const int nslab = (int)((kend - kbeg + GB_BK - 1) / GB_BK);
  OpA oa;
  OpB ob;
  oa.init(g.A, g.lda, nullptr, row0, g.M, g.K, t);
  ob.init(g.B, g.ldb, g.b_rows, col0, g.N, g.K, t);
  const bool tile_edge = (!AKC && row0 + BM > g.M) || (!BKC && col0 + BN > g.N);
  int a_off[MT], b_off[NT];
#pragma unroll
  for (int i = 0; i < MT; ++i) a_off[i] = OpA::frag_off(wm * (BM / 2) + 32 * i, lane);
#pragma unroll
  for (int j = 0; j < NT; ++j) b_off[j] = OpA::BYTES + OpB::frag_off(wn * (BN / 2) + 32 * j, lane);

  f32x16 acc[MT][NT];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  gb_u32x4 va[2][OpA::NCH], vb[2][OpB::NCH];
  auto fetch = [&](int p, int s) {                 // slabs past the last one repeat it and are not multiplied
    const int64_t k0 = kbeg + (int64_t)(s < nslab ? s : nslab - 1) * GB_BK;
    oa.load(va[p], k0, FEW > 0);
    ob.load(vb[p], k0, FEW > 0);
  };
  auto step = [&](int p, int s) {
    const int64_t k0 = kbeg + (int64_t)s * GB_BK;
    unsigned char* st = smem + p * STAGE;
    const bool edge = tile_edge || k0 + GB_BK > g.K;
    oa.put(va[p], st, k0, edge, FEW > 0);
    ob.put(vb[p], st + OpA::BYTES, k0, edge, FEW > 0);
    sb_barrier_lds();                              // (the half of slab s - 2 was left before slab s - 1's barrier)
    if (FEW == 0) fetch(p, s + 2);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (FEW && k0 + 16 * ks >= g.K) break;
      bf16x8 a[MT], b[NT];
#pragma unroll
      for (int i = 0; i < MT; ++i) a[i] = OpA::frag(st, a_off[i], ks, lane);
#pragma unroll
      for (int j = 0; j < NT; ++j) b[j] = OpB::frag(st, b_off[j], ks, lane);
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
          acc[i][j] = TURN ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[j], a[i], acc[i][j], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  };
  if (FEW > 0) {
    fetch(0, 0);
    if (FEW == 2) fetch(1, 1);
    step(0, 0);
    if (FEW == 2) step(1, 1);
  } else if (nslab > 0) {
    fetch(0, 0);
    fetch(1, 1);
    int s = 0;
    for (; s + 2 <= nslab; s += 2) { step(0, s); step(1, s + 1); }
    if (s < nslab) step(0, s);
  }

  // accumulator register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of its tile
  if (TURN) {
    bf16_t* const cs = (bf16_t*)smem;
    __syncthreads();                               // the last slab has been read
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          bf16x4 o;
#pragma unroll
          for (int u = 0; u < 4; ++u) o[u] = (bf16_t)acc[i][j][4 * q + u];
          *(bf16x4*)(cs + (wm * (BM / 2) + 32 * i + (lane & 31)) * LDC + wn * (BN / 2) + 32 * j + 8 * q + 4 * (lane >> 5)) = o;
        }
    __syncthreads();
#pragma unroll 4
    for (int e = t; e < BM * (BN / 8); e += 256) {
      const int r = e / (BN / 8), c = (e % (BN / 8)) * 8;
      const int64_t row = row0 + r, col = col0 + c;
      if (row >= g.M || col >= g.N) continue;
      bf16_t* dst = (bf16_t*)g.C + row * g.ldc + col;
      const bf16_t* src = cs + r * LDC + c;
      if (col + 8 <= g.N) *(gb_u32x4_any*)dst = *(const gb_u32x4*)src;
      else
        for (int u = 0; col + u < g.N; ++u) dst[u] = src[u];
    }
    return;
  }
  const bool split = gridDim.z > 1;
#pragma unroll
  for (int j = 0; j < NT; ++j) {
    const int64_t col = col0 + wn * (BN / 2) + 32 * j + (lane & 31);
    if (col >= (split ? g.N : (g.N > g.n_pad ? g.N : g.n_pad))) continue;
    const bool live = col < g.N;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int64_t row = row0 + wm * (BM / 2) + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (row >= g.M) continue;
        const float v = live ? acc[i][j][r] : 0.0f;
        if (split) g.Cpart[((int64_t)blockIdx.z * g.M + row) * g.N + col] = v;
        else if (g.out_kind == EK_F32) ((float*)g.C)[row * g.ldc + col] = v;
        else ((bf16_t*)g.C)[row * g.ldc + col] = (bf16_t)v;
      }
  }
}

// out[row][col] = sum over splits (ascending, eight loads in flight) of part[s][row][col], converted to
// out_kind; columns N .. n_pad-1 are written as zero.
__global__ __launch_bounds__(256) void reduce_partials_f32(const float* part, int splits, int64_t M, int64_t N,
                                                           int64_t n_pad, void* out, int64_t ldc, int out_kind) {
  const int64_t total = M * N, width = N > n_pad ? N : n_pad;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < M * width; i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = i / width, col = i - row * width;
    const float* src = part + row * N + (col < N ? col : N - 1);
    float s = 0.0f;
    for (int z = 0; z < splits; z += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = src[(int64_t)(z + u < splits ? z + u : splits - 1) * total];
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (z + u < splits) s += v[u];
    }
    if (col >= N) s = 0.0f;
    if (out_kind == EK_F32) ((float*)out)[row * ldc + col] = s;
    else ((bf16_t*)out)[row * ldc + col] = (bf16_t)s;
  }
}

static inline int gb_tile_for(int64_t extent) { return extent <= 64 ? 64 : 128; }
// Slabs of a product with one or two of them (reconstructions of low rank), which are all load latency and stores:
// 64 x 64 tiles, of which a CU holds five to ten, beat 128 x 128 tiles, of which it holds two.  float32 output
// 12608 x 768 of rank 32 20.5 -> 11.1 us, 16384 x 3072 of rank 64 57 -> 36, of rank 96 68 -> 54, of rank 128 66 -> 62;
// bf16 output 8192 x 4097 of rank 12 30 -> 18, 1000000 x 33 of rank 33 90 -> 40, but with both sides long the narrow
// row segments cost as much from rank 33 on (65536 x 4095: rank 12 232 -> 208, rank 33 228 -> 233, rank 60 234 -> 249).
static inline int gb_few_slabs(int64_t M, int64_t N, int64_t K, int out_kind) {
  if (N > 64 * 65535ll || M >= 1ll << 30) return 0;  // (the grid's second dimension; 2^32 threads in its first)
  if (out_kind == EK_F32) return K <= GB_BK ? 1 : (K <= 2 * GB_BK ? 2 : 0);
  return K <= GB_BK / 2 || (K <= GB_BK && std::min(M, N) <= 64) ? 1 : 0;
}
// K splits: two workgroups per CU with at least 256 of K each, at most 64.  Where that leaves fewer than 128
// workgroups, slabs of 64 for as many, if there are six: a workgroup that walks 384 of K takes longer than the launch
// that sums the parts (compress 1000 x 768 of rank 33 59.6 -> 55.2 us, 500 x 75 of rank 5 50.3 -> 43.3), one that walks
// 256 does not (128 x 300 of rank 5 45 -> 49), and splitting finer everywhere costs the large ones the sum (30000 x 300
// of rank 100 151 -> 163).
static inline int gemm_bf16_splits(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = ceil_div64(M, gb_tile_for(M)) * ceil_div64(N, gb_tile_for(N));
  const int64_t s = std::max(std::min<int64_t>(512 / tiles, K / 256),
                             K >= 6 * GB_BK ? std::min<int64_t>(128 / tiles, K / GB_BK) : 1);
  return (int)std::max<int64_t>(1, std::min<int64_t>(s, 64));
}
static inline size_t gemm_bf16_part_bytes(int64_t M, int64_t N, int64_t K) {
  const int s = gemm_bf16_splits(M, N, K);
  return s > 1 ? (size_t)s * M * N * 4 : 0;
}

// Enqueue C = opA * opB^T.  Cpart: room for max_splits * M * N floats (null = no splits; max_splits 0: as many
// as gemm_bf16_part_bytes allows for).
static int launch_gemm_bf16(const char* name, hipStream_t stream, const bf16_t* A, int64_t lda,
                            int a_kc, const bf16_t* B, int64_t ldb, int b_kc,
                            const int32_t* b_rows, int64_t M, int64_t N, int64_t K, void* C,
                            int64_t ldc, int out_kind, float* Cpart, int max_splits = 0, int64_t n_pad = 0) {
  if (M <= 0 || N <= 0 || K <= 0) return LORACT_OK;
  GemmBf16Args g;
  g.n_pad = n_pad;
  g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.b_rows = b_rows;
  g.C = C; g.ldc = ldc; g.Cpart = Cpart; g.M = M; g.N = N; g.K = K;
  g.out_kind = out_kind;
  int splits = Cpart ? gemm_bf16_splits(M, N, K) : 1;
  if (max_splits > 0) splits = std::min(splits, max_splits);
  g.k_per_split = ceil_div64(ceil_div64(K, splits), GB_BK) * GB_BK;
  splits = (int)ceil_div64(K, g.k_per_split);
  const int few = a_kc && !b_kc && splits == 1 ? gb_few_slabs(M, N, K, out_kind) : 0;
  // the projection with fewer workgroups than CUs: 64 x 64 tiles, four times as many (compress 300 x 4096 of rank 100
  // 81 -> 70 us, 788 x 768 of rank 20 50 -> 46; with 2000 x 4096 of rank 250, 64 tiles of 128 x 128, 201 -> 196)
  const bool thin = !a_kc && !b_kc && ceil_div64(M, gb_tile_for(M)) * ceil_div64(N, 128) * splits < 256 &&
                    N <= 64 * 65535ll;
  const int bm = few || thin ? 64 : (!a_kc && !b_kc) ? gb_tile_for(M) : 128;
  const int bn = few || thin ? 64 : (a_kc && b_kc) ? gb_tile_for(N) : 128;
  dim3 grid((unsigned)ceil_div64(M, bm), (unsigned)ceil_div64(std::max(N, n_pad), bn), (unsigned)splits);
  if (grid.y > 65535 || grid.z > 65535) return LORACT_ERR_UNSUPPORTED;
  {
    KernelScope scope(name, stream);
#define GB_LAUNCH(...) hipLaunchKernelGGL((gemm_bf16_kernel<__VA_ARGS__>), grid, dim3(256), 0, stream, g)
    if (a_kc && b_kc) {
      if (bn == 64) GB_LAUNCH(true, true, 128, 64, false);
      else GB_LAUNCH(true, true, 128, 128, false);
    } else if (!a_kc && !b_kc) {
      if (thin) GB_LAUNCH(false, false, 64, 64, false);
      else if (bm == 64) GB_LAUNCH(false, false, 64, 128, false);
      else GB_LAUNCH(false, false, 128, 128, false);
    } else if (few) {
      if (out_kind == EK_BF16) GB_LAUNCH(true, false, 64, 64, true, 1);
      else if (few == 1) GB_LAUNCH(true, false, 64, 64, false, 1);
      else GB_LAUNCH(true, false, 64, 64, false, 2);
    } else if (a_kc) {
      if (splits == 1 && out_kind == EK_BF16) GB_LAUNCH(true, false, 128, 128, true);
      else GB_LAUNCH(true, false, 128, 128, false);
    } else {
      return LORACT_ERR_INVALID_ARG;
    }
#undef GB_LAUNCH
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, name);
  if (splits > 1) {
    const int64_t total = M * std::max(N, n_pad);
    int blocks = (int)(ceil_div64(total, 256) < 2048 ? ceil_div64(total, 256) : 2048);
    LORACT_LAUNCH("reduce_partials_f32", stream, reduce_partials_f32, dim3(blocks), dim3(256), 0,
                  (const float*)Cpart, splits, M, N, n_pad, C, ldc, out_kind);
  }
  return LORACT_OK;
}
