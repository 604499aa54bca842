// LoRA gradient of a compressed input on the bf16 matrix cores (Section 3.1, Eqs. 4-5):
//   dA = scale * V^T T,   T = U^T G,   G = dY B_lora^T
// dY (m x n_out) is the one large operand and is read once.
//
// Up to LoRA rank 32: lora_gt_kernel forms G and its share of T in one pass over dY, lora_tsum_kernel
// adds the shares, lora_vtt_kernel multiplies by V.  Higher ranks form G and T with the sketch and
// the projection kernels (their 64-column tiles are then in use, and B_lora no longer fits beside a
// ring of dY slabs in LDS), and so does a dY from HBM where that is the faster way (lora_one_pass).
#pragma once
#include "common.h"
#include "lora_plan.h"
#include "stream_bf16.h"

// ---------------------------------------------------------------------------------------------
// lora_gt: T shares.  Work items are (32-row tile of dY, slab of 256 columns), tile major; every
// workgroup takes an equal contiguous share and may begin or end inside a tile, since T is linear in
// G.  Slabs of dY and B_lora run through an LDS ring of asynchronous copies; each wave multiplies its
// own part of a slab's columns, so that a tile's G is spread over the waves and is added up once per
// tile (fixed order).  G then becomes the bf16 pair (hi, lo), ~16 mantissa bits, and is multiplied
// with the tile's rows of U, which came in with the tile's first slab; T stays in registers from tile
// to tile.  The ring runs on across tiles, so that dY keeps streaming behind the end of a tile.
//
// Bound by dY from HBM.  Against the launches it replaces (G with K splits and their sum, U^T G and its sum), the
// whole gradient at LoRA rank 16, called again and again: 58 -> 42 us at 20000 x 4096 with 64 columns of U, 32 -> 22 at
// 197 x 4096 with 256, 127 -> 117 at 65536 x 4096 with 256.  There the dY pass alone is slower, 120 against 86 us inside
// a step, where nothing of dY is cached, and what it saves are the passes over G (141 -> 134 us in all).
//
// LDS layout of a slab: [row][32 chunks of 16 bytes], chunk c of row r at position c ^ (r & 15), for dY
// and B_lora; U as in the projection: chunk c of row r at position c ^ 2 (r & 3), read transposed.

#define LG_ROWS 32
#define LG_BK 256
#define LG_WGS 256       // one workgroup per CU (the ring fills its LDS)
#define LG_RED_LD 36     // floats per column of the G shares
#define LG_GT_LD 40      // bf16 per column of the G pair

struct LoraGtArgs {
  const bf16_t* U;       // m x k, ld = k (multiple of 8)
  const bf16_t* dY;      // m x n_out, n_out a multiple of 64
  const bf16_t* B;       // r x n_out
  int64_t m, n_out;
  int k, r;
  int slabs;             // ceil(n_out / 256)
  int64_t items;         // row tiles * slabs
  int cq;                // chunks per LDS row of U: ceil(k / 64) * 8
  int stream_x;          // dY is too large to stay cached: copy it non-temporally
  float* part;           // [workgroups][k][RP]
};

static size_t lora_gt_lds_bytes(int rp, int stages, int cq) {
  return (size_t)stages * (LG_ROWS + rp) * 512 + (size_t)2 * LG_ROWS * cq * 16 +
         (size_t)128 * LG_RED_LD * 4 + (size_t)2 * rp * LG_GT_LD * 2;
}

// S: stages of the ring (a fifth one at rank 16, where LDS has room for it, changed nothing)
template <int RP, int S>
__global__ __launch_bounds__(512) void lora_gt_kernel(LoraGtArgs g) {
  constexpr int CW = RP / 16, KW = 8 / CW;          // waves: KW parts of a slab's columns x CW tiles of 16 G columns
  constexpr int KS = LG_BK / (32 * KW);             // K steps of 32 per wave and slab
  constexpr int A_BYTES = LG_ROWS * 512, STAGE_BYTES = A_BYTES + RP * 512;
  constexpr int NB = RP / 16;                       // B copy instructions per wave and slab (dY: 2)
  constexpr int LOADS = 2 + NB;
  extern __shared__ __attribute__((aligned(16))) unsigned char sb_smem[];
  unsigned char* const Us = sb_smem + S * STAGE_BYTES;
  const int u_bytes = LG_ROWS * g.cq * 16;
  float* const Red = (float*)(Us + 2 * u_bytes);                    // [KW][RP][LG_RED_LD]
  bf16_t* const Gt = (bf16_t*)(Red + 128 * LG_RED_LD);              // [2][RP][LG_GT_LD]

  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int kw = wave / CW, cw = wave % CW;
  const int l16 = lane & 15, grp = lane >> 4;
  const int64_t item0 = g.items * blockIdx.x / gridDim.x;
  const int total = (int)(g.items * (blockIdx.x + 1) / gridDim.x - item0);

  // Where dY may be served by the memory-side cache, a tile's slabs are taken from a starting point that
  // differs from tile to tile: with a power-of-two row pitch, workgroups that all read the same columns at the
  // same time crowd a few of its channels (8192 x 4096: 23.2 -> 19.7 us with the sum).  From HBM the plain order is
  // the faster one (65536 x 4096: 112 against 124 us).
  auto slab_at = [&](int64_t tile, int sl) {
    if (g.stream_x) return sl;
    const int pos = sl + (int)((((uint32_t)tile * 2654435761u) >> 16) % (uint32_t)g.slabs);
    return pos < g.slabs ? pos : pos - g.slabs;
  };
  // ---- copies: slab `is` of tile `it` (the it_ord-th of this workgroup), U ahead of a tile's first slab
  int64_t it = item0 / g.slabs;
  int is = (int)(item0 - it * g.slabs), it_ord = 0, issued = 0;
  auto issue = [&]() {
    const int64_t row0 = it * LG_ROWS;
    if (issued == 0 || is == 0) {
      unsigned char* ub = Us + (it_ord & 1) * u_bytes;
      // (a copy instruction moves 64 chunks; the counts differ by wave, which only makes waits stricter)
      for (int ins = wave; ins < g.cq / 2; ins += 8) {
        const int p = ins * 64 + lane, row = p / g.cq;
        const int ch = (p - row * g.cq) ^ (2 * (row & 3));
        const int64_t grow = row0 + row < g.m ? row0 + row : g.m - 1;
        sb_async16(g.U + grow * g.k + (ch * 8 < g.k ? ch * 8 : 0), ub + ins * 1024);
      }
    }
    unsigned char* st = sb_smem + (issued % S) * STAGE_BYTES;
    const int64_t k0 = (int64_t)slab_at(it, is) * LG_BK;
    const int chunks = (int)((g.n_out - k0 < LG_BK ? g.n_out - k0 : LG_BK) >> 3);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int row = (wave * 2 + i) * 2 + (lane >> 5);
      const int ch = (lane & 31) ^ (row & 15);
      const int64_t grow = row0 + row < g.m ? row0 + row : g.m - 1;
      const bf16_t* src = g.dY + grow * g.n_out + k0 + (ch < chunks ? ch : 0) * 8;
      if (g.stream_x) sb_async16_stream(src, st + (wave * 2 + i) * 1024);
      else sb_async16(src, st + (wave * 2 + i) * 1024);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const int row = (wave * NB + i) * 2 + (lane >> 5);
      const int ch = (lane & 31) ^ (row & 15);
      sb_async16(g.B + (int64_t)(row < g.r ? row : 0) * g.n_out + k0 + (ch < chunks ? ch : 0) * 8,
                 st + A_BYTES + (wave * NB + i) * 1024);
    }
    ++issued;
    if (++is == g.slabs) { is = 0; ++it; ++it_ord; }
  };

  f32x4 tacc[3][CW];                                // T columns 16 (wave + 8 i) .. + 15 of U, all of G's
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int c = 0; c < CW; ++c) tacc[i][c] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 acc[2];
  acc[0] = acc[1] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};

  int64_t ct = it;
  int cs = is, ct_ord = 0;
  // at most one tile ahead: U has two buffers
  while (issued < total && issued < S - 1 && it_ord <= ct_ord + 1) issue();
  for (int s = 0; s < total; ++s) {
    // slab s has landed once at most the copies of the younger slabs are pending
    const int ahead = issued - s - 1;
    if (ahead >= 2) SB_WAIT_VMCNT(2 * LOADS);
    else if (ahead == 1) SB_WAIT_VMCNT(LOADS);
    else SB_WAIT_VMCNT(0);
    sb_barrier_lds();                                // everyone's copies landed; slab s - 1 and the tile before are consumed
    while (issued < total && issued < s + S && it_ord <= ct_ord + 1) issue();
    const unsigned char* st = sb_smem + (s % S) * STAGE_BYTES;
    const int64_t kvalid = g.n_out - (int64_t)slab_at(ct, cs) * LG_BK;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int kb = (kw * KS + ks) * 32;
      if (kb < kvalid) {
        const int pos = (((kb >> 3) + grp) ^ l16) << 4;
        const bf16x8 b = *(const bf16x8*)(st + A_BYTES + (cw * 16 + l16) * 512 + pos);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const bf16x8 a = *(const bf16x8*)(st + (i * 16 + l16) * 512 + pos);
          acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[i], 0, 0, 0);
        }
      }
    }
    if (cs + 1 == g.slabs || s + 1 == total) {
      // ---- end of the tile (or of the share): G = sum over the waves, then T += U^T [G_hi + G_lo]
      unsigned char* const ub = Us + (ct_ord & 1) * u_bytes;
      const int64_t left = g.m - ct * LG_ROWS;       // rows past m: zero in U and in G
      if (left < LG_ROWS) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        for (int e = (int)left * g.cq + t; e < LG_ROWS * g.cq; e += 512) *(u32x4*)(ub + e * 16) = z;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        *(f32x4*)(Red + (kw * RP + cw * 16 + l16) * LG_RED_LD + 16 * i + 4 * grp) = acc[i];
        acc[i] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
      }
      sb_barrier_lds();
#pragma unroll
      for (int e0 = 0; e0 < RP * LG_ROWS; e0 += 512) {
        const int c = (e0 + t) >> 5, row = t & 31;
        float v = Red[c * LG_RED_LD + row];
#pragma unroll
        for (int w = 1; w < KW; ++w) v += Red[(w * RP + c) * LG_RED_LD + row];
        if (row >= left || c >= g.r) v = 0.0f;
        const bf16_t hi = (bf16_t)v;
        Gt[c * LG_GT_LD + row] = hi;
        Gt[(RP + c) * LG_GT_LD + row] = (bf16_t)(v - (float)hi);
      }
      sb_barrier_lds();
      bf16x8 gf[2][CW];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < CW; ++c) gf[h][c] = *(const bf16x8*)(Gt + (h * RP + c * 16 + l16) * LG_GT_LD + 8 * grp);
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const int kt = wave + 8 * i;
        if (kt * 16 < g.k) {
          const int row = 8 * grp + (l16 >> 2), col = kt * 16 + 4 * (l16 & 3);
          const unsigned char* p = ub + row * g.cq * 16 + (((col >> 3) ^ (2 * (l16 >> 2))) << 4) + (col & 7) * 2;
          const s16x4 lo = sb_read_tr(p), hi = sb_read_tr(p + 4 * g.cq * 16);
          const bf16x8 a = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
          for (int c = 0; c < CW; ++c) {
            tacc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, gf[0][c], tacc[i][c], 0, 0, 0);
            tacc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, gf[1][c], tacc[i][c], 0, 0, 0);
          }
        }
      }
    }
    if (++cs == g.slabs) { cs = 0; ++ct; ++ct_ord; }
  }
  float* const out = g.part + (int64_t)blockIdx.x * g.k * RP;
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int kc = (wave + 8 * i) * 16 + 4 * grp + r;
        if (kc < g.k) out[kc * RP + c * 16 + l16] = tacc[i][c][r];
      }
}

// T = sum of the shares.  A workgroup owns 16 groups of 4 values; 16 lanes per group add the shares
// sub, sub + 16, ... in ascending order, and the 16 sums are added in order: the result depends on the
// number of shares only.
__global__ __launch_bounds__(256) void lora_tsum_kernel(const float* part, int shares, int count4, float* T) {
  __shared__ f32x4 red[16][16];
  const int gi = threadIdx.x & 15, sub = threadIdx.x >> 4;
  const int e = blockIdx.x * 16 + gi;
  const int ec = e < count4 ? e : count4 - 1;
  f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
  for (int w0 = sub; w0 < shares; w0 += 128) {
    f32x4 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int w = w0 + 16 * u < shares ? w0 + 16 * u : w0;
      v[u] = *(const f32x4*)(part + ((int64_t)w * count4 + ec) * 4);
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (w0 + 16 * u < shares) s += v[u];
  }
  red[sub][gi] = s;
  __syncthreads();
  if (threadIdx.x < 16 && e < count4) {
    f32x4 v = red[0][gi];
#pragma unroll
    for (int u = 1; u < 16; ++u) v += red[u][gi];
    *(f32x4*)(T + (int64_t)e * 4) = v;
  }
}

// One pass over dY, or the two products?  A matter of dY's bytes: the one pass takes 8 us (LoRA ranks 17 to 32 from
// the memory-side cache 12) and 5.35 TB/s at LoRA ranks up to 16, 4.38 above; the sketch kernel takes 6.8 TB/s in
// rounds of 256 workgroups of 128 rows, of which a partly filled one lasts at least 0.7 of a full one, and what the
// two products do besides takes 20 us and 0.4 ns per row.  Fitted to 449 pairs of measurements (dY 30 MB to 2.3 GB, n_out
// 1024 to 28672, 16 to 256 columns of U; below 128 MB it is one pass), where the choice is at most 4 % behind; one pass
// alone is up to 28 % behind (25600 x 16384 at rank 32: 206 against 162 us), the two products up to 65 %.
static bool lora_one_pass(int64_t m, int64_t n_out, int rp, int g_splits) {
  if (rp > 32) return false;
  const int64_t bytes = m * n_out * 2;
  if (bytes < (128ll << 20) || m > 65535ll * 128) return true;                    // (the sketch kernel's grid)
  const int64_t per = ceil_div64(ceil_div64(n_out, g_splits), SB_BK) * SB_BK;     // columns of dY per workgroup
  const int64_t wgs = ceil_div64(m, 128) * ceil_div64(n_out, per), last = wgs % 256;
  const double rounds = (double)(wgs / 256) + (last ? std::max(0.7, (double)last / 256.0) : 0.0);
  const double two_us = 20.0 + 0.4e-3 * (double)m + rounds * (256.0 * 128.0 * 2.0) * (double)per / 6.8e6;
  const double one_us = rp == 16 ? 8.0 + (double)bytes / 5.35e6
                                 : (sb_streams_past_cache(bytes) ? 8.0 : 12.0) + (double)bytes / 4.38e6;
  return one_us <= 1.02 * two_us;
}

// Workgroups of lora_gt for a partial buffer of `part_bytes`.
static int lora_gt_wgs(int64_t items, int k, int rp, size_t part_bytes) {
  const int64_t fit = (int64_t)(part_bytes / ((size_t)k * rp * 4));
  return (int)std::min<int64_t>(std::min<int64_t>(LG_WGS, items), fit);
}

template <int RP, int S>
static int launch_lora_gt_rp(hipStream_t s, const LoraGtArgs& g, int wgs) {
  static std::atomic<bool> attr_done{false};
  if (!attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)lora_gt_kernel<RP, S>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       160 * 1024);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(lora_gt LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("lora_gt", s, (lora_gt_kernel<RP, S>), dim3((unsigned)wgs), dim3(512), lora_gt_lds_bytes(RP, S, g.cq), g);
  return LORACT_OK;
}

// T (k x rp, fp32) for rp = 16 or 32, in *T_out and *shares pieces: few small shares are left to the product with V
// (lora_product_adds_shares) instead of to a launch.  Needs 16-byte aligned rows of U, dY and B, n_out a multiple of 64
// and k <= LORACT_MAX_RANK (checked by the caller).  part: scratch of part_bytes, room for one share at least.
static int launch_lora_t(hipStream_t s, LoraGtArgs g, int rp, int64_t n, float* T, size_t part_bytes, const float** T_out,
                         int* shares) {
  g.slabs = (int)ceil_div64(g.n_out, LG_BK);
  g.items = ceil_div64(g.m, LG_ROWS) * g.slabs;
  g.cq = (g.k + 63) / 64 * 8;
  g.stream_x = sb_streams_past_cache(g.m * g.n_out * 2);
  const int wgs = lora_gt_wgs(g.items, g.k, rp, part_bytes);
  if (wgs < 1) return LORACT_ERR_WORKSPACE_TOO_SMALL;
  if (g.items / wgs >= (1ll << 31) - 1) return LORACT_ERR_UNSUPPORTED;
  // (cq <= 40: 160256 and 162816 bytes of LDS at most)
  LORACT_TRY((rp == 16 ? launch_lora_gt_rp<16, 4>(s, g, wgs) : launch_lora_gt_rp<32, 3>(s, g, wgs)));
  const int count4 = g.k * rp / 4;
  *T_out = g.part;
  *shares = wgs;
  if (lora_product_adds_shares(wgs, g.k, rp, n)) return LORACT_OK;
  *T_out = T;
  *shares = 1;
  LORACT_LAUNCH("lora_tsum", s, lora_tsum_kernel, dim3((unsigned)((count4 + 15) / 16)), dim3(256), 0,
                (const float*)g.part, wgs, count4, T);
  return LORACT_OK;
}

// ---------------------------------------------------------------------------------------------
// Last contraction of the LoRA gradient: dA (n x r) = scale * V^T T, with V (k x n, bf16) and T, fp32, k x rp (LV_ONE), the
// k x 2 rp pair [T_hi | T_lo] (LV_PAIR) or some k x rp shares of it one after the other (LV_SHARES; a kind of its own, because
// the loop over them costs the others 0.9 us at 64 columns).  The kernel is one chain of latencies -- loads, products, a sum
// over the waves.  The products run on the float32 matrix cores: a workgroup owns
// 16 EC columns of V, wave w takes the groups of four rows w, w + WAVES, ..., a lane's EC consecutive columns of a row serve EC
// matrix instructions, whose other operand is four rows of T straight from memory.  The waves' results are added in their order
// through LDS.  The loads are all written before the first product, but the compiler moves them towards their use: with shares of T all of them
// are in flight together, else eight to ten of the 4 k / 64 at EC = 2 and LoRA ranks up to 16, and two at EC = 4 (of whatever k: 36 registers).
// As vector arithmetic on 32 columns per workgroup, T staged in LDS and every thread reading all of its rows from there,
// those reads took the longest.  us, so and now: k = 256, n = 11008 8.4 and 5.0, n = 4096 8.0 and 3.8; k = 128, n = 4096 4.7 and 3.3.

enum { LV_ONE, LV_PAIR, LV_SHARES };
static constexpr int lv_waves(int rp16) { return rp16 <= 2 ? 8 : 4; }          // (LDS: 17 to 66 KB)
static constexpr int lv_pitch(int rp16) { return 16 * rp16 + 1; }
template <int RP16, int Q8, int KIND, int EC>
__global__ __launch_bounds__(64 * lv_waves(RP16)) void lora_vtt_kernel(const bf16_t* V, const float* Tin, int shares, int k, int64_t n,
                                                                       int r, float scale, float* dA) {
  typedef __bf16 vec_t __attribute__((ext_vector_type(EC)));
  constexpr int RP = 16 * RP16, WAVES = lv_waves(RP16), STEPS = 16 * Q8 / WAVES, COLS = 16 * EC, LD = lv_pitch(RP16);
  extern __shared__ float lv_red[];            // [WAVES][COLS][LD]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, l16 = lane & 15, grp = lane >> 4;
  const int64_t j0 = (int64_t)blockIdx.x * COLS;
  const int64_t jl = j0 + l16 * EC, jc = jl + EC <= n ? jl : n - EC;     // (columns past the end repeat the last ones, never stored)
  vec_t v[STEPS];
  float tv[STEPS][RP16];
#pragma unroll
  for (int u = 0; u < STEPS; ++u) {
    const int q = 4 * (wave + WAVES * u) + grp, qc = q < k ? q : k - 1;
    v[u] = *(const vec_t*)(V + (int64_t)qc * n + jc);
#pragma unroll
    for (int c = 0; c < RP16; ++c) {
      const float* const src = Tin + (int64_t)qc * (KIND == LV_PAIR ? 2 : 1) * RP + 16 * c + l16;
      tv[u][c] = src[0];
      if (KIND == LV_PAIR) tv[u][c] += src[RP];
    }
  }
  if (KIND == LV_SHARES) {                     // (added in ascending order, the loads of a few shares in flight together)
    constexpr int B = STEPS * RP16 <= 8 ? 8 : 4;
    for (int w0 = 1; w0 < shares; w0 += B) {
      float sv[B][STEPS][RP16];
#pragma unroll
      for (int x = 0; x < B; ++x)
#pragma unroll
        for (int u = 0; u < STEPS; ++u) {
          const int w = w0 + x < shares ? w0 + x : w0;
          const int q = 4 * (wave + WAVES * u) + grp, qc = q < k ? q : k - 1;
#pragma unroll
          for (int c = 0; c < RP16; ++c) sv[x][u][c] = Tin[((int64_t)w * k + qc) * RP + 16 * c + l16];
        }
#pragma unroll
      for (int x = 0; x < B; ++x)
#pragma unroll
        for (int u = 0; u < STEPS; ++u)
#pragma unroll
          for (int c = 0; c < RP16; ++c)
            if (w0 + x < shares) tv[u][c] += sv[x][u][c];
    }
  }
  f32x4 acc[EC][RP16];
#pragma unroll
  for (int e = 0; e < EC; ++e)
#pragma unroll
    for (int c = 0; c < RP16; ++c) acc[e][c] = (f32x4){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int u = 0; u < STEPS; ++u) {
    const bool on = 4 * (wave + WAVES * u) + grp < k;                    // rows from k on are zero on both sides
#pragma unroll
    for (int e = 0; e < EC; ++e)
#pragma unroll
      for (int c = 0; c < RP16; ++c)
        acc[e][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(on ? (float)v[u][e] : 0.0f, on ? tv[u][c] : 0.0f, acc[e][c], 0, 0, 0);
  }
  // register x of lane l: column EC (4 (l / 16) + x) + e of the workgroup, entry 16 c + l % 16 of its row
#pragma unroll
  for (int e = 0; e < EC; ++e)
#pragma unroll
    for (int c = 0; c < RP16; ++c)
#pragma unroll
      for (int x = 0; x < 4; ++x) lv_red[(wave * COLS + EC * (4 * grp + x) + e) * LD + 16 * c + l16] = acc[e][c][x];
  __syncthreads();
  for (int o = threadIdx.x; o < COLS * RP; o += 64 * WAVES) {
    const int col = o / RP, c = o - col * RP;
    float sum = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) sum += lv_red[(w * COLS + col) * LD + c];
    if (j0 + col < n && c < r) dA[(j0 + col) * r + c] = scale * sum;
  }
}

// Columns of V per workgroup: 64 where that still gives two workgroups to a CU, else 32, with which half of a wave's loads are in flight together, not
// two at a time.  Whole gradient of 512 rows and 512 columns of dY, us, with 32 and with 64: k = 256, LoRA rank 16, n = 4096 9.8 and 11.1, 11008 10.7 and 11.2, 32768
// 14.0 and 13.2; rank 64, n = 11008 27.6 and 29.7, 32768 36.8 and 34.6.  Where it adds the shares of T (all loads in flight either way), 64 where that gives every other CU a
// workgroup (200 rows, n = 11008: k = 16 9.1 and 8.7, k = 128 11.3 and 10.9).
static constexpr int lv_wide_wgs(int kind) { return kind == LV_SHARES ? 128 : 512; }
template <int RP16, int Q8, int KIND, int EC>
static int launch_lora_vtt_ec(hipStream_t s, const bf16_t* V, const float* T, int shares, int k, int64_t n, int r, float scale,
                              float* dA) {
  constexpr size_t lds = (size_t)lv_waves(RP16) * 16 * EC * lv_pitch(RP16) * sizeof(float);
  static std::atomic<bool> attr_done{false};
  if (lds > 64 * 1024 && !attr_done.load(std::memory_order_acquire)) {
    hipError_t e = hipFuncSetAttribute((const void*)lora_vtt_kernel<RP16, Q8, KIND, EC>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return hip_fail(e, "hipFuncSetAttribute(lora_vtt LDS)");
    attr_done.store(true, std::memory_order_release);
  }
  LORACT_LAUNCH("lora_vtt", s, (lora_vtt_kernel<RP16, Q8, KIND, EC>), dim3((unsigned)ceil_div64(n, 16 * EC)),
                dim3(64 * lv_waves(RP16)), lds, V, T, shares, k, n, r, scale, dA);
  return LORACT_OK;
}
template <int RP16, int Q8, int KIND>
static int launch_lora_vtt_q8(hipStream_t s, const bf16_t* V, const float* T, int shares, int k, int64_t n, int r, float scale,
                              float* dA) {
  return ceil_div64(n, 64) >= lv_wide_wgs(KIND) ? launch_lora_vtt_ec<RP16, Q8, KIND, 4>(s, V, T, shares, k, n, r, scale, dA)
                                          : launch_lora_vtt_ec<RP16, Q8, KIND, 2>(s, V, T, shares, k, n, r, scale, dA);
}
template <int RP16, int KIND>
static int launch_lora_vtt_rp(hipStream_t s, const bf16_t* V, const float* T, int shares, int k, int64_t n, int r, float scale,
                              float* dA) {
  switch ((k + 63) / 64) {
    case 1: return launch_lora_vtt_q8<RP16, 1, KIND>(s, V, T, shares, k, n, r, scale, dA);
    case 2: return launch_lora_vtt_q8<RP16, 2, KIND>(s, V, T, shares, k, n, r, scale, dA);
    case 3: return launch_lora_vtt_q8<RP16, 3, KIND>(s, V, T, shares, k, n, r, scale, dA);
    case 4: return launch_lora_vtt_q8<RP16, 4, KIND>(s, V, T, shares, k, n, r, scale, dA);
    case 5: return launch_lora_vtt_q8<RP16, 5, KIND>(s, V, T, shares, k, n, r, scale, dA);
    default: return LORACT_ERR_UNSUPPORTED;
  }
}
// T: k x rp, in one piece or in shares that lie one after the other, or (pair) the k x 2 rp pair above; the one-pass route's ranks have both.
static int launch_lora_vtt(hipStream_t s, const bf16_t* V, const float* T, int k, int64_t n, int r, int rp, bool pair,
                           float scale, float* dA, int shares = 1) {
#define LV_CASE(N, KIND) launch_lora_vtt_rp<N, KIND>(s, V, T, shares, k, n, r, scale, dA)
  const int kind = pair ? LV_PAIR : (shares > 1 ? LV_SHARES : LV_ONE);
  switch (rp / 16) {
    case 1: return kind == LV_PAIR ? LV_CASE(1, LV_PAIR) : (kind == LV_SHARES ? LV_CASE(1, LV_SHARES) : LV_CASE(1, LV_ONE));
    case 2: return kind == LV_PAIR ? LV_CASE(2, LV_PAIR) : (kind == LV_SHARES ? LV_CASE(2, LV_SHARES) : LV_CASE(2, LV_ONE));
    case 3: return kind == LV_PAIR ? LV_CASE(3, LV_PAIR) : LORACT_ERR_INVALID_ARG;
    case 4: return kind == LV_PAIR ? LV_CASE(4, LV_PAIR) : LORACT_ERR_INVALID_ARG;
    default: return LORACT_ERR_UNSUPPORTED;
  }
#undef LV_CASE
}
