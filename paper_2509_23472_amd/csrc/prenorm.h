// Pre-norm unit of Section 3.3: the RMS normalisation whose OUTPUT A = Norm(X) is the activation
// that gets stored (compressed) and shared by Norm and the sub-layer, and the backward step that
// recovers dL/dX from the stored A, the RMS vector and dL/dA (Eqs. 6-10):
//
//   forward   rms_i = sqrt(mean_j X_ij^2 + eps),  A_ij = X_ij / rms_i * gamma_j
//   backward  Xbar = A / gamma,  dXbar = dA * gamma,
//             dX_ij = (dXbar_ij - Xbar_ij * mean_j(dXbar_ij Xbar_ij)) / rms_i
//             (the mean is mean_j(dA_ij A_ij): gamma cancels in the product)
//
// Both are bandwidth-bound row kernels.  Rows that allow 16-byte accesses and are not too long are
// held in registers between the sum over the row and the result (prenorm_rows_kernel below); the
// others take two sweeps with one wavefront per row, the second one served by the caches.
#pragma once
#include "common.h"

#include <algorithm>

#define PN_GRID 2048   // workgroups that walk over the rows: eight per CU

struct PrenormArgs {
  const void* X;       // forward: X; backward: A (reconstructed activation)
  int64_t ldx;
  const void* dA;      // backward only
  int64_t ldda;
  const float* gamma;  // n
  float* rms;          // forward: out (m); backward: in
  void* out;           // forward: A; backward: dX
  int64_t ldo;
  int64_t m, n;
  int ek;              // element kind of X / dA / out (EK_F32 or EK_BF16)
  int vec;             // two sweeps: 16-byte accesses legal (bf16 only)
  float eps;
};

__device__ inline float pn_wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ inline float pn_load(const void* p, int64_t i, int ek) {
  return ek == EK_F32 ? ((const float*)p)[i] : (float)((const bf16_t*)p)[i];
}
__device__ inline void pn_store(void* p, int64_t i, int ek, float v) {
  if (ek == EK_F32) ((float*)p)[i] = v; else ((bf16_t*)p)[i] = (bf16_t)v;
}

// Rows in registers.  A row belongs to WPR waves of a workgroup of four; every lane owns NC pieces of
// 16 bytes per row, at the same columns in all rows, so that its gamma (and 1 / gamma) stays in
// registers while the workgroup walks over the rows, R at a time.  Against two sweeps that read X and
// gamma (twice the bytes of a bf16 row) again for every row: 34.6 -> 25.2 us
// forward and 49.9 -> 41.3 us backward at 8192 x 4096 bf16, where a device copy of X takes 26.2 us.
//
// The backward quotient A / gamma is formed as q = A rg, q + (A - q gamma) rg with rg = 1 / gamma,
// which rounds like the division; pieces whose gamma is outside 2^+-100 (where the residual could
// overflow or vanish) divide.
template <typename T, int WPR, int NC, int R, bool BWD>
__global__ __launch_bounds__(256) void prenorm_rows_kernel(PrenormArgs g) {
  constexpr int E = 16 / sizeof(T);                  // elements per piece
  constexpr int RG = 4 / WPR;                        // row groups per workgroup
  typedef T piece __attribute__((ext_vector_type(E)));
  __shared__ float red[2][4][R];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int part = wave % WPR;
  const int n = (int)g.n;
  int col[NC];                                       // clamped to the row's first piece when past its end
  bool on[NC];
  float gm[NC][E], rg[NC][E];
  bool exact_div = false;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int at = ((c * WPR + part) * 64 + lane) * E;
    on[c] = at < n;
    col[c] = on[c] ? at : 0;
#pragma unroll
    for (int e = 0; e < E; e += 4) {
      const f32x4 v = *(const f32x4*)(g.gamma + col[c] + e);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        gm[c][e + u] = v[u];
        if (BWD) {
          rg[c][e + u] = 1.0f / v[u];
          const float mag = fabsf(v[u]);
          exact_div = exact_div || !(mag > 0x1p-100f && mag < 0x1p100f);
        }
      }
    }
  }
  const int64_t step = (int64_t)gridDim.x * RG * R;
  int buf = 0;
  for (int64_t r0 = ((int64_t)blockIdx.x * RG + wave / WPR) * R; r0 - (wave / WPR) * R < g.m; r0 += step, buf ^= 1) {
    piece x[R][NC], d[R][NC];
    float rms[R], s[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = r0 + r < g.m ? r0 + r : g.m - 1;      // rows past the end are not stored
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        x[r][c] = *(const piece*)((const T*)g.X + row * g.ldx + col[c]);
        if (BWD) d[r][c] = *(const piece*)((const T*)g.dA + row * g.ldda + col[c]);
      }
      if (BWD) rms[r] = g.rms[row];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      s[r] = 0.0f;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        float p = 0.0f;
#pragma unroll
        for (int e = 0; e < E; ++e) p += (float)x[r][c][e] * (BWD ? (float)d[r][c][e] : (float)x[r][c][e]);
        s[r] += on[c] ? p : 0.0f;
      }
      s[r] = pn_wave_sum(s[r]);
    }
    if (WPR > 1) {
      // (two buffers: the barrier of the next trip separates this trip's reads from the writes after it)
      if (lane == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) red[buf][wave][r] = s[r];
      }
      __syncthreads();
      const int w0 = wave - part;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        s[r] = red[buf][w0][r];
#pragma unroll
        for (int w = 1; w < WPR; ++w) s[r] += red[buf][w0 + w][r];
      }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int64_t row = r0 + r;
      if (row >= g.m) continue;
      float inner = 0.0f;
      if (BWD) {
        inner = s[r] / (float)n;
      } else {
        rms[r] = sqrtf(s[r] / (float)n + g.eps);
        if (part == 0 && lane == 0) g.rms[row] = rms[r];
      }
      const float inv = 1.0f / rms[r];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        piece o;
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const float xv = (float)x[r][c][e], gv = gm[c][e];
          if (BWD) {
            float q = xv * rg[c][e];
            if (exact_div) q = xv / gv;
            else if (fabsf(q) < INFINITY) q = fmaf(fmaf(-q, gv, xv), rg[c][e], q);
            o[e] = (T)(((float)d[r][c][e] * gv - q * inner) * inv);
          } else {
            o[e] = (T)(xv * inv * gv);
          }
        }
        if (on[c]) *(piece*)((T*)g.out + row * g.ldo + col[c]) = o;
      }
    }
  }
}

// Any row length, alignment and element kind: one wavefront per row, two sweeps; 16-byte accesses for bf16
// rows that allow them (2048 x 24584, forward and backward: 49 and 83 us, element by element 283 and 491).
__global__ __launch_bounds__(256) void prenorm_forward_kernel(PrenormArgs g) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= g.m) return;
  const int64_t xo = row * g.ldx, oo = row * g.ldo;
  float ss = 0.0f;
  if (g.vec) {
    const bf16_t* x = (const bf16_t*)g.X + xo;
    for (int64_t c = lane * 8; c < g.n; c += 512) {
      const bf16x8 v = *(const bf16x8*)(x + c);
#pragma unroll
      for (int e = 0; e < 8; ++e) { const float f = (float)v[e]; ss += f * f; }
    }
  } else {
    for (int64_t c = lane; c < g.n; c += 64) { const float f = pn_load(g.X, xo + c, g.ek); ss += f * f; }
  }
  ss = pn_wave_sum(ss);
  const float rms = sqrtf(ss / (float)g.n + g.eps);
  if (lane == 0) g.rms[row] = rms;
  const float inv = 1.0f / rms;
  if (g.vec) {
    const bf16_t* x = (const bf16_t*)g.X + xo;
    bf16_t* o = (bf16_t*)g.out + oo;
    for (int64_t c = lane * 8; c < g.n; c += 512) {
      const bf16x8 v = *(const bf16x8*)(x + c);
      const f32x4 g0 = *(const f32x4*)(g.gamma + c), g1 = *(const f32x4*)(g.gamma + c + 4);
      bf16x8 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r[e] = (bf16_t)((float)v[e] * inv * g0[e]);
        r[e + 4] = (bf16_t)((float)v[e + 4] * inv * g1[e]);
      }
      *(bf16x8*)(o + c) = r;
    }
  } else {
    for (int64_t c = lane; c < g.n; c += 64)
      pn_store(g.out, oo + c, g.ek, pn_load(g.X, xo + c, g.ek) * inv * g.gamma[c]);
  }
}

__global__ __launch_bounds__(256) void prenorm_backward_kernel(PrenormArgs g) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= g.m) return;
  const int64_t ao = row * g.ldx, go = row * g.ldda, oo = row * g.ldo;
  float dot = 0.0f;
  if (g.vec) {
    const bf16_t* a = (const bf16_t*)g.X + ao;
    const bf16_t* d = (const bf16_t*)g.dA + go;
    for (int64_t c = lane * 8; c < g.n; c += 512) {
      const bf16x8 va = *(const bf16x8*)(a + c), vd = *(const bf16x8*)(d + c);
#pragma unroll
      for (int e = 0; e < 8; ++e) dot += (float)va[e] * (float)vd[e];
    }
  } else {
    for (int64_t c = lane; c < g.n; c += 64) dot += pn_load(g.X, ao + c, g.ek) * pn_load(g.dA, go + c, g.ek);
  }
  const float inner = pn_wave_sum(dot) / (float)g.n;
  const float inv = 1.0f / g.rms[row];
  if (g.vec) {
    const bf16_t* a = (const bf16_t*)g.X + ao;
    const bf16_t* d = (const bf16_t*)g.dA + go;
    bf16_t* o = (bf16_t*)g.out + oo;
    for (int64_t c = lane * 8; c < g.n; c += 512) {
      const bf16x8 va = *(const bf16x8*)(a + c), vd = *(const bf16x8*)(d + c);
      const f32x4 g0 = *(const f32x4*)(g.gamma + c), g1 = *(const f32x4*)(g.gamma + c + 4);
      bf16x8 r;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r[e] = (bf16_t)(((float)vd[e] * g0[e] - (float)va[e] / g0[e] * inner) * inv);
        r[e + 4] = (bf16_t)(((float)vd[e + 4] * g1[e] - (float)va[e + 4] / g1[e] * inner) * inv);
      }
      *(bf16x8*)(o + c) = r;
    }
  } else {
    for (int64_t c = lane; c < g.n; c += 64) {
      const float gm = g.gamma[c];
      const float v = (pn_load(g.dA, go + c, g.ek) * gm - pn_load(g.X, ao + c, g.ek) / gm * inner) * inv;
      pn_store(g.out, oo + c, g.ek, v);
    }
  }
}

// Widths in units of 256 pieces (a lane of each of four waves): up to 12 are kept in registers, and up to 6
// of the backward step's bf16 rows, of which a lane holds two rows, gamma and its reciprocal, 24 floats per
// piece: with 7 of them it spills and two sweeps are faster (4096 rows of 12288 columns: 64 us against 75 in
// two sweeps, 12296: 117 against 79).  A wave of its own is enough for a row of up to 128 pieces; the backward
// step takes bf16 ones one at a time (12608 x 768: 16.4 us by twos, 12.5 one by one; float32 rows of 64 columns the
// other way round, 100000 of them: 17.8 against 19.5; forward it makes no difference).
constexpr int pn_most_pieces(bool bf16, bool bwd) { return bf16 && bwd ? 6 : 12; }

template <typename T, bool BWD>
static int launch_prenorm_rows(hipStream_t s, const PrenormArgs& g, const char* name) {
  const int64_t pieces = ceil_div64(g.n, 16 / (int64_t)sizeof(T));
  const int64_t per_wave = pieces <= 128 ? ceil_div64(pieces, 64) : ceil_div64(pieces, 256);
#define PN_LAUNCH(WPR, NC, R)                                                                                    \
  {                                                                                                              \
    const int64_t wgs = std::min<int64_t>(ceil_div64(g.m, (4 / WPR) * R), PN_GRID);                               \
    LORACT_LAUNCH(name, s, (prenorm_rows_kernel<T, WPR, NC, R, BWD>), dim3((unsigned)wgs), dim3(256), 0, g);       \
    return LORACT_OK;                                                                                            \
  }
  if (pieces <= 128) {
    constexpr int R = BWD && sizeof(T) == 2 ? 1 : 2;
    if (per_wave == 1) PN_LAUNCH(1, 1, R)
    PN_LAUNCH(1, 2, R)
  }
  switch (per_wave) {
    case 1: PN_LAUNCH(4, 1, 2)
    case 2: PN_LAUNCH(4, 2, 2)
    case 3: PN_LAUNCH(4, 3, 1)
    case 4: PN_LAUNCH(4, 4, 1)
    case 5: case 6: PN_LAUNCH(4, 6, 1)
    default: break;
  }
  if constexpr (pn_most_pieces(sizeof(T) == 2, BWD) == 12) {
    if (per_wave <= 8) PN_LAUNCH(4, 8, 1)
    PN_LAUNCH(4, 12, 1)
  }
  return LORACT_ERR_INVALID_ARG;                     // (prenorm_rows_fit)
#undef PN_LAUNCH
}
static bool prenorm_rows_fit(int64_t n, int dtype, bool bwd) {
  const int64_t e = dtype == LORACT_BF16 ? 8 : 4;
  return n % e == 0 && n / e <= pn_most_pieces(dtype == LORACT_BF16, bwd) * 256;
}
