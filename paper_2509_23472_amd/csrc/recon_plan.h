// Rules of the reconstruction from bf16 factors (reconstruct_mfma_kernel, reconstruct_narrow_kernel in stream_bf16.h).  Plain C++, so that they can
// be tested without a GPU.
#pragma once
#include <cstdint>

// Whether blocks of 128 columns are taken instead of 256 (up to rank 256; above it there are no others).
//  - Tiles of 64 x 128 that find a CU each: both forms then last as long as one workgroup, which loads V, one tile of U, and stores.  us, narrow and
//    wide: 200 x 768 of rank 32 3.8 and 4.1, of rank 128 5.5 and 5.7, of rank 144 5.9 and 6.6; 1024 x 2048 of rank 64 4.8 and 4.9, of rank 256 8.1 and
//    8.8.  One and a half times as many, 4096 x 768: rank 32 4.9 and 4.8, rank 144 7.5 and 7.4, rank 256 12.7 and 9.2.
//  - Xhat of at most 128 columns, half of a wide block at most (32768 x 128: rank 32 5.3 and 5.6, rank 128 7.3 and 7.7).
static inline bool reconstruct_narrow_wins(int64_t m, int64_t n, int k) {
  return (m + 63) / 64 * ((n + 127) / 128) <= 256 || (n <= 128 && k <= 128);
}

// Whether Xhat is stored non-temporally: from 128 MB on, where its rows are whole lines of 128 bytes.
// The memory-side cache (256 MB) takes plain stores faster than memory does, but then holds little else for the kernels that follow, the first of
// which may read Xhat, and for the next step's X.  Plain stores against non-temporal ones, time of the whole sequence, mean of 45 sizes of rank 8 to 120, with
// n columns of dY, at most 4096:
//                                              128..144 MB   ..160   ..192   ..256
//   reconstruction, LoRA gradient                     0.94    0.97    1.04    0.99   (alone 0.75 to 1)
//   the same and the pre-norm backward, which reads   1.03    1.03    1.05    1.04
//   with that backward between the two                0.98    1.00    1.02    1.02
//   compress, reconstruction, gradient                1.06    1.08    1.09    1.01
//   the same and the backward                         1.00    1.01    1.01    1.02
// and at higher ranks, whose matrix instructions hide the stores, us, plain and non-temporal, of the reconstruction alone, with the gradient behind
// it, with the backward, with both:
//   16384 x 4096, 128 MB, rank 256     41  39     79  77    120 126    168 160
//   8192 x 9600, 150 MB, rank 192      42  47     66  68    147 145    178 169
//   16384 x 5120, 160 MB, rank 256     54  52     93  86    155 150    203 184
//   8192 x 11008, 172 MB, rank 256     54  56     78  76    176 167    204 191
//   20480 x 4992, 195 MB, rank 192     54  53    110  94    183 171    235 211
// Smaller ones lose: 8192 x 6144, 96 MB, of rank 64 with the gradient 43 and 45, with both 99 and 104.  (A product dY^T Xhat right behind it takes 2 to 4 % longer with
// non-temporal stores up to 224 MB, the same with the gradient between them.)
// A line that two non-temporal stores fill in part goes to memory twice, and not as a whole: 50000 x 3000 of rank 32 67 us, non-temporal 164.
static inline bool reconstruct_streams_out(int64_t m, int64_t n, bool whole_lines) { return whole_lines && m * n * 2 >= (int64_t)128 << 20; }
