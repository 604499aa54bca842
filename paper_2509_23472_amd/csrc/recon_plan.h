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

// Whether Xhat is stored non-temporally: where it is so large that with the operands of the next kernels it does not stay in the memory-side cache, and its
// rows are whole lines of 128 bytes.  A line that two such stores fill in part goes to memory twice, and not as a whole (50000 x 3000 of rank 32 67 us, non-temporal 164;
// 50048 x 3008 of rank 64 58 and 64).
static inline bool reconstruct_streams_out(int64_t m, int64_t n, bool whole_lines) { return whole_lines && m * n * 2 >= (int64_t)128 << 20; }
