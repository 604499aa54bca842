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

// Whether Xhat is stored non-temporally.  The memory-side cache (256 MB) takes plain stores faster than memory does, but then holds little else for
// the kernels that follow.  Above rank 128 the matrix instructions hide the stores, mostly, and the second counts more; up to rank 128 the
// stores are what the kernel waits for.  us, plain and non-temporal, of the reconstruction alone, with the LoRA gradient of 4096 columns behind it, with the
// pre-norm backward that reads Xhat, and with both:
//   16384 x 4096, 128 MB, rank 256     41  39     79  77    120 126    168 160
//     rank 192                         36  35     75  71    114 117    161 153
//   8192 x 9600, 150 MB, rank 192      42  47     66  68    147 145    178 169
//   16384 x 5120, 160 MB, rank 256     54  52     93  86    155 150    203 184
//   8192 x 11008, 172 MB, rank 256     54  56     78  76    176 167    204 191
//     rank 192                         46  53     71  76    170 159    196 183
//     rank 64                          43  42     57  62    160 154    183 175
//   20480 x 4992, 195 MB, rank 192     54  53    110  94    183 171    235 211
//   28672 x 4096, 224 MB, rank 64      41  49     94 102    202 184    252 236
//   16384 x 8192, 256 MB, rank 64      51  52    100  85    232 209    270 246
//   24576 x 5632, 264 MB, rank 64      48  61     95 107    237 222    282 268
//   40000 x 4096, 312 MB, rank 64      75  67    137 137    285 256    352 325
//   65536 x 4096, 512 MB, rank 64     111 102    211 207    458 409    562 517
// (A product dY^T Xhat right behind it takes 2 to 4 % longer with non-temporal stores up to 224 MB, the same with the gradient between them.)
// The rows have to be whole lines of 128 bytes: one that two non-temporal stores fill in part goes to memory twice, and not as a whole (50000 x 3000
// of rank 32 67 us, non-temporal 164; 50048 x 3008 of rank 64 58 and 64).
static inline bool reconstruct_streams_out(int64_t m, int64_t n, int k, bool whole_lines) {
  return whole_lines && m * n * 2 >= (int64_t)(k > 128 ? 128 : 256) << 20;
}
