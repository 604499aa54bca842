// Rules of the LoRA gradient.  Plain C++, so that they can be tested without a GPU.
#pragma once
#include <cstdint>

// K splits of dY B^T by the general product, for a dY whose rows are not aligned.  planned: the streaming kernel's number, of at least 512
// columns each; wanted: what the general product would take; fit: partial results that there is room for.  Where K is split anyway, so that a
// launch adds the shares, as many as are wanted and fit; more than 6 MB of them only up to 12 MB and if they are at least twice the planned number, because then
// they cost what they gain and a few more than planned are worse than either.  Whole gradient of 64 columns of U and 1024 of V, us, by the planned number and by
// more: 3001 x 1030 of LoRA rank 16 (shares of 0.2 MB) 23.6 and 20.7, of 64 (0.8 MB) 28.3 and 26.6; 1000 x 2050 of rank 32 26.9 and 24.3; 16000 x 11000 of rank 16 (1 MB)
// 111 and 95, of 40 (2.4 MB, 2 shares) 118 and, with 3, 123, with 4, 107; of 64 (3.9 MB) 122 and, with 3, 129, with 4, 130; 3001 x 11000 of rank 64 (10 shares)
// 39.6 and, with 16, 42.0.
// A product in one piece stays so: split, 4982 x 526 takes 1.8 us less on the GPU, but 3 more for a program whose launches the GPU waits for.
static inline int lora_general_splits(int planned, int64_t wanted, int64_t fit, int64_t m, int r) {
  if (planned == 1) return 1;
  const int64_t s = wanted < fit ? wanted : fit, bytes = s * m * r * 4;
  if (s < 1) return 1;
  return s <= planned || bytes <= 6 << 20 || (bytes <= 12 << 20 && s >= 2 * planned) ? (int)s : planned;
}

// Whether the product with V adds the shares of T itself instead of leaving that to a launch.  Every workgroup of it reads all
// shares (k x rp float32), eight after the first at a time; the launch costs about 1.8 us, a batch of eight some 0.5 us with
// 4 KB of it in a share, twice and four times that with 8 and 16 KB.  Whole gradient of 512 columns of dY, us, by launch minus
// by the product, with 8, 16 and 24 shares (two columns of V or 11008 make no difference):
//   4 KB (rank 64, LoRA rank 16)   1.8   1.3   0.7       (32 shares 0.2, 48 -0.9)
//   8 KB (64, 32; 128, 16)         1.4   0.4  -0.7
//   16 KB (128, 32)                0.7  -1.2  -3.1
//   32 KB (256, 32)               -0.5  -4.4  -4.3
// So the batches times the bytes of a share are kept to 16 KB, and what all workgroups together read again to 8 MB.
static inline bool lora_product_adds_shares(int shares, int k, int rp, int64_t n) {
  const int64_t share_bytes = (int64_t)k * rp * 4, batches = (shares + 6) / 8;
  return shares <= 24 && batches * share_bytes <= 16 * 1024 && shares * share_bytes * ((n + 31) / 32) <= 8 << 20;
}
