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

// Whether the product with V (lora_vtt_kernel in lora_bf16.h) adds the shares of T itself instead of leaving that to a launch.  A lane of it loads what its steps
// need of every share, eight shares after the first at a time where that is at most eight values, else four; the launch costs about 2.2 us, such a
// batch 0.6 us with two values in a share, 0.9 with four, 2.4 with eight, at LoRA ranks above 16 a half more.  Whole gradient of 256 columns of dY, us, by launch minus by the
// product, 4, 8, 12, 16, 24 and 32 shares; mean of 256 and 4096 columns of V, which differ by at most 0.3:
//   k, rp
//    64, 16      1.7    1.7    1.1    1.1    0.5   -0.2
//   128, 16      1.6    1.6    0.8    0.8   -0.1   -1.1
//   192, 16      0.7    0.8   -0.6   -0.6   -2.1   -3.5
//   256, 16      0.1   -0.3   -2.3   -2.8   -5.3   -8.1
//   320, 16      1.1    0.1   -0.9   -1.9   -4.0   -6.1
//    64, 32      1.4    1.1    0.1   -0.2   -1.5   -3.1
//   128, 32      0.5    0.3   -1.6   -1.9   -4.2   -6.6
//   192, 32      1.4    0.2   -1.0   -2.2   -4.6   -7.1
//   256, 32      1.2   -0.3   -1.8   -3.3   -6.3   -9.3
//   320, 32      1.0   -0.8   -2.6   -4.2   -7.8  -11.3
// All workgroups together read at most 64 MB of shares again: timed up to 45 MB (11008 columns).
static inline bool lora_product_adds_shares(int shares, int k, int rp, int64_t n) {
  const int steps = 2 * ((k + 63) / 64), values = steps * rp / 16, batch = values <= 8 ? 8 : 4;
  const int batches = (shares + batch - 2) / batch, few = (rp <= 16 ? 8 : 4) / values;
  return shares <= 24 && batches <= (few > 1 ? few : 1) && (int64_t)shares * k * rp * 4 * ((n + 31) / 32) <= 64 << 20;
}
