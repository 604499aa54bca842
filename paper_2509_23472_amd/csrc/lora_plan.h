// Rule of the LoRA gradient's last product (lora_vtt_kernel in lora_bf16.h).  Plain C++, so that it can be tested without a GPU.
#pragma once
#include <cstdint>

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
