"""Copies to LDS take their LDS address as 32 bits: where the compiler cannot tell that the pointer is one into LDS it
forms the 64-bit generic address and compares it with null for every copy, six instructions more per kilobyte."""
import os
import subprocess

PKG = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd")
KERNEL = r'''
#include "%s/csrc/common.h"
__global__ void ring(const float4* src, float* out, int slabs, int pitch) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  float s = 0.0f;
  for (int i = 0; i < slabs; ++i) {
    unsigned char* st = smem + (i & 1) * 8192;
    for (int u = 0; u < 2; ++u) {
      sb_async16(src + i * pitch + u * 64 + lane, st + (wave * 2 + u) * 1024);
      sb_async16_stream(src + i * pitch + u * 64 + lane, st + 4096 + (wave * 2 + u) * 1024);
      sb_async16_device(src + i * pitch + u * 64 + lane, st + 6144 + (wave * 2 + u) * 1024);
    }
    SB_WAIT_VMCNT(0);
    sb_barrier_lds();
    s += ((const float*)st)[threadIdx.x];
    sb_barrier_lds();
  }
  out[threadIdx.x] = s;
}
'''


def test_no_generic_addresses(tmp_path):
    from paper_2509_23472_amd import build
    src, asm = tmp_path / "ring.hip", tmp_path / "ring.txt"
    src.write_text(KERNEL % PKG)
    flags = [f for f in build.HIPCC_FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.hipcc_path()] + flags + ["-S", "--offload-device-only", str(src), "-o", str(asm)], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    text = asm.read_text()
    assert text.count("global_load_lds_dwordx4") >= 6
    assert "src_shared_base" not in text and "s_cmp_lg_u64" not in text
