"""Reconstructions whose rank is one or two slabs of the general bf16 product: ranks at the steps of 16, 32, 64
and 128, sides at the 64-wide tiles, and that low ranks do not cost more than high ones.

Products of bf16 values are exact in float32 and K of them are added in float32, in whatever order:
|d| <= K 2^-24 sum |terms| (float32 results); bf16 results add 2^-8 |ref|."""
import numpy as np
import pytest
import torch

from workloads import synth

from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 15, 16, 17, 32, 33, 47, 63, 64, 65, 80, 97, 127, 128, 129])
@pytest.mark.parametrize("m,n", [(63, 65), (64, 128), (131, 8), (200, 323)])
def test_low_rank_reconstruction(m, n, k):
    import paper_2509_23472_amd as L
    print("case", m, n, k, flush=True)
    rng = np.random.default_rng(1000 * m + k)
    u = synth.round_to_bf16(rng.standard_normal((m, k)).astype(np.float32))
    v = synth.round_to_bf16(rng.standard_normal((k, n)).astype(np.float32))
    ud, vd = to_device(u, "bf16"), to_device(v, "bf16")
    wide = torch.full((m + 1, n + 3), 5.0, dtype=torch.float32, device="cuda")
    half = torch.full((m + 1, n + 3), 5.0, dtype=torch.bfloat16, device="cuda")
    L.loract_reconstruct(ud, vd, out_dtype=torch.float32, out=wide[:m, 1:n + 1])
    L.loract_reconstruct(ud, vd, out=half[:m, 1:n + 1])
    torch.cuda.synchronize()
    u, v = u.astype(np.float64), v.astype(np.float64)
    ref, acc = u @ v, k * 2.0 ** -24 * (np.abs(u) @ np.abs(v))
    assert np.all(np.abs(to_host(wide[:m, 1:n + 1]) - ref) <= acc)
    assert np.all(np.abs(to_host(half[:m, 1:n + 1]) - ref) <= acc + 2.0 ** -8 * (np.abs(ref) + acc))
    for guard in (wide, half):
        assert torch.all(guard[m:] == 5.0) and torch.all(guard[:, 0] == 5.0) and torch.all(guard[:, n + 1:] == 5.0)


def _us(fn):
    best = float("inf")
    for _ in range(6):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(10):
            fn()
        e1.record()
        torch.cuda.synchronize()
        best = min(best, e0.elapsed_time(e1) * 100.0)
    return best


def test_float32_output_of_low_rank_costs_less_than_of_high_rank():
    # 16384 x 3072 (201 MB to write): rank 16 33 us, rank 128 54; with tiles too large for the one slab 60 and 65
    import paper_2509_23472_amd as L
    t = {}
    for k in (16, 128):
        u, v = torch.randn((16384, k), device="cuda").bfloat16(), torch.randn((k, 3072), device="cuda").bfloat16()
        out = torch.empty((16384, 3072), dtype=torch.float32, device="cuda")
        t[k] = _us(lambda: L.loract_reconstruct(u, v, out_dtype=torch.float32, out=out))
    print(t)
    assert t[16] <= 0.75 * t[128], t
