"""GPU parity of the general bf16 product (rows of any alignment) at the edges of its tiles: rows shorter
than a 16-byte piece, sizes one off the 64 / 128 tiles and the 64-deep slabs, one and several slabs,
and K split over workgroups.

Products of bf16 values are exact in float32 and K of them are added in float32, in whatever order:
|d| <= K 2^-24 sum |terms| (fp32 results); bf16 results add half a unit in the last place, at most
2^-8 |ref| with 8 significant bits (1.0 and its neighbour are 2^-7 apart)."""
import numpy as np
import pytest
import torch

from oracle import loract_oracle as orc
from workloads import synth

from gpu_util import check_compress_parity, to_device, to_host

pytestmark = pytest.mark.gpu


def _bf16(rng, *shape):
    return synth.round_to_bf16(rng.standard_normal(shape).astype(np.float32))


@pytest.mark.parametrize("m,n,k", [(1, 7, 3), (130, 129, 1), (127, 130, 9), (128, 136, 63), (257, 1031, 65), (129, 255, 192),
                                   (1000, 77, 321)])
def test_reconstruct_of_unaligned_factors(m, n, k):
    import paper_2509_23472_amd as L
    print("case", m, n, k, flush=True)
    rng = np.random.default_rng(m + n + k)
    u, v = _bf16(rng, m, k), _bf16(rng, k, n)
    ud, vd = to_device(u, "bf16"), to_device(v, "bf16")
    guard = torch.full((m + 1, n + 3), 5.0, dtype=torch.bfloat16, device="cuda")     # rows that are not contiguous
    L.loract_reconstruct(ud, vd, out=guard[:m, 1:n + 1])
    wide = L.loract_reconstruct(ud, vd, out_dtype=torch.float32)
    torch.cuda.synchronize()
    u, v = u.astype(np.float64), v.astype(np.float64)
    ref, acc = u @ v, k * 2.0 ** -24 * (np.abs(u) @ np.abs(v))
    assert np.all(np.abs(to_host(wide) - ref) <= acc)
    assert np.all(np.abs(to_host(guard[:m, 1:n + 1]) - ref) <= acc + 2.0 ** -8 * (np.abs(ref) + acc))
    assert torch.all(guard[m:] == 5.0) and torch.all(guard[:, 0] == 5.0) and torch.all(guard[:, n + 1:] == 5.0)


@pytest.mark.parametrize("m,n_out,r", [(150, 5, 5), (129, 75, 64), (128, 1031, 33), (300, 2047, 12)])
def test_unaligned_gradient_product(m, n_out, r):
    # with U = V = I the LoRA gradient is dY B^T itself: both operands contiguous along K
    import paper_2509_23472_amd as L
    print("case", m, n_out, r, flush=True)
    rng = np.random.default_rng(m + r)
    dy, b, eye = _bf16(rng, m, n_out), _bf16(rng, r, n_out), np.eye(m, dtype=np.float32)
    out = L.loract_lora_grad(to_device(eye, "bf16"), to_device(eye, "bf16"), to_device(dy, "bf16"), to_device(b, "bf16"))
    torch.cuda.synchronize()
    dy, b = dy.astype(np.float64), b.astype(np.float64)
    # (the product is handed on in float32 or as two bf16 halves: 2^-16 of the value)
    bound = n_out * 2.0 ** -24 * (np.abs(dy) @ np.abs(b).T) + 2.0 ** -16 * np.abs(dy @ b.T) + 1e-30
    assert np.all(np.abs(to_host(out) - dy @ b.T) <= bound)


@pytest.mark.parametrize("m,n,k", [(1030, 1031, 65), (2050, 517, 130), (700, 2051, 64)])
def test_unaligned_compress_with_split_contractions(m, n, k):
    import paper_2509_23472_amd as L
    print("case", m, n, k, flush=True)
    x64 = synth.spectrum_matrix(m, n, 0.95 ** np.arange(min(m, n)), 1e-3, m + k)
    w = synth._finish("unaligned_%dx%d" % (m, n), x64, "bf16", k, m + k)
    u, v = L.loract_compress(to_device(w.x, "bf16"), k, seed=w.seed)
    xhat = L.loract_reconstruct(u, v)
    torch.cuda.synchronize()
    print(check_compress_parity(w, u, v, xhat))
