"""GPU parity of the float64-accumulating product at the edges of its tiles: a side of 16 and less,
outputs of a few 32 x 32 tiles, outputs of 64 x 64 tiles, K below, at and between multiples of 16,
and K split over workgroups.  The operands are float32 and the accumulation float64, so the result is
the float32 rounding of the exact product up to 2^-53 sqrt(K) of its terms: |d| <= 2^-24 |ref| for
the rounding, and 1e-14 sum |terms| for the accumulation."""
import numpy as np
import pytest
import torch

from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


def _check(got, ref, mag):
    bound = 2.0 ** -24 * np.abs(ref) + 1e-14 * mag + 1e-300
    assert np.all(np.abs(got - ref) <= bound), np.max(np.abs(got - ref) / bound)


@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (16, 1000, 17), (777, 15, 16), (33, 33, 15), (100, 47, 64), (17, 500, 33),
                                   (1473, 1537, 40), (1500, 1471, 47)])
def test_fp32_reconstruct_at_the_tile_edges(m, n, k):
    import paper_2509_23472_amd as L
    print("case", m, n, k, flush=True)
    rng = np.random.default_rng(m + n + k)
    u = rng.standard_normal((m, k)).astype(np.float32)
    v = rng.standard_normal((k, n)).astype(np.float32)
    out = L.loract_reconstruct(to_device(u, "f32"), to_device(v, "f32"))
    torch.cuda.synchronize()
    u, v = u.astype(np.float64), v.astype(np.float64)
    _check(to_host(out), u @ v, np.abs(u) @ np.abs(v))


@pytest.mark.parametrize("m,k,r", [(255, 16, 4), (256, 17, 17), (5003, 40, 33), (8191, 5, 64)])
def test_fp32_split_contraction_over_the_rows(m, k, r):
    # U^T G splits its m-long contraction over workgroups from 512 rows on; with V = I the gradient is
    # that product (stored in float32 twice: G, then the result)
    import paper_2509_23472_amd as L
    print("case", m, k, r, flush=True)
    rng = np.random.default_rng(m)
    u = rng.standard_normal((m, k)).astype(np.float32)
    g = rng.standard_normal((m, r)).astype(np.float32)
    out = L.loract_lora_grad(to_device(u, "f32"), to_device(np.eye(k, dtype=np.float32), "f32"), to_device(g, "f32"),
                             to_device(np.eye(r, dtype=np.float32), "f32"))
    torch.cuda.synchronize()
    u, g = u.astype(np.float64), g.astype(np.float64)
    _check(to_host(out), u.T @ g, np.abs(u).T @ np.abs(g))
