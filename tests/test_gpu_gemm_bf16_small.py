"""Projections of unaligned operands that have fewer tiles than the GPU has CUs: 64 x 64 tiles, K split finer
from 384 rows on.  V against U^T X of the U that was returned, and the compression against the oracle."""
import numpy as np
import pytest
import torch

from workloads import synth

from gpu_util import check_compress_parity, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [65, 256, 319, 383, 384, 385, 449, 1000])
@pytest.mark.parametrize("n,k", [(63, 5), (65, 33), (129, 63), (200, 65), (1031, 12)])
def test_compress_with_few_tiles(m, n, k):
    import paper_2509_23472_amd as L
    if k >= m // 4:
        k = m // 4
    print("case", m, n, k, flush=True)
    x64 = synth.spectrum_matrix(m, n, 0.95 ** np.arange(min(m, n)), 1e-3, m + n)
    w = synth._finish("few_tiles_%dx%d" % (m, n), x64, "bf16", k, m + k)
    x = to_device(w.x, "bf16")
    u, v = L.loract_compress(x, k, seed=w.seed)
    xhat = L.loract_reconstruct(u, v)
    torch.cuda.synchronize()
    check_compress_parity(w, u, v, xhat)
    # V is U^T X in float32, stored in bf16: fp32 sums of m terms and half a unit in the last place
    ref = u.double().t().contiguous() @ x.double()
    mag = u.double().abs().t().contiguous() @ x.double().abs()
    assert torch.all((v.double() - ref).abs() <= m * 2.0 ** -24 * mag + 2.0 ** -8 * ref.abs())
    again = L.loract_compress(x, k, seed=w.seed)
    assert torch.equal(again[0], u) and torch.equal(again[1], v)
