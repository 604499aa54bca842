"""Orthonormalisation of narrow sketches (up to 64 columns) at the edges of the Gram kernel's row chunks
and 16-column blocks: U must be orthonormal and U V the projection of X onto the sketch's range."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 16, 17, 40, 64])
@pytest.mark.parametrize("m", [64, 65, 127, 4096, 4097, 16385, 33000, 70001])
def test_basis_of_a_narrow_sketch(m, k):
    import paper_2509_23472_amd as L
    n = 128
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn((m, n), generator=g, device="cuda").bfloat16()
    status = torch.zeros((1,), dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=5, factor_dtype=torch.float32, status=status)
    ud = u.double()
    defect = float((ud.t() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm())
    # entries of U carry one fp32 rounding (2^-24 of an entry), E = Q1^T Q1 - I is accepted up to 1e-6
    assert defect <= 2e-6, defect
    assert int(status.item()) == 0
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 5), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t()
    q, _ = torch.linalg.qr(y)
    # V is formed from the bf16 copy of U (2^-9 of an entry) and projects X, of which k / n lies in the range
    proj = q @ (q.t() @ x.double())
    assert float((u.double() @ v.double() - proj).norm() / proj.norm()) <= 8e-3
