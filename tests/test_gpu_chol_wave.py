"""QR of narrow float32 sketches at the widths where the factor-and-invert kernel changes (16, 32 columns),
against float64 on the GPU's own inputs, and with dependent sampled rows (columns that drop out)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


# m: one pass over the rows, one split sixteen ways inside a workgroup (uneven), and further splits over workgroups
@pytest.mark.parametrize("m,k", [(700, k) for k in (1, 2, 15, 16, 17, 31, 32, 33)] + [(m, 16) for m in (300, 513, 1025, 5001)])
def test_basis_of_a_float32_sketch(m, k):
    import paper_2509_23472_amd as L
    n = 96
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn((m, n), generator=g, device="cuda")
    status = torch.zeros((1,), dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=9, status=status)
    assert int(status.item()) == 0
    ud, idx = u.double(), torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 9), dtype=np.int64)).cuda()
    # float64 inside, one float32 rounding of U: 2^-24 of an entry
    assert float((ud.t() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm()) <= 1e-6
    q, _ = torch.linalg.qr(x.double() @ x[idx].double().t())
    proj = q @ (q.t() @ x.double())
    assert float((ud @ v.double() - proj).norm() / proj.norm()) <= 1e-6


@pytest.mark.parametrize("k", [8, 24])
def test_dependent_rows_drop_out(k):
    # half of the rows are zero (padding tokens): the projection onto the independent sampled rows remains
    import paper_2509_23472_amd as L
    m, n = 256, 64
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn((m, n), generator=g, device="cuda")
    x[::2] = 0.0
    u, v = L.loract_compress(x, k, seed=4)
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 4), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t()
    p = y @ torch.linalg.pinv(y, rtol=1e-10)
    ref = p @ x.double()
    assert torch.isfinite(u).all() and torch.isfinite(v).all()
    assert float((u.double() @ v.double() - ref).norm() / ref.norm()) <= 1e-5


@pytest.mark.parametrize("k", [11, 12, 16])
def test_dependent_rows_among_11_to_16_columns_drop_out(k):
    # pivots at the rounding level: the row-broadcast form raises its flag and the guarded form takes over
    test_dependent_rows_drop_out(k)
