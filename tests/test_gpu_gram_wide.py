"""Orthonormalisation of sketches of more than 64 columns at the edges of the Gram kernel: every split of the columns into
blocks (two to four 16-column tiles), rows that end inside a wave's group, a workgroup's step, a slice, and shares that
go on into the next pair of blocks; and of short sketches, which another kernel takes.  U must be orthonormal and U V the
projection of X onto the sketch's range."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k", [(331, k) for k in (65, 81, 112, 128, 144, 160, 176, 192, 208, 257, 289, 320)] +
                         [(m, k) for m in (257, 1025, 4099, 16385) for k in (80, 130, 256)] +
                         [(33001, 80), (33001, 192), (40003, 256), (40003, 320)])
def test_basis_of_a_wide_sketch(m, k):
    import paper_2509_23472_amd as L
    k = min(k, m - 1)
    n = 384
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn((m, n), generator=g, device="cuda").bfloat16()
    status = torch.zeros((1,), dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=5, factor_dtype=torch.float32, status=status)
    ud = u.double()
    # Q1 is accepted up to ||E||_F = 1e-6; entries of U carry one float32 rounding, 2^-24 of an entry.  The first-order finish
    # leaves 3/4 ||E||^2 <= 2e-4 (||E||_F <= 0.015), the series 8e-5.
    defect = float((ud.t() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm())
    assert defect <= 2e-4, defect
    assert int(status.item()) == 0
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 5), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t()
    q, _ = torch.linalg.qr(y)
    # V is formed from the bf16 copy of U (2^-9 of an entry) and projects X, of which k / n lies in the range
    proj = q @ (q.t() @ x.double())
    assert float((ud @ v.double() - proj).norm() / proj.norm()) <= 8e-3


@pytest.mark.parametrize("m,k", [(6307, k) for k in (65, 81, 112, 128)] + [(4211, k) for k in (144, 160, 176, 192, 208, 225, 256)] +
                         [(2171, k) for k in (257, 289, 304, 320)])
def test_every_split_above_the_rows_of_a_short_sketch(m, k):
    # (shorter ones have a kernel of their own, gram_is_short in gram_plan.h; these have the one that cuts the columns into blocks)
    test_basis_of_a_wide_sketch(m, k)
