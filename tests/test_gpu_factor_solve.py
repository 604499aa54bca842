"""Factorisation and solve in one launch at the edges of its strips (64 rows per workgroup up to 16320 rows, 128 above,
several strips per workgroup), of its panels of 16 columns, and with a restart (an unshifted attempt that breaks down
sends the solving workgroups back to their first strip), against float64; and the same launch of the second round, on
spectra where a float64 model says that the first one is not enough."""
import numpy as np
import pytest
import torch

from gpu_util import first_round

pytestmark = pytest.mark.gpu


def _sketch_q(x, m, k, seed):
    import paper_2509_23472_amd as L
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, seed), dtype=np.int64)).cuda()
    return x.double() @ x[idx].double().t().contiguous()


@pytest.mark.parametrize("m,k", [(700, 72), (700, 80), (704, 240), (705, 256), (4095, 112), (16320, 96), (16321, 96),
                                 (16321, 176), (32768, 136), (40000, 80)])
@pytest.mark.parametrize("decades", [0.5, 2.0])
def test_basis(m, k, decades):
    import paper_2509_23472_amd as L
    print("shape", m, k, decades, flush=True)
    n = 384
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn((m, n), generator=g, device="cuda")
    x = (x * 10.0 ** (-decades * torch.arange(n, device="cuda") / n)).bfloat16()
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=3, factor_dtype=torch.float32, status=status)
    assert int(status.item()) == 0
    ud = u.double()
    gram = ud.t().contiguous() @ ud
    # 1e-3 is the library's own bound (first-order finish of the second round); nothing here is near it
    assert float(torch.linalg.matrix_norm(gram - torch.eye(k, device="cuda", dtype=torch.float64), 2)) <= 2e-4
    q, _ = torch.linalg.qr(_sketch_q(x, m, k, 3))
    ref = q @ (q.t().contiguous() @ x.double())
    # V is formed from the bf16 copy of the basis (2^-9 of an entry), the sketch accumulated in float32
    assert float((ud @ v.double() - ref).norm() / ref.norm()) <= 1e-2


@pytest.mark.parametrize("m,k", [(700, 72), (704, 240), (705, 208), (4095, 112), (16320, 96), (16321, 176), (32768, 136),
                                 (40000, 80), (700, 128), (4095, 256)])
def test_second_round(m, k):
    import paper_2509_23472_amd as L
    print("shape", m, k, flush=True)
    n = 384
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn((m, n), generator=g, device="cuda")
    x = (x * 10.0 ** (-3.0 * torch.arange(n, device="cuda").clamp(max=k) / k)).bfloat16()
    defect, pivot = first_round(x, k, 3)
    assert defect >= 1e-5, "the first round (accepted up to 1e-6) would do"
    assert k % 64 or defect <= 1.2e-2, "beyond the first-order finish (0.015)"
    assert pivot >= 8.0, "the unshifted attempt would be abandoned"
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=3, factor_dtype=torch.float32, status=status)
    assert int(status.item()) == 0
    ud = u.double()
    got = float((ud.t().contiguous() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm())
    print("defect of the first round", defect, "now", got, flush=True)
    # float32 storage of U, 2^-24 of an entry: sqrt(k) of them at most; at a multiple of 64 columns the first-order finish
    # leaves 3/4 of the defect's square and has rounded the correction to bf16 (2^-8 of it)
    bound = 5e-7 * k ** 0.5 + 1e-6
    if k % 64 == 0:
        bound += 2 * defect ** 2 + 2.0 ** -8 * defect
    assert got <= bound
    q, _ = torch.linalg.qr(_sketch_q(x, m, k, 3))
    ref = q @ (q.t().contiguous() @ x.double())
    assert float((ud @ v.double() - ref).norm() / ref.norm()) <= 1e-2


@pytest.mark.parametrize("m,k", [(1000, 96), (9000, 144), (20000, 256)])
def test_restart_with_dependent_rows(m, k):
    # a third of the rows are zero (padding tokens): pivots vanish, the first attempt is abandoned
    import paper_2509_23472_amd as L
    print("shape", m, k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn((m, 320), generator=g, device="cuda").bfloat16()
    x[::3] = 0.0
    for _ in range(2):
        u, v = L.loract_compress(x, k, seed=4, factor_dtype=torch.float32)
        y = _sketch_q(x, m, k, 4)
        y = y[:, y.norm(dim=0) > 0].contiguous()
        q, _ = torch.linalg.qr(y)
        ref = q @ (q.t().contiguous() @ x.double())
        assert torch.isfinite(u).all() and torch.isfinite(v).all()
        # the independent sampled rows give orthonormal columns, the others (their number is known here) zero ones
        sv, rank = torch.linalg.svdvals(u.double()), y.shape[1]
        bound = 2e-4 if k % 64 == 0 else 5e-7 * k ** 0.5 + 1e-6       # (first-order finish; float32 storage)
        assert float((sv[:rank] - 1.0).abs().max()) <= bound and float(sv[rank:].max()) <= 1e-6
        assert float((u.double() @ v.double() - ref).norm() / ref.norm()) <= 1e-2


@pytest.mark.parametrize("m,k", [(40000, 144), (33000, 185), (40000, 208)])
def test_basis_of_tall_matrices_above_128_columns(m, k):
    # a launch each for factorisation and solve, with registers for 12 blocks of columns and for 16
    test_basis(m, k, 1.0)


@pytest.mark.parametrize("m,k", [(33000, 14), (33000, 44), (33000, 64), (33000, 96), (33001, 185), (33000, 250), (33000, 256)])
def test_restart_of_a_factorisation_of_its_own(m, k):
    # a launch each for factorisation and solve: every instantiation of the first (1, 4, 8, 12 and 16 blocks of 16 columns) reads its
    # matrix again from the copy in blocks, with the shift of the sum of the diagonal, and says that rows were dependent
    import paper_2509_23472_amd as L
    test_restart_with_dependent_rows(m, k)
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn((m, 320), generator=g, device="cuda").bfloat16()
    for zero, flag in ((True, L.STATUS_RANK_DEFICIENT), (False, 0)):
        if zero:
            x0 = x.clone()
            x0[::3] = 0.0
        status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
        L.loract_compress(x0 if zero else x, k, seed=4, factor_dtype=torch.float32, status=status)
        assert int(status.item()) == flag
