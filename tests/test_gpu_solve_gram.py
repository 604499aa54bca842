"""The Gram matrix that the solving workgroups leave beside Q1 (sketches of up to 64 columns): a last workgroup with one row,
one with all of its rows, the last row count before the solve goes over to wider strips and the first after it."""
import numpy as np
import pytest
import torch

from test_gpu_factor_solve import test_restart_with_dependent_rows as check_restart
from test_gpu_factor_solve import test_second_round as check_second_round

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k", [(513, 16), (1024, 17), (577, 33), (640, 48), (129, 64), (192, 64), (16320, 32), (16321, 32),
                                 (16320, 64), (16321, 64)])
@pytest.mark.parametrize("decades", [0.0, 3.0])
def test_basis(m, k, decades):
    import paper_2509_23472_amd as L
    n = 256
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn((m, n), generator=g, device="cuda") * 10.0 ** (-decades * torch.arange(n, device="cuda") / n)
    x = x.bfloat16()
    status = torch.zeros((1,), dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=5, factor_dtype=torch.float32, status=status)
    ud = u.double()
    defect = float((ud.t() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm())
    # Q1 is accepted up to ||E||_F = 1e-6; the first-order finish (64 columns) leaves 3/4 ||E||^2 <= 2e-4 (||E||_F <= 0.015)
    assert defect <= (2e-4 if k > 48 else 2e-6), defect
    assert int(status.item()) == 0
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 5), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t()
    q, _ = torch.linalg.qr(y)
    # V is formed from the bf16 copy of U (2^-9 of an entry) and projects X
    proj = q @ (q.t() @ x.double())
    assert float((ud @ v.double() - proj).norm() / proj.norm()) <= 8e-3


@pytest.mark.parametrize("m,k", [(1000, 64), (577, 16), (5000, 20), (9001, 33), (16320, 48), (16319, 64)])
def test_tiles_of_an_abandoned_attempt_are_overwritten(m, k):
    # dependent rows send the solving workgroups, the last of them with rows missing, back to their first panel: tiles or rows of
    # the attempt before would show in the singular values of U
    check_restart(m, k)


@pytest.mark.parametrize("m,k", [(700, 40), (1025, 50), (3000, 63), (9001, 33), (16320, 44), (5000, 64)])
def test_second_round_from_the_tiles(m, k):
    # (spectra where a float64 model says that the first round is not enough, asserted there)
    check_second_round(m, k)
