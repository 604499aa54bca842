"""Factorisation and solve in one launch at the edges of its strips (64 rows per workgroup up to 16320 rows, 128 above,
several strips per workgroup), of its panels of 16 columns, and with a restart (an unshifted attempt that breaks down
sends the solving workgroups back to their first strip), against float64."""
import numpy as np
import pytest
import torch

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
        assert float((u.double() @ v.double() - ref).norm() / ref.norm()) <= 1e-2
