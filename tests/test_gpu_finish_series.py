"""The degree-4 finish of tall matrices at every width it has a kernel for: spectra on which a float64 model of the first round says
that the first-order finish does not reach, orthogonality of float32 factors and the basis against float64."""
import numpy as np
import pytest
import torch

from gpu_util import first_round

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [64, 128, 192, 256, 320])
def test_series_at_width(k):
    import paper_2509_23472_amd as L
    m, n = 32771, 400
    g = torch.Generator(device="cuda").manual_seed(k)
    noise = torch.randn((m, n), generator=g, device="cuda")
    for decades in np.arange(3.0, 4.2, 0.1):
        x = (noise * 10.0 ** (-float(decades) * torch.arange(n, device="cuda").clamp(max=k) / k)).bfloat16()
        defect, pivot = first_round(x, k, 3)
        if defect >= 0.04:
            break
    print(k, "decades", decades, "defect", defect, "pivot", pivot, flush=True)
    assert 0.04 <= defect <= 1.0 and pivot >= 4.0
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=3, factor_dtype=torch.float32, status=status)
    assert int(status.item()) == 0
    ud = u.double()
    got = float((ud.t().contiguous() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm())
    print("after", got, flush=True)
    # what the series leaves out is below 8e-5 (of a spectral norm of 0.2 at most, else the second factorisation is taken); the correction
    # is rounded to bf16, 2^-9 of its entries on either side of the product
    assert got <= 1e-4 * k ** 0.5 + 2.0 ** -8 * defect
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 3), dtype=np.int64)).cuda()
    q, _ = torch.linalg.qr(x.double() @ x[idx].double().t().contiguous())
    ref = q @ (q.t().contiguous() @ x.double())
    assert float((ud @ v.double() - ref).norm() / ref.norm()) <= 1e-2
