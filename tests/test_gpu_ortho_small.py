"""The one-launch QR of small sketches at the edges of its range, of its strips of rows and of its tiles, against
float64: the rows and columns on either side of where the separate launches take over, second factorisations (steep
spectra, where a float64 model says that the first one is not enough), dependent sampled rows, float32 factors,
unaligned widths."""
import numpy as np
import pytest
import torch

from gpu_util import first_round

pytestmark = pytest.mark.gpu


def _projection(x, m, l, seed):
    import paper_2509_23472_amd as L
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, l, seed), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t().contiguous()
    q, _ = torch.linalg.qr(y)
    return q @ (q.t().contiguous() @ x.double())


def _eye(k):
    return torch.eye(k, device="cuda", dtype=torch.float64)


BF16 = [(16, 1), (16, 16), (17, 16), (64, 33), (127, 64), (128, 64), (129, 64), (170, 48), (171, 48), (256, 32), (257, 32),
        (200, 17), (511, 16), (512, 9), (513, 16)]


@pytest.mark.parametrize("m,k", BF16)
@pytest.mark.parametrize("decades,n", [(0.0, 192), (2.5, 192), (0.0, 190)])
def test_bf16_site(m, k, decades, n):
    import paper_2509_23472_amd as L
    print("shape", m, n, k, decades, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m * 97 + k)
    x = torch.randn((m, n), generator=g, device="cuda")
    x = (x * 10.0 ** (-decades * torch.arange(n, device="cuda") / n)).bfloat16()
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=3, factor_dtype=torch.float32, status=status)
    assert int(status.item()) == 0
    ud = u.double()
    # float32 storage of U, 2^-24 of an entry: sqrt(k) of them at most
    assert float((ud.t().contiguous() @ ud - _eye(k)).norm()) <= 5e-7 * k ** 0.5 + 1e-6
    # V is formed from the bf16 copy of the basis: 2^-9 of an entry, and the sketch is accumulated in float32
    ref = _projection(x, m, k, 3)
    assert float((ud @ v.double() - ref).norm() / ref.norm()) <= 1e-2
    ub, vb = L.loract_compress(x, k, seed=3)
    assert torch.equal(ub, u.bfloat16()) and torch.equal(vb, v.bfloat16())


@pytest.mark.parametrize("m,k", [(512, 16), (300, 9), (16, 16), (256, 32), (200, 17), (33, 32), (170, 48), (170, 33), (100, 41)])
@pytest.mark.parametrize("n", [192, 190])
def test_second_factorisation(m, k, n):
    import paper_2509_23472_amd as L
    print("shape", m, n, k, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m * 97 + k)
    x = torch.randn((m, n), generator=g, device="cuda")
    x = (x * 10.0 ** (-3.5 * torch.arange(n, device="cuda").clamp(max=k) / k)).bfloat16()
    defect, pivot = first_round(x, k, 3)
    assert defect >= 1e-5, "the first round (accepted up to 1e-6) would do"
    assert pivot >= 8.0, "the unshifted attempt would be abandoned"
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=3, factor_dtype=torch.float32, status=status)
    assert int(status.item()) == 0
    ud = u.double()
    # float32 storage of U, 2^-24 of an entry: sqrt(k) of them at most
    assert float((ud.t().contiguous() @ ud - _eye(k)).norm()) <= 5e-7 * k ** 0.5 + 1e-6
    # V is formed from the bf16 copy of the basis: 2^-9 of an entry; what the float32 accumulation of the sketch loses are
    # directions below 1e-7 of its first, i.e. 3e-4 of X's
    ref = _projection(x, m, k, 3)
    assert float((ud @ v.double() - ref).norm() / ref.norm()) <= 1e-2
    ub, vb = L.loract_compress(x, k, seed=3)
    assert torch.equal(ub, u.bfloat16()) and torch.equal(vb, v.bfloat16())


@pytest.mark.parametrize("m,l", [(m, 16) for m in (16, 17, 127, 128, 129, 256, 257, 512, 513, 1023, 1024, 1025)]
                         + [(300, l) for l in (1, 2, 7, 15)] + [(1024, 3)])
def test_float32_site(m, l):
    import paper_2509_23472_amd as L
    print("shape", m, l, flush=True)
    g = torch.Generator(device="cuda").manual_seed(m + l)
    x = torch.randn((m, 100), generator=g, device="cuda") * 10.0 ** (-2.0 * torch.arange(100, device="cuda") / 100)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for t in (0, 1):                                     # (t = 1: the basis of a power round goes on in float64)
        u, v = L.loract_compress(x, l, seed=5, t=t, status=status)
        assert int(status.item()) == 0
        ud = u.double()
        assert float((ud.t().contiguous() @ ud - _eye(l)).norm()) <= 1e-6      # float32 storage of U
        if t == 0:
            ref = _projection(x, m, l, 5)
            assert float((ud @ v.double() - ref).norm() / ref.norm()) <= 1e-6


@pytest.mark.parametrize("dtype,m,k", [(torch.bfloat16, 256, 24), (torch.bfloat16, 128, 64), (torch.float32, 512, 12)])
def test_dependent_rows(dtype, m, k):
    # half of the rows are zero (padding tokens): the projection onto the independent sampled rows remains
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(k)
    x = torch.randn((m, 128), generator=g, device="cuda").to(dtype)
    x[::2] = 0.0
    u, v = L.loract_compress(x, k, seed=4, factor_dtype=torch.float32)
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 4), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t().contiguous()
    ref = y @ (torch.linalg.pinv(y, rtol=1e-10) @ x.double())
    assert torch.isfinite(u).all() and torch.isfinite(v).all()
    assert float((u.double() @ v.double() - ref).norm() / ref.norm()) <= (1e-2 if dtype == torch.bfloat16 else 1e-5)


@pytest.mark.parametrize("k,small", [(48, True), (49, False), (64, False)])
def test_first_order_finish_where_there_is_one(k, small):
    # from 49 columns on the separate launches finish without a second factorisation, which is faster than one of
    # one workgroup
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(k)
    x = (torch.randn((128, 256), generator=g, device="cuda") * (torch.arange(256, device="cuda") + 1.0) ** -1.5).bfloat16()
    L.loract_profile_begin()
    try:
        L.loract_compress(x, k, seed=3)
        torch.cuda.synchronize()
    finally:
        launches = L.loract_profile_end()
    assert ("ortho_small" in launches) == small
