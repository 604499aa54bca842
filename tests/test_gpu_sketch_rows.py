"""The sketch on tiles of 64 rows (few of those of 128 rows, at most 32 sampled rows) at their edges, as sketch, in a power round and as
the product dY B^T, against float64 sums."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [32, 63, 64, 65, 129, 4095, 16384, 16385])
@pytest.mark.parametrize("n,k,t", [(64, 8, 0), (448, 17, 0), (768, 32, 1), (192, 33, 0)])
def test_basis_and_projection(m, n, k, t):
    import paper_2509_23472_amd as L
    k = min(k, m // 2)
    g = torch.Generator(device="cuda").manual_seed(m + n)
    x = torch.randn((m, n), generator=g, device="cuda") * 10.0 ** (-1.0 * torch.arange(n, device="cuda") / n)
    x = x.bfloat16()
    u, v = L.loract_compress(x, k, t=t, seed=5, factor_dtype=torch.float32)
    idx = torch.from_numpy(np.asarray(L.loract_sample_indices(m, k, 5), dtype=np.int64)).cuda()
    y = x.double() @ x[idx].double().t().contiguous()
    for _ in range(t):
        q, _ = torch.linalg.qr(y)
        y = x.double() @ (x.double().t().contiguous() @ q)
    q, _ = torch.linalg.qr(y)
    ref = q @ (q.t().contiguous() @ x.double())
    # V is formed from the bf16 copy of the basis (2^-9 of an entry), a power round from bf16 factors besides
    assert float((u.double() @ v.double() - ref).norm() / ref.norm()) <= 1e-2
    assert float((u.double().t().contiguous() @ u.double() - torch.eye(k, device="cuda", dtype=torch.float64)).norm()) <= 1e-3


@pytest.mark.parametrize("m,n_out", [(63, 64), (65, 640), (4100, 1024)])
def test_product_with_float32_factors(m, n_out):
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(m)
    u, v = torch.randn((m, 24), generator=g, device="cuda"), torch.randn((24, 96), generator=g, device="cuda")
    dy, b = torch.randn((m, n_out), generator=g, device="cuda").bfloat16(), torch.randn((9, n_out), generator=g, device="cuda").bfloat16()
    got = L.loract_lora_grad(u, v, dy, b)
    ref = v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t()))
    assert float((got.double() - ref).norm() / ref.norm()) <= 5e-6


@pytest.mark.parametrize("n_out,r", [(128, 7), (512, 16), (768, 32), (960, 25)])
def test_sums_of_a_row_do_not_depend_on_the_tile(n_out, r):
    """128 tiles of 128 rows are taken as 256 of 64, 129 are not: the same rows of dY B^T, bit for bit.  U picks rows and V is the identity, so
    that a row of dA is a row of the product."""
    import paper_2509_23472_amd as L
    m, k = 128 * 128, 256
    g = torch.Generator(device="cuda").manual_seed(n_out)
    dy, b = torch.randn((m + 1, n_out), generator=g, device="cuda").bfloat16(), torch.randn((r, n_out), generator=g, device="cuda").bfloat16()
    u = torch.zeros((m + 1, k), device="cuda")
    at = 64 * torch.arange(k, device="cuda") + (7 * torch.arange(k, device="cuda")) % 64
    u[at, torch.arange(k, device="cuda")] = 1.0
    v = torch.eye(k, device="cuda")
    got = L.loract_lora_grad(u[:m], v, dy[:m], b)
    ref = L.loract_lora_grad(u, v, dy, b)
    assert torch.equal(got, ref)
    want = dy[at].double() @ b.double().t()
    # (sums of n_out products of either sign in float32)
    assert float((got.double() - want).norm() / want.norm()) <= 2e-6
