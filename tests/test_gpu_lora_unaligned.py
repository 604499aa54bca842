"""LoRA gradient of a dY whose rows are no multiple of 64 columns, on either side of the number of columns from which K is split, with few
rows (many splits fit) and many (the room for the shares decides), against float64 products."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [4, 33, 64])
@pytest.mark.parametrize("m,n_out", [(96, 526), (3001, 1023), (96, 1025), (3001, 1030), (12000, 2050), (33000, 1537)])
def test_unaligned_gradient(m, n_out, r):
    import paper_2509_23472_amd as L
    n, k = 136, 24
    g = torch.Generator(device="cuda").manual_seed(m + n_out + r)

    def rnd(*shape):
        return torch.randn(shape, generator=g, device="cuda").bfloat16()

    u, v, dy, b = rnd(m, k), rnd(k, n), rnd(m, n_out), rnd(r, n_out)
    got = L.loract_lora_grad(u, v, dy, b, scale=0.5)
    ref = 0.5 * (v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t())))
    # G in fp32 (sums of at most 2050 terms of either sign: sqrt(2050) 2^-24 = 2.7e-6 of a value), the rest in float64, a float32 result
    assert float((got.double() - ref).norm() / ref.norm()) <= 1e-5
    assert torch.equal(got.clone(), L.loract_lora_grad(u, v, dy, b, scale=0.5))
