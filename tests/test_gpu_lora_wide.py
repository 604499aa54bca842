"""Last product of the LoRA gradient on either side of the line between workgroups of 64 and of 32 columns of V, at ragged numbers
of columns and rows of V, for every padded LoRA rank and for shares of T, against float64 products."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("r", [7, 16, 25, 40, 64])
@pytest.mark.parametrize("n,k", [(8, 8), (40, 72), (8128, 136), (8136, 8), (8200, 72), (11008, 256), (8264, 320),
                                 (32704, 72), (32712, 136), (32776, 264)])
def test_columns_of_v(n, k, r):
    import paper_2509_23472_amd as L
    m, n_out = 96, 128
    g = torch.Generator(device="cuda").manual_seed(n + k + r)

    def rnd(*shape):
        return torch.randn(shape, generator=g, device="cuda").bfloat16()

    u, v, dy, b = rnd(m, k), rnd(k, n), rnd(m, n_out), rnd(r, n_out)
    out = torch.full((n + 8, r), 7.0, device="cuda")
    got = L.loract_lora_grad(u, v, dy, b, scale=0.5, out=out[:n])
    ref = 0.5 * (v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t())))
    assert (out[n:] == 7).all()
    # G as a bf16 pair (2^-17 of a value) and fp32 sums of at most 320 terms of either sign
    assert float((got.double() - ref).norm() / ref.norm()) <= 3e-5
    assert torch.equal(got.clone(), L.loract_lora_grad(u, v, dy, b, scale=0.5))
