"""LoRA gradient on given bf16 factors against float64 products: row tiles of 32, column slabs of 256,
shares that begin and end inside a tile, both padded LoRA ranks of the one-pass route and one above."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # m, n, k, n_out, r
    (1, 8, 8, 64, 1),               # one row, one short slab
    (31, 264, 24, 320, 16),         # rows and the last slab partly filled
    (33, 40, 72, 192, 17),          # second row tile with one row; rank padded to 32
    (197, 768, 32, 768, 16),        # one slab per workgroup
    (2050, 136, 320, 1088, 32),     # widest U; tiles cut between workgroups
    (8229, 96, 136, 256, 5),        # more tiles than workgroups, one slab each: U two tiles ahead is refused
    (300, 1000, 200, 4096, 12),     # few shares fit: long walks inside a tile
    (1000, 72, 64, 512, 33),        # above the one-pass ranks
]


@pytest.mark.parametrize("m,n,k,n_out,r", CASES)
def test_gradient_of_given_factors(m, n, k, n_out, r):
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(m + r)

    def rnd(*shape):
        return torch.randn(shape, generator=g, device="cuda").bfloat16()

    u, v, dy, b = rnd(m, k), rnd(k, n), rnd(m, n_out), rnd(r, n_out)
    got = L.loract_lora_grad(u, v, dy, b, scale=0.5)
    ref = 0.5 * (v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t())))
    err = float((got.double() - ref).norm() / ref.norm())
    # G as a bf16 pair (2^-17 of a value) and fp32 sums of at most 4096 terms of either sign
    assert err <= 3e-5, err
    assert torch.equal(got, L.loract_lora_grad(u, v, dy, b, scale=0.5))      # fixed order of all sums


def test_rows_past_the_end_do_not_leak():
    # an infinity in the last row of dY makes its own contributions infinite or NaN and nothing else:
    # the tile's padding rows repeat that row and have to be dropped
    import paper_2509_23472_amd as L
    m, n, k, n_out, r = 37, 64, 16, 64, 4
    g = torch.Generator(device="cuda").manual_seed(3)
    u = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    v = torch.randn((k, n), generator=g, device="cuda").bfloat16()
    dy = torch.randn((m, n_out), generator=g, device="cuda").bfloat16()
    b = torch.zeros((r, n_out), device="cuda").bfloat16()
    b[0, 0], b[1, 1], b[2, 2], b[3, 3] = 1.0, 1.0, 1.0, 1.0
    dy[m - 1, 2] = float("inf")
    got = L.loract_lora_grad(u, v, dy, b)
    dy[m - 1, 2] = 0.0
    clean = L.loract_lora_grad(u, v, dy, b)
    assert torch.equal(got[:, [0, 1, 3]].isnan(), torch.ones_like(got[:, [0, 1, 3]], dtype=torch.bool))  # inf * 0 in G
    assert not got[:, 2].isfinite().any()
    assert clean.isfinite().all()


@pytest.mark.parametrize("m,n_out,r", [(1, 64, 1), (130, 192, 16), (1000, 256, 17), (4099, 1024, 64), (515, 72, 9)])
def test_gradient_of_float32_factors(m, n_out, r):
    # aligned and unaligned (72 columns) bf16 dY with float32 factors
    import paper_2509_23472_amd as L
    n, k = 100, 24
    g = torch.Generator(device="cuda").manual_seed(m + r)
    u = torch.randn((m, k), generator=g, device="cuda")
    v = torch.randn((k, n), generator=g, device="cuda")
    dy = torch.randn((m, n_out), generator=g, device="cuda").bfloat16()
    b = torch.randn((r, n_out), generator=g, device="cuda").bfloat16()
    got = L.loract_lora_grad(u, v, dy, b, scale=2.0)
    ref = 2.0 * (v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t())))
    # fp32 sums of up to 1024 products in G, float64 from there on
    assert float((got.double() - ref).norm() / ref.norm()) <= 5e-6
