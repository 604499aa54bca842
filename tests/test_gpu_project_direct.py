"""The projection of few rows, one workgroup per output tile: at the row counts where it goes over to shares and partial
tiles, at the edges of the tiles, and the LoRA gradient with its shares of T added by the last product or by a launch."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [64, 65, 448, 511, 512, 513])
@pytest.mark.parametrize("n,k", [(72, 8), (128, 40), (136, 64), (520, 56), (1032, 16), (2048, 64)])
def test_v_is_the_projection(m, n, k):
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    x = torch.randn((m, n), generator=g, device="cuda").bfloat16()
    u, v = L.loract_compress(x, min(k, m // 2), seed=3)
    ref = u.double().t() @ x.double()
    # float32 sums of m products (2^-24 each of |u| |x| <= |x column|) and one bf16 rounding
    bound = 2.0 ** -8 * ref.abs() + m * 2.0 ** -24 * x.double().norm(dim=0)[None, :] * u.double().norm(dim=0)[:, None]
    assert bool(((v.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("m,n_out", [(32, 256), (64, 256), (96, 768), (256, 768), (257, 768), (513, 512)])     # 1 to 34 shares
def test_lora_gradient_of_few_shares(m, n_out):
    import paper_2509_23472_amd as L
    n, k, r = 520, 24, 12
    g = torch.Generator(device="cuda").manual_seed(m)
    u = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    v = torch.randn((k, n), generator=g, device="cuda").bfloat16()
    dy = torch.randn((m, n_out), generator=g, device="cuda").bfloat16()
    b = torch.randn((r, n_out), generator=g, device="cuda").bfloat16()
    da = L.loract_lora_grad(u, v, dy, b, scale=0.5)
    ref = 0.5 * v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t()))
    # G travels as a pair of bf16 values (2^-17 of a value), sums are float32
    assert float((da.double() - ref).norm() / ref.norm()) <= 2.0 ** -15


@pytest.mark.parametrize("m", [1, 63, 256, 257, 320, 321, 384, 385, 448, 449, 512])
@pytest.mark.parametrize("k,r", [(16, 33), (64, 64), (72, 48), (128, 33), (256, 64)])          # 1, 1, 2, 2 and 4 tiles of U^T G
def test_lora_gradient_above_rank_32_of_few_rows(m, k, r):
    import paper_2509_23472_amd as L
    n, n_out = 136, 320
    g = torch.Generator(device="cuda").manual_seed(m + k + r)
    u = torch.randn((m, k), generator=g, device="cuda").bfloat16()
    v = torch.randn((k, n), generator=g, device="cuda").bfloat16()
    dy = torch.randn((m, n_out), generator=g, device="cuda").bfloat16()
    b = torch.randn((r, n_out), generator=g, device="cuda").bfloat16()
    da = L.loract_lora_grad(u, v, dy, b, scale=0.5)
    ref = 0.5 * v.double().t() @ (u.double().t() @ (dy.double() @ b.double().t()))
    # G travels as a pair of bf16 values (2^-17 of a value), sums are float32
    assert float((da.double() - ref).norm() / ref.norm()) <= 2.0 ** -15
