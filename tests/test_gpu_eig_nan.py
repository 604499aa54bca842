"""An activation with a NaN or an infinity through the truncation: every eigenvalue is then NaN, the order of the
columns still has to be a permutation (its entries index memory), the outputs say that they are not
finite, and the next call is not affected."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("l", [40, 96, 97, 136, 264])
def test_not_finite_activation(l, dtype, bad):
    import paper_2509_23472_amd as L
    print("order", l, dtype, bad, flush=True)
    m, n, k = 640, 384, l - 8
    g = torch.Generator(device="cuda").manual_seed(l)
    x = torch.randn((m, n), generator=g, device="cuda").to(dtype)
    broken = x.clone()
    broken[17, 5] = bad
    clean = L.loract_compress(x, k, l=l, seed=3)
    u, v = L.loract_compress(broken, k, l=l, seed=3)
    ua, va, rank = L.loract_compress_adaptive(broken, k, 0.9, l=l, seed=3)
    again = L.loract_compress(x, k, l=l, seed=3)
    torch.cuda.synchronize()
    assert not torch.isfinite(u).all() and not torch.isfinite(v).all()
    assert not torch.isfinite(ua).all() and not torch.isfinite(va).all()
    assert int(rank.item()) == k            # no count reaches a share of a sum that is NaN: all that is allowed
    assert torch.equal(clean[0], again[0]) and torch.equal(clean[1], again[1])
