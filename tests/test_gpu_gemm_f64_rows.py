"""Float32 products large enough for 64-wide tiles: whole wave tiles leave as rows, the rest element by element, whatever
the pitch and the alignment of the output."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(4096, 512, 32), (4097, 513, 5), (4127, 543, 17), (4128, 545, 16), (4095, 511, 33), (20000, 130, 3)])
@pytest.mark.parametrize("pad", [0, 1, 6])
def test_float32_reconstruction(m, n, k, pad):
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    u = torch.randn((m, k), generator=g, device="cuda")
    v = torch.randn((k, n), generator=g, device="cuda")
    buf = torch.full((m, n + pad), 7.0, device="cuda")
    out = buf[:, pad // 2:pad // 2 + n]
    L.loract_reconstruct(u, v, out=out)
    ref = u.double() @ v.double()
    # float64 sums, one float32 rounding
    assert bool(((out.double() - ref).abs() <= 2.0 ** -24 * ref.abs() + 1e-13 * k).all())
    assert bool((buf[:, :pad // 2] == 7.0).all()) and bool((buf[:, pad // 2 + n:] == 7.0).all())
