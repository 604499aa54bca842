"""float32 products with 2^28 rows and a narrow side: tiles of 16 rows would take more threads than a launch can
have.  (About 3 GB; products of single values, so every element is known.)"""
import pytest
import torch

pytestmark = pytest.mark.gpu


def test_reconstruction_with_2_to_the_28_rows():
    import paper_2509_23472_amd as L
    m = (1 << 28) + 3
    u = torch.arange(m, device="cuda", dtype=torch.int32).remainder_(1021).float().view(m, 1)
    v = torch.full((1, 1), 3.0, device="cuda")
    out = torch.full((m, 1), -1.0, device="cuda")
    L.loract_reconstruct(u, v, out=out)
    torch.cuda.synchronize()
    assert torch.equal(out, u.mul_(3.0))
