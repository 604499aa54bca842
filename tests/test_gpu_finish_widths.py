"""Bases of widths that are no multiple of 64 columns, where round 2 of the orthonormalisation factors and solves a second time: the basis of the
sketch and U V against the oracle, and that bf16 factors are no less accurate than float32 ones before they are rounded.  Power-law
spectra put ||Q1^T Q1 - I|| above the 1e-6 at which Q1 is the answer."""
import numpy as np
import pytest
import torch

from workloads import synth

from gpu_util import check_compress_parity, first_round, to_device

pytestmark = pytest.mark.gpu

SIZES = [(130, 640, 65), (700, 640, 72), (999, 832, 80), (3001, 1030, 100), (515, 1024, 112), (8200, 1280, 88), (1500, 1440, 104),
         (4500, 1536, 140), (8200, 1536, 176), (900, 1536, 272), (1200, 1536, 300)]


def _site(m, n, k):
    s = (np.arange(min(m, n)) + 1.0) ** -1.5
    w = synth._finish("finish_%dx%d_k%d" % (m, n, k), synth.spectrum_matrix(m, n, s, 1e-3, k), "bf16", k, k)
    x = to_device(w.x, "bf16")
    e = first_round(x, k, w.seed)[0]
    print(m, n, k, "E", e, flush=True)
    assert e > 1e-6
    return w, x


@pytest.mark.parametrize("m,n,k", SIZES[:8])
def test_basis_at_widths_between(m, n, k):
    import paper_2509_23472_amd as L
    w, x = _site(m, n, k)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=w.seed, status=status)
    check_compress_parity(w, u, v, L.loract_reconstruct(u, v))
    assert int(status.item()) == 0


@pytest.mark.parametrize("t", [0, 1])
@pytest.mark.parametrize("m,n,k", SIZES)
def test_bf16_factors_are_float32_factors_rounded(m, n, k, t):
    import paper_2509_23472_amd as L
    w, x = _site(m, n, k)
    u, v = L.loract_compress(x, k, t=t, seed=w.seed)
    uf, vf = L.loract_compress(x, k, t=t, seed=w.seed, factor_dtype=torch.float32)
    assert torch.equal(u, uf.bfloat16()) and torch.equal(v, vf.bfloat16())
    if t == 0:
        ud = uf.double()
        # (the solve is in float64; a value of U is rounded to float32, 2^-24 of it, and k of them meet in an entry)
        assert float((ud.t().contiguous() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm()) <= 2.0 ** -23 * k ** 0.5


@pytest.mark.parametrize("m,k", [(m, k) for m in (707, 12611, 40001) for k in (7, 20, 48, 72, 100, 112, 176, 240, 264)] + [(262144, 16), (262145, 16)])
def test_accepted_basis_in_either_type(m, k):
    """Flat spectra: Q1 is the answer, converted by the launch that finds this or, of more than 4M values or 112 columns, by one of its own."""
    import paper_2509_23472_amd as L
    g = torch.Generator(device="cuda").manual_seed(m + k)
    x = torch.randn((m, 640), generator=g, device="cuda").bfloat16()
    e = first_round(x, k, 5)[0]
    print(m, k, "E", e, flush=True)
    assert e <= 1e-6
    u, v = L.loract_compress(x, k, seed=5)
    uf, vf = L.loract_compress(x, k, seed=5, factor_dtype=torch.float32)
    assert torch.equal(u, uf.bfloat16()) and torch.equal(v, vf.bfloat16())
    ud = uf.double()
    assert float((ud.t().contiguous() @ ud - torch.eye(k, device="cuda", dtype=torch.float64)).norm()) <= 1e-6 + 2.0 ** -23 * k ** 0.5
