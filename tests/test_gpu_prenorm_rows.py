"""The pre-norm kernel that keeps its rows in registers, at the edges of its row widths, against
float64 arithmetic; and its quotient A / gamma where gamma is extreme."""
import numpy as np
import pytest
import torch

from oracle import loract_oracle as orc

from gpu_util import to_host

pytestmark = pytest.mark.gpu

# pieces per row on either side of every width: one wave (64, 128 pieces), four waves (256 c pieces,
# c = 1, 2, 3, 4, 6, 8, 12), one piece past the widest (two sweeps)
PIECES = [1, 64, 65, 128, 129, 256, 257, 512, 513, 769, 1025, 1537, 2049, 3072, 3073]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("pieces", PIECES)
def test_row_widths(dtype, pieces):
    import paper_2509_23472_amd as L
    n = pieces * (8 if dtype == torch.bfloat16 else 4)
    m = 4099 if pieces <= 2 else (37 if pieces % 2 else 5)     # more rows than one trip of the grid; odd counts
    g = torch.Generator(device="cuda").manual_seed(pieces)
    x = torch.randn((m, n), generator=g, device="cuda").to(dtype)
    grad = torch.randn((m, n), generator=g, device="cuda").to(dtype)
    gamma = 0.5 + torch.rand((n,), generator=g, device="cuda")
    a, rms = L.loract_prenorm_forward(x, gamma, eps=1e-5)
    dx = L.loract_prenorm_backward(a, rms, gamma, grad)
    a_ref, rms_ref = orc.prenorm_forward(to_host(x), to_host(gamma), 1e-5)
    dx_ref = orc.prenorm_backward(to_host(a), to_host(rms), to_host(gamma), to_host(grad))
    # fp32 sums of n terms, then one rounding of the result: 2^-8 of a value for bf16
    one = 2.0 ** -7.95 if dtype == torch.bfloat16 else 4e-6
    assert np.max(np.abs(to_host(rms) - rms_ref) / rms_ref) <= 2e-6
    assert np.max(np.abs(to_host(a) - a_ref) / np.maximum(np.abs(a_ref), 1e-3)) <= one
    # the difference of the backward step may cancel: relative to the larger of its two terms (~ 1 / rms)
    assert np.max(np.abs(to_host(dx) - dx_ref)) <= one * max(1.0, np.max(np.abs(dx_ref)))


def test_quotient_by_extreme_gamma():
    import paper_2509_23472_amd as L
    m, n = 6, 2048
    g = torch.Generator(device="cuda").manual_seed(7)
    a = torch.randn((m, n), generator=g, device="cuda")
    grad = torch.randn((m, n), generator=g, device="cuda")
    gamma = torch.ones((n,), device="cuda")
    gamma[3], gamma[700], gamma[1301], gamma[2047] = 2.0 ** -120, 2.0 ** 120, 1e-30, -3.0
    rms = 0.5 + torch.rand((m,), generator=g, device="cuda")
    dx = L.loract_prenorm_backward(a, rms, gamma, grad)
    inner = (a * grad).double().sum(1, keepdim=True) / n
    want = (grad.double() * gamma.double() - a.double() / gamma.double() * inner) / rms.double()[:, None]
    # 1e-5: fp32 sum of 2048 products of which much cancels, on top of a few roundings
    scale = (a.double() / gamma.double()).abs() * (a * grad).double().abs().sum(1, keepdim=True) / n + (grad * gamma).double().abs()
    assert torch.all((dx.double() - want).abs() <= 1e-5 * scale / rms.double()[:, None] + 1e-37)
