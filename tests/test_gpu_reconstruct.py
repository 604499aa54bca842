"""Xhat = U V from bf16 factors at the edges of its tiles (64 rows, 256 or 128 columns, K steps of 16, slabs of 64), in both
forms of the kernel and with either kind of store, against the product in float64.  LDS is left full of NaN first: padding that no copy
writes must not reach a result.

Tolerance: products of bf16 values are exact in float32 and are added in float32 in steps of the matrix instruction, so an
element is off by at most k 2^-24 sum |u| |v| before it is rounded to bf16, and half a unit of that afterwards."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _check(m, n, k, pad=8):
    import paper_2509_23472_amd as L
    nan = torch.full((64, 256), float("nan"), dtype=torch.bfloat16, device="cuda")
    L.loract_reconstruct(nan.repeat(64, 1), nan.t().contiguous().repeat(1, 64))          # every CU's LDS
    g = torch.Generator(device="cuda").manual_seed(m * 7 + n * 3 + k)
    u = torch.randn((m, k), generator=g, device="cuda").to(torch.bfloat16)
    v = torch.randn((k, n), generator=g, device="cuda").to(torch.bfloat16)
    big = torch.full((m + 1, n + pad), 7.0, dtype=torch.bfloat16, device="cuda")
    L.loract_reconstruct(u, v, out=big[:m, :n])
    assert (big[m:] == 7).all() and (big[:, n:] == 7).all()
    ids = torch.arange(0, n, 512, device="cuda")
    for c0 in ids.tolist():
        c1 = min(n, c0 + 512)
        want = u.double() @ v[:, c0:c1].double()
        size = u.double().abs() @ v[:, c0:c1].double().abs()
        bound = k * 2.0 ** -24 * size
        bound = bound + (want.abs() + bound) * 2.0 ** -8
        off = (big[:m, c0:c1].double() - want).abs()
        assert (off <= bound).all(), (m, n, k, c0, float((off - bound).max()))


@pytest.mark.parametrize("k", [8, 24, 64, 72, 128, 136, 144, 200, 248, 256, 264, 320])
@pytest.mark.parametrize("m,n", [(1, 8), (63, 248), (64, 256), (65, 264), (449, 1032)])
def test_few_tiles(m, n, k):
    _check(m, n, k)


@pytest.mark.parametrize("k", [8, 16, 40, 64, 96, 128, 184, 256])
@pytest.mark.parametrize("m,n", [(4033, 1032), (16321, 264), (130, 25608), (7000, 2568)])
def test_shares_of_several_tiles(m, n, k):
    _check(m, n, k)


# (wide tiles at the other K steps above rank 128, narrow ones that share a workgroup, the last sizes of either form)
@pytest.mark.parametrize("m,n,k", [(4033, 1032, 136), (4033, 1032, 160), (4033, 1032, 176), (4033, 1032, 208), (4033, 1032, 224), (4033, 1032, 232),
                                   (32769, 120, 8), (32769, 128, 128), (8192, 256, 248), (8193, 256, 248)])
def test_either_form(m, n, k):
    _check(m, n, k)


# non-temporal stores: from 128 MB, where rows are whole lines of 128 bytes (n + pad a multiple of 64); the last size before and the first one from there
@pytest.mark.parametrize("mb,n,k", [(128, 4104, 32), (128, 4096, 128), (128, 4096, 136), (128, 11272, 256), (128, 11264, 264)])
@pytest.mark.parametrize("past", [0, 1])
@pytest.mark.parametrize("lines", [0, 1])
def test_past_the_cache(mb, n, k, past, lines):
    m = ((mb << 20) - 1) // (2 * n) + past
    assert (m * n * 2 >= mb << 20) == bool(past)
    _check(m, n, k, 64 - n % 64 if lines else 8)
