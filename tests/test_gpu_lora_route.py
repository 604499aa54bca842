"""LoRA gradient of a dY too large for the caches, on both sides of the line between the one pass over dY and
the two products, against float64 products formed on the GPU in row blocks."""
import pytest
import torch

pytestmark = pytest.mark.gpu

CASES = [
    # m, n, k, n_out, r: just past the size that stays cached (ragged row tile), one pass
    (24600, 136, 256, 4096, 16),
    (25601, 72, 24, 4096, 32),
    # two products: full rounds of workgroups, long rows, LoRA ranks of one and two tiles (one of them filled up)
    (65536, 264, 64, 4096, 32),
    (25600, 40, 200, 16384, 16),
    (10241, 64, 320, 28672, 17),
    (32768, 96, 128, 11008, 5),
]


def _case(m, n, k, n_out, r):
    g = torch.Generator(device="cuda").manual_seed(m + r)

    def rnd(*shape):
        out = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        step = max(1, (1 << 26) // shape[-1])
        for i in range(0, shape[0], step):
            part = out[i:i + step]
            part.copy_(torch.randn(part.shape, generator=g, device="cuda"))
        return out

    return rnd(m, k), rnd(k, n), rnd(m, n_out), rnd(r, n_out)


@pytest.mark.parametrize("m,n,k,n_out,r", CASES)
def test_gradient_of_a_large_dy(m, n, k, n_out, r):
    import paper_2509_23472_amd as L
    print("case", m, n, k, n_out, r, flush=True)
    u, v, dy, b = _case(m, n, k, n_out, r)
    got = L.loract_lora_grad(u, v, dy, b, scale=0.5)
    t = torch.zeros((k, r), dtype=torch.float64, device="cuda")
    bt = b.double().t().contiguous()
    for i in range(0, m, 4096):
        t += u[i:i + 4096].double().t().contiguous() @ (dy[i:i + 4096].double() @ bt)
    ref = 0.5 * (v.double().t().contiguous() @ t)
    err = float((got.double() - ref).norm() / ref.norm())
    # G as a bf16 pair (2^-17 of a value) and fp32 sums of at most 65536 terms of either sign, in a few hundred parts
    assert err <= 3e-5, err
    assert torch.equal(got, L.loract_lora_grad(u, v, dy, b, scale=0.5))      # fixed order of all sums


def test_the_slower_route_is_not_taken():
    # 25600 x 16384 at LoRA rank 32: two products 154 us, one pass 206; rank 40 always takes the two products
    import paper_2509_23472_amd as L
    us = {}
    u, v, dy, b = _case(25600, 256, 64, 16384, 40)
    for r in (32, 40):
        br = b[:r].contiguous()
        L.loract_lora_grad(u, v, dy, br)
        best = float("inf")
        for _ in range(8):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for _ in range(10):
                L.loract_lora_grad(u, v, dy, br)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, e0.elapsed_time(e1) * 100.0)
        us[r] = best
    print(us)
    assert us[32] <= 1.1 * us[40], us
