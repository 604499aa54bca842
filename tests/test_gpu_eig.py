"""GPU parity of the truncation eigensolver at the edges of its forms: orders that fill their lanes and
that do not, odd ones, one workgroup (up to 96) and blocks of columns (above, with full and with
padded blocks), and a semidefinite matrix.  Reached through loract_compress with more sampled rows
than the rank; float32 sites, so that what is compared is the eigensolver and not bf16 rounding.

Bounds: U V against the oracle's to the 1e-4 of the float32 truncation cases; U^T U - I to 1e-5
(float32 storage of k <= 320 columns: 2^-24 sqrt(k) with slack); V = diag(s) W^T with orthonormal
rows, so V V^T is diagonal and descending to float32 storage of V, 2^-23 sqrt(n) ~ 2.4e-6 of the
product of the rows' norms, 2e-5 taken."""
import numpy as np
import pytest
import torch

from oracle import loract_oracle as orc
from workloads import synth

from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [2, 15, 32, 33, 64, 65, 96, 97, 112, 129, 160, 161, 264, 288, 320])
def test_truncation_at_the_orders_where_the_form_changes(l):
    import paper_2509_23472_amd as L
    print("order", l, flush=True)
    m, n, k = 700, 400, max(1, l - 3)
    s = np.exp(-np.arange(n) / 48.0)
    w = synth._finish("eig_%d" % l, synth.spectrum_matrix(m, n, s, 1e-3, l), "f32", k, l)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(to_device(w.x, "f32"), k, seed=w.seed, l=l, status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == 0
    u, v = to_host(u), to_host(v)
    uo, vo = orc.decompose(w.x.astype(np.float64), k, seed=w.seed, l=l)
    assert orc.rel_fro(u @ v, uo @ vo) <= 1e-4
    assert orc.orthogonality_defect(u) <= 1e-5
    g = v @ v.T
    d = np.sqrt(np.diag(g))
    assert np.all(np.diff(d) <= 1e-6 * d[:-1])
    off = (g - np.diag(np.diag(g))) / np.outer(d, d)
    assert np.max(np.abs(off)) <= 2e-5, np.max(np.abs(off))


@pytest.mark.parametrize("l", [40, 120])
def test_truncation_of_a_semidefinite_factor(l):
    # rank 8 and l sampled rows: all but 8 eigenvalues are rounding; the product is still X
    import paper_2509_23472_amd as L
    print("order", l, flush=True)
    w = synth.exact_rank(300, 200, 8, seed=l, dtype="f32")
    u, v = L.loract_compress(to_device(w.x, "f32"), 16, seed=w.seed, l=l)
    torch.cuda.synchronize()
    u, v = to_host(u), to_host(v)
    assert np.all(np.isfinite(u)) and np.all(np.isfinite(v))
    assert orc.rel_fro(u @ v, w.x.astype(np.float64)) <= 1e-5


def test_block_form_on_three_streams_at_once():
    # workgroups that wait for each other, from three launches that share the GPU: same bits as alone
    import paper_2509_23472_amd as L
    xs = [to_device(synth.round_to_bf16(np.random.default_rng(i).standard_normal((2048, 512)).astype(np.float32)), "bf16")
          for i in range(3)]
    alone = [[t.clone() for t in L.loract_compress(x, 120, l=128, seed=1)] for x in xs]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in xs]
    got = []
    for x, s in zip(xs, streams):
        with torch.cuda.stream(s):
            got.append(L.loract_compress(x, 120, l=128, seed=1))
    torch.cuda.synchronize()
    for (u, v), (uo, vo) in zip(got, alone):
        assert torch.equal(u, uo) and torch.equal(v, vo)
