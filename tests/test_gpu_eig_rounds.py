"""The truncation eigensolver at the edges of its blocks of eight columns and of its two forms (one workgroup up to
order 64), on a spectrum graded over three decades: singular values and vectors against numpy's float64 SVD.
(The sketch has the square of the spectrum and its Gram matrix the fourth power: twelve decades, which float64
resolves to 1e-4 of the smallest pivot; with eight decades of spectrum it would be 32 and the trailing directions,
below 3e-6 of the largest singular value, are dropped by the orthonormalisation before the eigensolver sees them.)

Bounds: the factors are stored in float32 (2^-24 per entry, so a row norm of V to 6e-8) and come from a basis and a
projection that are float64 throughout; a singular value of the sketch's range moves by the sketch's own
rounding, relative to the largest one, 2^-24 at most.  Taken: 1e-6 of the value plus 2e-7 of the largest."""
import numpy as np
import pytest
import torch

from oracle import loract_oracle as orc
from workloads import synth

from gpu_util import to_device, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("l", [3, 8, 9, 16, 17, 31, 48, 49, 63, 66, 72, 80, 81, 128, 176, 272, 273, 304])
def test_singular_values_and_order(l):
    import paper_2509_23472_amd as L
    print("order", l, flush=True)
    m, n, k = 500, 360, max(1, l - 2)
    s = 10.0 ** (-3.0 * np.arange(n) / n)
    w = synth._finish("eigr_%d" % l, synth.spectrum_matrix(m, n, s, 0.0, l), "f32", k, l)
    u, v = L.loract_compress(to_device(w.x, "f32"), k, seed=w.seed, l=l)
    torch.cuda.synchronize()
    u, v = to_host(u), to_host(v)
    x = w.x.astype(np.float64)
    q, _ = np.linalg.qr(x @ x[orc.sample_indices(m, l, w.seed)].T)
    sv = np.linalg.svd(q.T @ x)[1][:k]
    got = np.linalg.norm(v, axis=1)
    assert np.all(np.abs(got - sv) <= 1e-6 * sv + 2e-7 * sv[0]), np.max(np.abs(got - sv) / (1e-6 * sv + 2e-7 * sv[0]))
    assert orc.orthogonality_defect(u) <= 1e-5
    uo, vo = orc.decompose(x, k, seed=w.seed, l=l)
    assert orc.rel_fro(u @ v, uo @ vo) <= 1e-6
