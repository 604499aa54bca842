"""The first-order finish of the orthonormalisation at widths that are no multiple of 64 columns, where the last slab of its
contraction is in part past the matrix: the basis of the sketch, its orthogonality and U V against the oracle.  Power-law
spectra put ||Q1^T Q1 - I|| between the 1e-6 at which Q1 is the answer and the 4e-3 up to which the step is taken."""
import numpy as np
import pytest
import torch

from workloads import synth

from gpu_util import check_compress_parity, first_round, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(130, 640, 65), (700, 640, 72), (999, 832, 80), (3001, 1030, 100), (515, 1024, 112), (8200, 1280, 88),
                                   (1500, 1440, 104), (4500, 1536, 140)])
def test_basis_at_widths_between(m, n, k):
    import paper_2509_23472_amd as L
    s = (np.arange(min(m, n)) + 1.0) ** -1.5
    w = synth._finish("finish_%dx%d_k%d" % (m, n, k), synth.spectrum_matrix(m, n, s, 1e-3, k), "bf16", k, k)
    x = to_device(w.x, "bf16")
    e = first_round(x, k, w.seed)[0]
    print(m, n, k, "E", e, flush=True)
    assert e > 1e-6                                          # (140 columns may lie on either side of the upper line)
    status = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    u, v = L.loract_compress(x, k, seed=w.seed, status=status)
    check_compress_parity(w, u, v, L.loract_reconstruct(u, v))
    assert int(status.item()) == 0
