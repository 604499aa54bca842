"""The adaptive rank at orders above 96, where the eigenvalues are ranked and the columns past the rank
cleared by a kernel of their own (several workgroups, each of which ranks for itself): the same checks as
at the smaller orders."""
import pytest

from test_gpu_adaptive import test_adaptive_rank_matches_oracle as check_adaptive_rank

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,m,n,k_max,l,decay", [("bf16", 1500, 512, 90, 97, 0.9), ("f32", 640, 300, 80, 97, 0.9),
                                                      ("bf16", 2048, 640, 128, 136, 0.95), ("f32", 700, 400, 136, 136, 0.95),
                                                      ("bf16", 1600, 768, 200, 264, 0.97), ("f32", 900, 512, 256, 264, 0.97)])
def test_adaptive_rank_of_a_large_sketch(dtype, m, n, k_max, l, decay):
    check_adaptive_rank(dtype, m, n, k_max, l, decay)
