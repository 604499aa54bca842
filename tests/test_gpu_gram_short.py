"""The Gram matrix of more than 64 columns and few rows: rows that end inside a trip of 16, inside a group of four, and inside the
last chunk; odd numbers of 16-column tiles, whose last block holds one; and both sides of the lines between the kernels."""
import pytest

from test_gpu_factor_solve import test_restart_with_dependent_rows as check_restart
from test_gpu_gram_wide import test_basis_of_a_wide_sketch as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,k", [(97, 65), (98, 80), (111, 96), (130, 128), (145, 144), (259, 240), (273, 272), (321, 304), (337, 320),
                                 (513, 100), (1000, 112), (2000, 208), (6143, 80), (6144, 128), (6145, 128), (6145, 80),
                                 (4096, 144), (4096, 256), (4097, 256), (4097, 144), (2048, 257), (2048, 320), (2049, 320)])
def test_basis_of_a_short_wide_sketch(m, k):
    check(m, k)


@pytest.mark.parametrize("m,k", [(300, 80), (1000, 128), (4096, 250), (1000, 272), (2048, 320)])
def test_restart_from_the_copy_that_the_sum_leaves(m, k):
    # (in blocks for the factorisation in registers, in rows above 256 columns)
    check_restart(m, k)
