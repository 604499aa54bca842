"""The factorisation at 257 to 272 columns, whose first block row waits in LDS, beside its neighbours on either side: bases of
graded spectra, a second round that has to factor, a restart with the shift, and the factorisation of a truncation."""
import numpy as np
import pytest
import torch

from test_gpu_factor_solve import test_basis as check_basis
from test_gpu_factor_solve import test_restart_of_a_factorisation_of_its_own as check_restart
from test_gpu_factor_solve import test_second_round as check_second_round
from test_gpu_eig_rounds import test_singular_values_and_order as check_truncation

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [256, 257, 264, 272, 273])
@pytest.mark.parametrize("m,decades", [(700, 0.5), (4095, 2.0), (16321, 1.0), (40000, 1.0)])
def test_basis_of(m, k, decades):
    check_basis(m, k, decades)


@pytest.mark.parametrize("m,k", [(705, 257), (4095, 264), (16320, 272)])
def test_second_round_of(m, k):
    check_second_round(m, k)


@pytest.mark.parametrize("m,k", [(1000, 264), (33000, 257), (33000, 272)])
def test_restart_of(m, k):
    check_restart(m, k)


@pytest.mark.parametrize("l", [257, 264, 265, 272])
def test_truncation_of(l):
    check_truncation(l)
