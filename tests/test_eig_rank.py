"""The order of the eigenvalues is a permutation whatever they are: the eigensolver's last step indexes
with it.  Compiled for the host from the header that the kernels include."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")


@pytest.fixture(scope="module")
def ranks(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    assert cxx, "needs a host C++ compiler"
    d = tmp_path_factory.mktemp("eig_rank")
    src = d / "rank.cpp"
    src.write_text('#include "%s/eig_rank.h"\nextern "C" void ranks(const double* lam, int l, int* out) {\n'
                   "  for (int i = 0; i < l; ++i) out[i] = ej_rank_of(lam, l, i);\n}\n" % CSRC)
    so = d / "rank.so"
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))

    def call(lam):
        lam = np.ascontiguousarray(lam, dtype=np.float64)
        out = np.full(lam.size, -1, dtype=np.int32)
        lib.ranks(lam.ctypes.data_as(ctypes.c_void_p), ctypes.c_int(lam.size), out.ctypes.data_as(ctypes.c_void_p))
        return out
    return call


def test_descending_with_ties_by_index(ranks):
    assert ranks([1.0, 3.0, 3.0, 0.0, 2.0, 0.0]).tolist() == [3, 0, 1, 4, 2, 5]


@pytest.mark.parametrize("l", [1, 2, 96, 97, 128, 320])
@pytest.mark.parametrize("kind", ["all_nan", "some_nan", "infinite", "any_bits"])
def test_always_a_permutation(ranks, l, kind):
    rng = np.random.default_rng(l)
    lam = rng.exponential(size=l)
    if kind == "all_nan":
        lam[:] = np.nan
    elif kind == "some_nan":
        lam[rng.random(l) < 0.9] = np.nan
    elif kind == "infinite":
        lam[rng.random(l) < 0.5] = np.inf
    else:                                    # what a work buffer held before
        lam = rng.integers(0, 2 ** 64, size=l, dtype=np.uint64).view(np.float64)
    r = ranks(lam)
    assert sorted(r.tolist()) == list(range(l))
    # what is kept first are the positive values, in descending order
    order = np.argsort(r)
    kept = lam[order][: int(np.sum(lam > 0))]
    assert np.all(kept > 0) and np.all(kept[:-1] >= kept[1:])
