"""The projection's work split: whether output tiles of few slabs go straight to V is decided the way that was the faster
one where both were timed.  The rules are compiled for the host from the header that kernels and launcher include."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")
MODEL = r'''
#include "%s/project_plan.h"
extern "C" int direct(long long slabs, long long tiles) { return project_goes_direct(slabs, tiles); }
'''


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("project_plan")
    (d / "m.cpp").write_text(MODEL % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    so = ctypes.CDLL(str(d / "m.so"))
    so.direct.argtypes = [ctypes.c_longlong] * 2
    return so


@pytest.mark.parametrize("slabs,tiles,direct", [
    (1, 1, 1), (4, 1, 1), (5, 2, 1), (5, 64, 1), (6, 2, 1), (6, 4, 1), (6, 64, 1), (7, 4, 1), (7, 16, 1), (7, 64, 1),
    (6, 1, 0), (7, 1, 0), (7, 2, 0), (8, 1, 0), (8, 2, 0), (8, 4, 0), (8, 16, 0), (9, 1, 0), (9, 64, 0), (200, 4, 0)])
def test_the_faster_way(lib, slabs, tiles, direct):
    assert lib.direct(slabs, tiles) == direct
