"""Which form of the reconstruction takes a result, and with which kind of store: on either side of the lines that were timed.  The rules are compiled for the host from the
header that the launcher includes."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("recon_plan")
    (d / "m.cpp").write_text('#include "%s/recon_plan.h"\nextern "C" int narrow(long long m, long long n, int k) '
                             "{ return reconstruct_narrow_wins(m, n, k); }\n"
                             'extern "C" int streams(long long m, long long n, int lines) { return reconstruct_streams_out(m, n, lines); }\n' % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    so = ctypes.CDLL(str(d / "m.so"))
    so.narrow.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    so.streams.argtypes = [ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    return so


# (pairs more than 3 % apart)
@pytest.mark.parametrize("m,n,k,narrow", [
    (64, 64, 16, 1), (200, 768, 32, 1), (200, 768, 128, 1), (200, 4096, 16, 1), (1024, 2048, 32, 1), (512, 256, 144, 1), (512, 768, 256, 1),
    (2048, 768, 160, 1), (2048, 1024, 256, 1), (8192, 256, 256, 1), (4096, 512, 192, 1),
    (32768, 64, 8, 1), (32768, 128, 32, 1), (32768, 128, 128, 1), (16384, 64, 32, 1),
    (4096, 768, 48, 0), (4096, 768, 128, 0), (4096, 768, 192, 0), (8192, 512, 64, 0), (1024, 4096, 96, 0), (12608, 256, 256, 0),
    (8192, 768, 16, 0), (8192, 768, 32, 0), (12608, 512, 16, 0), (16384, 768, 64, 0), (4096, 2048, 128, 0), (8192, 1024, 256, 0),
    (32768, 1024, 32, 0), (32768, 256, 128, 0), (8192, 4096, 64, 0), (12608, 4096, 128, 0)])
def test_the_faster_form(plan, m, n, k, narrow):
    assert plan.narrow(m, n, k) == narrow


def test_rows_that_are_no_whole_lines_are_stored_plainly(plan):
    for m, n in ((50000, 3000), (65536, 4100), (200000, 8), (30000, 8)):
        assert not plan.streams(m, n, 0)


@pytest.mark.parametrize("m,n,streams", [(8192, 4096, 0), (8192, 6144, 0), (16383, 4096, 0), (16384, 4096, 1), (16384, 5120, 1), (8192, 11008, 1), (65536, 4096, 1)])
def test_the_kind_of_store(plan, m, n, streams):
    assert plan.streams(m, n, 1) == streams
