"""Who adds the shares of T in the LoRA gradient: at the sizes that were timed both ways, the way that was the faster one.
The rule is compiled for the host from the header that the launcher includes."""
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
    d = tmp_path_factory.mktemp("lora_plan")
    (d / "m.cpp").write_text('#include "%s/lora_plan.h"\nextern "C" int adds(int s, int k, int rp, long long n) '
                             "{ return lora_product_adds_shares(s, k, rp, n); }\n"
                             'extern "C" int splits(int planned, long long wanted, long long fit, long long m, int r) '
                             "{ return lora_general_splits(planned, wanted, fit, m, r); }\n" % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    so = ctypes.CDLL(str(d / "m.so"))
    so.adds.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    so.splits.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_longlong, ctypes.c_int]
    return so


@pytest.fixture(scope="module")
def adds(plan):
    return plan.adds


@pytest.mark.parametrize("shares,k,rp,product", [
    # a launch is the slower way by 0.3 us and more
    (1, 320, 32, 1), (8, 8, 16, 1), (24, 32, 16, 1), (24, 64, 16, 1), (8, 128, 16, 1), (16, 128, 16, 1), (4, 192, 16, 1), (8, 192, 16, 1),
    (4, 320, 16, 1), (4, 8, 32, 1), (8, 32, 32, 1), (8, 64, 32, 1), (4, 128, 32, 1), (4, 192, 32, 1), (4, 256, 32, 1), (4, 320, 32, 1),
    # the product is
    (48, 8, 16, 0), (32, 128, 16, 0), (12, 192, 16, 0), (24, 192, 16, 0), (12, 256, 16, 0), (24, 256, 16, 0), (12, 320, 16, 0), (24, 8, 32, 0),
    (24, 32, 32, 0), (16, 32, 32, 0), (24, 64, 32, 0), (12, 128, 32, 0), (12, 192, 32, 0), (12, 256, 32, 0), (8, 320, 32, 0), (256, 256, 32, 0)])
@pytest.mark.parametrize("n", [64, 256, 4096, 11008])
def test_the_faster_way(adds, shares, k, rp, n, product):
    assert adds(shares, k, rp, n) == product


def test_bytes_read_again_are_bounded(adds):
    for shares in range(1, 65):
        for k in (8, 64, 128, 320):
            for rp in (16, 32):
                for n in (64, 4096, 11008, 10 ** 6, 10 ** 9):
                    if adds(shares, k, rp, n):
                        assert shares * k * rp * 4 * -(-n // 32) <= 64 << 20


# (planned, wanted by the general product, room for; the number is the planned one where all that are wanted were the slower way)
@pytest.mark.parametrize("planned,wanted,fit,m,r,splits", [
    (1, 8, 64, 4982, 16, 1), (2, 21, 64, 3001, 16, 21), (2, 4, 64, 3001, 64, 4), (2, 4, 64, 16000, 16, 4), (2, 4, 64, 16000, 4, 4),
    (2, 4, 64, 16000, 40, 4), (2, 4, 64, 16000, 64, 2), (2, 4, 3, 16000, 64, 2), (10, 21, 64, 3001, 64, 10),
    (10, 21, 16, 3001, 64, 10), (10, 21, 20, 3001, 16, 20), (16, 43, 20, 200, 64, 20), (4, 8, 5, 1000, 32, 5), (2, 4, 3, 16000, 40, 2), (16, 4, 64, 1000, 16, 4)])
def test_splits_of_the_general_product(plan, planned, wanted, fit, m, r, splits):
    assert plan.splits(planned, wanted, fit, m, r) == splits


def test_splits_of_the_general_product_fit(plan):
    for planned in (1, 2, 16):
        for wanted in (1, 3, 64):
            for fit in (planned, planned + 1, 500):
                for m in (1, 96, 3001, 70000, 10 ** 9):
                    for r in (1, 33, 64):
                        got = plan.splits(planned, wanted, fit, m, r)
                        assert 1 <= got <= fit and got <= max(1, wanted) and (got <= planned or got * m * r * 4 <= 12 << 20)
