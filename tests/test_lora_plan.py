"""Who adds the shares of T in the LoRA gradient: at the sizes that were timed both ways, the way that was the faster one.
The rule is compiled for the host from the header that the launcher includes."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")


@pytest.fixture(scope="module")
def adds(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("lora_plan")
    (d / "m.cpp").write_text('#include "%s/lora_plan.h"\nextern "C" int adds(int s, int k, int rp, long long n) '
                             "{ return lora_product_adds_shares(s, k, rp, n); }\n" % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    fn = ctypes.CDLL(str(d / "m.so")).adds
    fn.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_longlong]
    return fn


@pytest.mark.parametrize("shares,k,rp,product", [
    # a launch is the slower way by 0.3 us and more
    (8, 8, 16, 1), (24, 32, 16, 1), (24, 64, 16, 1), (24, 32, 32, 1), (8, 64, 32, 1), (16, 64, 32, 1), (16, 128, 16, 1),
    (8, 192, 16, 1), (8, 256, 16, 1), (8, 128, 32, 1),
    # the product is
    (2, 256, 32, 0), (8, 256, 32, 0), (16, 256, 32, 0), (24, 256, 32, 0), (8, 320, 32, 0), (12, 128, 32, 0), (24, 128, 32, 0),
    (12, 192, 16, 0), (24, 128, 16, 0), (24, 64, 32, 0), (12, 256, 16, 0), (24, 320, 16, 0), (48, 8, 16, 0)])
@pytest.mark.parametrize("n", [64, 256, 1024])
def test_the_faster_way(adds, shares, k, rp, n, product):
    assert adds(shares, k, rp, n) == product


def test_bytes_read_again_are_bounded(adds):
    for shares in range(1, 65):
        for k in (8, 64, 128, 320):
            for rp in (16, 32):
                for n in (64, 4096, 11008, 10 ** 6):
                    if adds(shares, k, rp, n):
                        assert shares * k * rp * 4 * -(-n // 32) <= 8 << 20
