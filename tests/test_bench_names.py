"""bench.py knows the kernels that the library launches: the cut to rank k is counted whole, and the kernels
that the step is made of have a cost."""
import importlib.util
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_23472_amd", "csrc")


def _bench():
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


def test_every_launch_of_the_truncation_is_counted_as_such():
    launched = set()
    for f in os.listdir(CSRC):
        launched |= set(re.findall(r'"((?:truncate|jacobi)_\w+)"', open(os.path.join(CSRC, f)).read()))
    assert {"jacobi_eig", "jacobi_init", "jacobi_finish", "truncate_bbt", "truncate_chol"} <= launched
    src = open(os.path.join(ROOT, "bench.py")).read()
    counted = set(re.findall(r'"(\w+)"', src[src.index("trunc_names = "):src.index("us_trunc = ")]))
    assert launched <= counted, launched - counted


def test_kernels_of_the_lora_gradient_have_a_cost():
    cost = _bench().algorithmic_cost
    m, n, k, n_out, r = 8192, 4096, 128, 4096, 16
    assert cost("lora_gt", m, n, k, 2, n_out, r, 1) == ("hbm", 2.0 * (m * n_out + r * n_out + m * k), "GB/s")
    assert cost("lora_tsum", m, n, k, 2, n_out, r, 1)[1] == 257 * k * r * 4
    assert cost("gram", 12608, 768, 32, 2, 768, r, 2)[1] == 2.0 * 12608 * 256 * 3
