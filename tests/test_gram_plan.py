"""The work split of the wide Gram matrix covers every (pair of blocks, step of rows) exactly once, every set of partial tiles
has one writer and all of them are summed.  The planner is compiled for the host from the header that the kernels include;
the walk over a workgroup's share is the kernel's."""
import ctypes
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")
MODEL = r'''
#include "%s/gram_plan.h"
#include <vector>
extern "C" int check(long long m, int kp) {
  const GramPlan g = gram_plan(m, kp);
  if (g.wgs < 1 || g.wgs > GRAM_MAX_WGS || g.units > GRAM_MAX_UNITS) return 1;
  if ((int64_t)g.slices * g.steps * GRAM_STEP < m || g.slices * g.wgs > 256) return 2;
  std::vector<int> cover((size_t)g.units * g.steps, 0), part(g.part_tiles, 0);
  int64_t tiles = 0;
  for (int n = 0; n < g.units; ++n) {
    const GramUnit& u = g.unit[n];
    if (u.ci + 16 * u.qi > kp || u.cj + 16 * u.qj > kp || u.qi < 2 || u.qi > u.qj || u.qj > 4) return 3;
    tiles += u.tiles;
  }
  if (tiles != (kp / 16) * (kp / 16 + 1) / 2) return 4;
  for (int w = 0; w < g.wgs; ++w) {
    const GramBound from = g.bound[w], to = g.bound[w + 1];
    for (int n = from.unit; n <= to.unit; ++n) {
      const int first = n == from.unit ? from.step : 0, last = n == to.unit ? to.step : g.steps;
      if (first == last) break;
      if (n >= g.units || first > last) return 5;
      const GramUnit& u = g.unit[n];
      if (w < u.wg0 || w >= u.wg0 + u.wgs) return 6;
      for (int s = first; s < last; ++s) ++cover[(size_t)n * g.steps + s];
      for (int slice = 0; slice < g.slices; ++slice)
        for (int t = 0; t < u.qi * u.qj; ++t) {
          const int at = u.part_at + ((w - u.wg0) * g.slices + slice) * u.qi * u.qj + t;
          if (at < 0 || at >= g.part_tiles) return 7;
          ++part[at];
        }
    }
  }
  for (int x : cover) if (x != 1) return 8;
  for (int x : part) if (x != 1) return 9;
  return 0;
}
'''


@pytest.fixture(scope="module")
def check(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("gram_plan")
    (d / "m.cpp").write_text(MODEL % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    fn = ctypes.CDLL(str(d / "m.so")).check
    fn.argtypes = [ctypes.c_longlong, ctypes.c_int]
    return fn


@pytest.mark.parametrize("kp", range(80, 321, 16))
def test_every_step_has_one_workgroup(check, kp):
    edges = [32 * a + b for a in (1, 2, 7, 8, 9, 31, 96, 255, 256, 257, 400, 1000, 2048) for b in (-1, 0, 1)]
    for m in [1, 2] + edges + [100003, 1000000]:
        assert check(m, kp) == 0, (m, kp, check(m, kp))


def test_the_split_is_made_once_a_call():
    # it costs the host 0.2 to 0.6 us; both rounds and the workspace's size share the one in the call's plan
    calls = []
    for name in sorted(os.listdir(CSRC)):
        for line in open(os.path.join(CSRC, name)):
            code = line.split("//")[0]
            if "gram_plan(" in code and "static GramPlan gram_plan(" not in code:
                calls.append((name, code.strip()))
    assert [c[0] for c in calls] == ["loract.hip"], calls


RULES = r'''
#include "%s/gram_plan.h"
extern "C" int kernel(long long m, int kp) { return gram_is_narrow(kp) ? 0 : (gram_is_short(m, kp) ? 1 : 2); }
extern "C" int short_rows(long long m, int kp) { return gram_short_rows(m, kp); }
extern "C" int short_blocks(int kp) { return gram_short_blocks(kp); }
'''


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("gram_rules")
    (d / "m.cpp").write_text(RULES % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(d / "m.cpp"), "-o", str(d / "m.so")], check=True)
    so = ctypes.CDLL(str(d / "m.so"))
    so.kernel.argtypes = so.short_rows.argtypes = [ctypes.c_longlong, ctypes.c_int]
    return so


@pytest.mark.parametrize("m,kp,kernel", [
    (200, 80, 1), (200, 192, 1), (331, 320, 1), (512, 256, 1), (1000, 96, 1), (1000, 128, 1), (1000, 320, 1), (1500, 192, 1), (2000, 128, 1),
    (2000, 320, 1), (3001, 80, 1), (3001, 256, 1), (4096, 128, 1), (5000, 128, 1),
    (3001, 320, 2), (5000, 256, 2), (7000, 160, 2), (7000, 80, 2), (8192, 192, 2), (8192, 256, 2), (65536, 256, 2), (1000, 64, 0)])
def test_the_faster_kernel(rules, m, kp, kernel):
    assert rules.kernel(m, kp) == kernel


def test_chunks_of_the_short_kernel(rules):
    for kp in range(80, 321, 16):
        for m in (1, 31, 32, 33, 100, 1000, 2048, 4096, 6144):
            rows = rules.short_rows(m, kp)
            chunks = -(-m // rows)
            assert rows % 16 == 0 and rows >= 32 and (chunks - 1) * rows < m
            assert chunks * rules.short_blocks(kp) <= 4 * 256 + rules.short_blocks(kp)
