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


WALK = r'''
#include "%s/project_plan.h"
static bool differs(int64_t items, int64_t wgs, int64_t slabs, int64_t tile, ProjectShares got) {
  // share by share, as they are defined; the walk begins two before where the first share has to be
  const int64_t lo = tile * slabs, hi = lo + slabs;
  auto begin = [&](int64_t w) { return (int64_t)((__int128)items * w / wgs); };
  int64_t first = (int64_t)((__int128)lo * wgs / items) - 2;
  if (first < 0) first = 0;
  while (begin(first + 1) <= lo) ++first;
  int64_t end = first;
  while (end < wgs && begin(end) < hi) ++end;
  return got.first != first || got.end != end || got.first_tile != begin(first) / slabs;
}
extern "C" long long check(long long tiles, int slabs, int wgs) {
  const int64_t items = (int64_t)tiles * slabs;
  long long bad = 0;
  for (int64_t tile = 0; tile < tiles; tile += tile < 300 || tile > tiles - 300 ? 1 : tiles / 300 + 1) {
    bad += differs(items, wgs, slabs, tile, project_shares(items, wgs, slabs, tile));
    bad += differs(items, wgs, slabs, tile, project_shares_of<int64_t>(items, wgs, slabs, tile));
    if (items < PJ_ITEMS_32) bad += differs(items, wgs, slabs, tile, project_shares_of<unsigned>(items, wgs, slabs, tile));
  }
  return bad;
}
extern "C" long long items_32() { return PJ_ITEMS_32; }
'''


def test_shares_of_a_tile(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    (tmp_path / "m.cpp").write_text(WALK % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m.so")], check=True)
    so = ctypes.CDLL(str(tmp_path / "m.so"))
    so.check.argtypes, so.check.restype, so.items_32.restype = [ctypes.c_longlong, ctypes.c_int, ctypes.c_int], ctypes.c_longlong, ctypes.c_longlong
    limit = so.items_32()
    for slabs in (1, 2, 5, 16, 47, 128, 1024):
        for tiles in (1, 2, 3, 16, 86, 255):
            for wgs in (1, 2, 7, 64, 255, 256, 511, 512):
                if wgs <= tiles * slabs:
                    assert so.check(tiles, slabs, wgs) == 0, (tiles, slabs, wgs)
    # both sides of the line between 32 and 64 bits, and the largest there are (2^31 rows and columns are far past the grid)
    for slabs in (9, 1000, 33554432):
        for tiles in (limit // slabs - 1, limit // slabs, limit // slabs + 1, limit // slabs + 2, 65535):
            for wgs in (1, 511, 512):
                if tiles >= 1 and wgs <= tiles * slabs:
                    assert so.check(tiles, slabs, wgs) == 0, (tiles, slabs, wgs)


ORDER = r'''
#include "%s/project_plan.h"
#include <algorithm>
// 0: the shares sorted by begin modulo period (in buckets of 2^shift) and dealt to the dies in runs, a die's longer ones first if asked
// for; 1: not a permutation; 2: another order
extern "C" int order(long long items, int wgs, long long period, int sorted, int long_first) {
  unsigned short got[PJ_MAX_WGS + 1], seen[PJ_MAX_WGS] = {0};
  int want[PJ_MAX_WGS], shift = 0;
  got[wgs] = 0xabcd;
  project_share_order(items, wgs, period, sorted, got, long_first);
  for (int b = 0; b < wgs; ++b)
    if (got[b] >= wgs || seen[got[b]]++) return 1;
  if (got[wgs] != 0xabcd) return 1;
  while (((period - 1) >> shift) > 255) ++shift;
  for (int w = 0; w < wgs; ++w) want[w] = w;
  auto key = [&](int w) { return (int64_t)((__int128)items * w / wgs %% period) >> shift; };
  if (sorted) std::stable_sort(want, want + wgs, [&](int a, int b) { return key(a) < key(b); });
  auto size = [&](int w) { return (int64_t)((__int128)items * (w + 1) / wgs) - (int64_t)((__int128)items * w / wgs); };
  for (int d = 0; long_first && d < 8; ++d)
    std::stable_sort(want + d * (wgs / 8) + std::min(d, wgs %% 8), want + (d + 1) * (wgs / 8) + std::min(d + 1, wgs %% 8),
                     [&](int a, int b) { return size(a) > size(b); });
  for (int b = 0; b < wgs; ++b)
    if (want[b %% 8 * (wgs / 8) + std::min(b %% 8, wgs %% 8) + b / 8] != got[b]) return 2;
  return 0;
}
'''


def test_order_of_the_shares(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    (tmp_path / "m.cpp").write_text(ORDER % CSRC)
    subprocess.run([gxx, "-O1", "-std=c++17", "-shared", "-fPIC", str(tmp_path / "m.cpp"), "-o", str(tmp_path / "m.so")], check=True)
    order = ctypes.CDLL(str(tmp_path / "m.so")).order
    order.argtypes = [ctypes.c_longlong, ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int]
    for items in (1, 7, 255, 256, 4096, 5504, 16384, 2 ** 31 * 1024 + 5):
        for wgs in (1, 2, 7, 8, 9, 255, 256, 511, 512):
            for period in (1, 2, 47, 255, 256, 257, 1024, 33554432):
                if wgs <= items:
                    for long_first in (0, 1):
                        assert order(items, wgs, period, 1, long_first) == 0, (items, wgs, period, long_first)
    assert order(4096, 300, 64, 0, 0) == 0
    assert order(768, 512, 256, 1, 1) == 0
