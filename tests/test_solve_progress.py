"""A solving workgroup of the fused factor-and-solve launch follows the progress word through restarts of the
factorisation: it starts over once per restart, takes every panel from the last attempt, and gives up when the
factorisation stops.  The rules are compiled for the host from the header that the kernel includes; the loop around
them is the kernel's, with its poll that is sent off a step ahead."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2509_23472_amd", "csrc")
MODEL = r'''
#include "%s/progress.h"
// words[i]: the progress word at poll i, the last one from then on.  taken[J]: attempt that panel J of the last pass came
// from.  Returns the passes that were started over, -1 after giving up, -2 when it polls on for ever.
extern "C" int follow(const int* words, int n, int panels, int strips, int limit, int* taken, int* polls) {
  int polled = 0, restarts = 0;
  *polls = 0;
  auto word = [&] { const int i = (*polls)++; return words[i < n ? i : n - 1]; };
  auto poll = [&](int spin) { return spin == 0 ? polled : word(); };
  CfProgress at;
  for (int strip = 0; strip < strips; ++strip) {
    bool restart = false;
    for (int J = 0; J < panels && !restart; ++J) {
      const int go = cf_wait_panel(at, J, limit, poll);
      if (go == CF_GIVE_UP) return -1;
      if (go == CF_RESTART) { restart = true; break; }
      taken[J] = at.attempt;
      polled = word();
    }
    if (restart) { strip = -1; ++restarts; }
    if (restarts > 1000) return -2;
  }
  return restarts;
}
'''


@pytest.fixture(scope="module")
def follow(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("clang++")
    assert cxx, "needs a host C++ compiler"
    d = tmp_path_factory.mktemp("progress")
    (d / "model.cpp").write_text(MODEL % CSRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", str(d / "model.cpp"), "-o", str(d / "model.so")], check=True)
    lib = ctypes.CDLL(str(d / "model.so"))

    def call(words, panels, strips=1, limit=100):
        w = (ctypes.c_int * len(words))(*[(a << 16) | p for a, p in words])
        taken, polls = (ctypes.c_int * panels)(), ctypes.c_int()
        r = lib.follow(w, len(words), panels, strips, limit, taken, ctypes.byref(polls))
        return r, list(taken), polls.value
    return call


def test_no_restart(follow):
    assert follow([(0, p) for p in range(5)], 4)[:2] == (0, [0] * 4)
    assert follow([(0, 4)], 4, strips=3)[:2] == (0, [0] * 4)


@pytest.mark.parametrize("before", [0, 1, 3])        # panels the abandoned attempt had published
@pytest.mark.parametrize("wait", [1, 2, 7, 40])      # polls that see the new attempt without a panel
def test_one_restart(follow, before, wait):
    words = [(0, p) for p in range(before + 1) for _ in range(3)] + [(1, 0)] * wait + [(1, p) for p in range(1, 5)]
    r, taken, polls = follow(words, 4, strips=2)
    assert (r, taken) == (1, [1] * 4)
    assert polls <= len(words) + 2 * 4 + 2


@pytest.mark.parametrize("before", [0, 2])
def test_gives_up_when_the_factorisation_stops_after_a_restart(follow, before):
    words = [(0, p) for p in range(before + 1)] + [(1, 0)]
    r, _, polls = follow(words, 4, limit=50)
    assert r == -1 and polls <= len(words) + 2 * 50
    assert follow([(0, before)], 4, limit=50)[0] == -1


@pytest.mark.parametrize("seed", range(50))
def test_any_pace(follow, seed):
    rng = random.Random(seed)
    panels = rng.randint(1, 16)
    path = [(0, p) for p in range(rng.randint(0, panels - 1) + 1)] + [(1, p) for p in range(panels + 1)]
    words = [w for w in path if rng.random() < 0.7 for _ in range(rng.randint(1, 5))] + [(1, panels)]
    r, taken, _ = follow(words, panels, strips=rng.randint(1, 3))
    assert taken == [1] * panels and 0 <= r <= 1
