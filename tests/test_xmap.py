"""Host-only check of the places a mapped token is read from (csrc/xmap.h):
every place lies inside the arrays that a call brings.  A call without drafts
brings no drafter rows (the launcher then passes t, B * V logits, in their
place), so a plain bonus row must name no place in them."""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_26004_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "xmap.h"
using namespace asym;
int main() {
  int bad = 0;
  const int sizes[][3] = {{1, 1, 3}, {3, 7, 5}, {3, 7, 50000}, {2, 513, 512}, {5, 40, 1}};
  for (auto& z : sizes) {
    const int rows = z[0], V = z[1], Vd = z[2];
    std::vector<int32_t> vmap(V);
    for (int x = 0; x < V; ++x) vmap[x] = x % 4 == 0 ? Vd - 1 : x % 4 == 1 ? -1 : x % 4 == 2 ? Vd : x % Vd;
    for (int row = 0; row < rows; ++row)
      // a sub-block of 512 tokens runs past the end of the vocabulary
      for (long long x = -3; x < V + 600; ++x)
        for (int ab = 0; ab < 2; ++ab) {
          const XPlace p = map_place(vmap.data(), row, V, Vd, x, ab != 0);
          const bool shared = x >= 0 && x < V && vmap[x] >= 0 && vmap[x] < Vd;
          bad += p.in != shared;
          bad += p.t < (long long)row * V || p.t >= (long long)(row + 1) * V;
          if (shared) bad += p.t != (long long)row * V + x;
          if (ab) {
            bad += p.ab < (long long)row * Vd || p.ab >= (long long)(row + 1) * Vd;
            if (shared) bad += p.ab != (long long)row * Vd + vmap[x];
          } else {
            bad += p.ab != -1;   // no drafter array, whatever is in its place, is read
          }
        }
  }
  printf("%d\n", bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("xmap")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return exe


def test_places_lie_in_the_arrays(driver):
    r = subprocess.run([str(driver)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "0", r.stdout


def test_plain_bonus_rows_name_no_drafter_array():
    """The readers of single mapped tokens take their places from map_place with
    the row's kind; none indexes a or b by the map itself."""
    for name in ("resolve.h", "device.h"):
        src = open(os.path.join(CSRC, name)).read()
        calls = re.findall(r"map_place\(A\.vmap,[^;]*;", src)
        assert calls, name
        for c in calls:
            assert re.search(r", (!bonus|ab)\);$", c), c
        for line in src.splitlines():
            if re.search(r"load_one\(A\.[ab],", line):
                assert "pl.ab)" in line or "pl[e].ab)" in line, line
