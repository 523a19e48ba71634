"""Host-only check of the tags (csrc/tags.h): an epoch has bits 31 and
30 set and no plain word of a cross-family call has both, so that a word which an earlier call
left in the workspace can never pass for a tagged slot of a later one."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2608_26004_amd", "csrc")

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include "tags.h"
using namespace asym;
static int bad = 0;
static bool epoch_like(uint32_t w) { return (w & kEpochBits) == kEpochBits; }
static uint32_t bits(float v) { uint32_t w; memcpy(&w, &v, 4); return w; }
template <int JBITS> void entries(uint32_t vmax) {
  using E = XEntry<JBITS>;
  const uint32_t lo = E::kSpan, ids = 1u << JBITS;
  for (uint32_t x = 0; x < vmax; x += x % 1000 == 7 ? 1013 : 1)
    for (uint32_t j : {0u, 1u, ids / 2, ids - 1}) {
      const uint32_t e = E::make(x, j);
      bad += epoch_like(e) || E::id(e) != j || E::token(e) + x / lo * lo != x;
    }
}
int main() {
  for (uint32_t n : {0u, 1u, 0x3FFFFFFFu, 0x7FFFFFFFu, 0x80000000u, 0xFFFFFFFFu}) bad += !epoch_like(epoch_of(n));
  // consecutive calls have different epochs, also around the counter's wrap
  for (uint32_t n = 0x3FFFFFF0u; n != 0x40000010u; ++n) bad += epoch_of(n) == epoch_of(n + 1);
  entries<14>(4194297);
  entries<13>(2097149);
  for (float v : {0.0f, -0.0f, 1.0f, -1e-9f, 3e38f, INFINITY, -INFINITY, NAN, -NAN, 1e-45f, -1e-45f}) {
    const float r = plain_sum(v);
    bad += epoch_like(bits(r)) || (v > 0 ? r != v : r != 0.0f);
  }
  printf("%d\n", bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("tags")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    return exe


def test_plain_words_never_match_an_epoch(driver):
    r = subprocess.run([str(driver)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "0", r.stdout


def test_the_launcher_and_the_kernels_use_them():
    host = open(os.path.join(CSRC, "asymspec.hip")).read()
    assert "return epoch_of(" in host[host.index("static uint32_t next_epoch"):]
    xv = open(os.path.join(CSRC, "xvocab.h")).read()
    for line in xv.splitlines():
        if "sums[cur] =" in line or "X.jpart[" in line:
            assert "plain_sum(" in line, line
    assert "Entry::make(" in xv
