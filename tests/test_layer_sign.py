"""The signs of the split products balance on the layers of every level, for any
coarsening factor (CPU only: a host program evaluates csrc/lp_layer_sign.h)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1812_04352_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "lp_layer_sign.h"

int main() {
  int bad = 0;
  for (int c = 2; c <= 32; ++c) {
    long m = 1;
    for (int l = 0; m <= 4096; ++l, m *= c) {
      int s = 0, most = 0;
      for (long n = 0; n < 16384; n += m) {
        const float f = lp::layer_sign((size_t)n);
        if (f != 1.f && f != -1.f) return 2;
        s += (int)f;
        if (abs(s) > most) most = abs(s);
      }
      if (most > (m == 1 ? 1 : 14)) ++bad, printf("c = %d level %d: %d of %ld layers\n", c, l, most, (16384 + m - 1) / m);
    }
  }
  return bad != 0;
}
"""


def test_layer_signs_balance_for_every_coarsening_factor(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "sign.cpp", tmp_path / "sign"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
