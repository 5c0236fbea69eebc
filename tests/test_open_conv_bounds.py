"""Every index that the convolutional opening layer's gradient forms stays inside its
array (CPU only): a host program evaluates the kernel's own index map
(csrc/lp_open_geo.h) for every supported image size, batches below, at and beside a
group of images, and every thread."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1812_04352_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <set>
#include "lp_open_geo.h"
using namespace lp::open_conv;

// the image sizes of the convolution kernels: an even height, at most 56 tiles of 16
// pixel pairs, two 8-channel images with padded channel stride and 584 weights in 64 KB
static bool supported(int H, int W) {
  const int phw = (H + 2) * (W + 2), cs = phw + (((16 - phw) % 64) + 64) % 64;
  return (H / 2 * W + 15) / 16 <= 56 && (2 * 8 * cs + 584) * 4 <= 65536;
}

static long bad = 0;
static void check(bool ok, const char* what, int H, int W, int B, int i) {
  if (!ok && ++bad <= 5) printf("%s: H %d W %d B %d pixel %d\n", what, H, W, B, i);
}

int main() {
  const int C = 8;
  int sizes = 0;
  for (int H = 2; H <= 1024; H += 2)
    for (int W = 1; W <= 1024; ++W) {
      if (!supported(H, W)) continue;
      ++sizes;
      const Group g = group(H, W);
      check(g.IM >= 1 && g.IM * g.PH <= OC_LDS, "group", H, W, 0, 0);
      for (int B : std::set<int>{1, 2, g.IM - 1, g.IM, g.IM + 1, 2 * g.IM, 2 * g.IM + 3}) {
        if (B < 1) continue;
        for (int e0 = 0; e0 < B; e0 += g.IM) {
          const int n = images(g, B, e0);
          check(n >= 1 && n <= g.IM && e0 + n <= B, "images", H, W, B, e0);
          long pixels = 0;
          for (int i = 0; i < GNT * OCP; ++i) {
            const Pixel p = pixel(g, W, C, C - 1, i);
            if (stored(g, p)) check(store_index(g, p) >= 0 && store_index(g, p) < g.IM * g.PH, "store", H, W, B, i);
            if (!live(p, n)) continue;
            ++pixels;
            check(stored(g, p), "live pixel without a place", H, W, B, i);
            check((long)e0 * g.P + i < (long)B * g.P, "read of y", H, W, B, i);
            check((long)e0 * C * g.P + p.gl < (long)B * C * g.P, "read of lam0", H, W, B, i);
            check(p.at >= 0 && p.at + 2 * g.PW + 2 < g.IM * g.PH, "window", H, W, B, i);
          }
          check(pixels == (long)n * g.P, "each pixel once", H, W, B, e0);
        }
      }
    }
  printf("%d sizes, %ld bad\n", sizes, bad);
  return bad || sizes < 1000;
}
"""


def test_conv_opening_gradient_indexes(tmp_path):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "bounds.cpp", tmp_path / "bounds"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-I", CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout
