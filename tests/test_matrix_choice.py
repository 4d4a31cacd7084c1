"""Which FP64 passes take the matrix products (host logic, CPU): the sides of
the rules that were measured."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_19130_amd", "csrc")

SRC = r"""
#include <cstdio>
#include <cstring>
#include "ibp_host.hpp"
int main() {
  char k[8];
  int n, blu;
  double w;
  while (scanf("%7s %d %d %lf", k, &n, &blu, &w) == 4) {
    const ibp::MdftShape m = ibp::mdft_shape(n);
    const bool on = !strcmp(k, "x") ? ibp::mdft_x_pays(n, m, blu, w)
                  : !strcmp(k, "z") ? ibp::mdft_z_pays(n, m, blu, w) : ibp::mdft_div_pays(n, blu != 0, w);
    printf("%d", on);
  }
}
"""

# (pass, points, register Bluestein length or 0 (div: direct sums), rows or column groups per compute unit): products
CASES = [
    # long product sums against a short convolution, and the paper's lengths at their grids
    (("x", 251, 512, 16), 0), (("z", 251, 512, 1000), 0), (("x", 502, 1024, 1000), 0), (("z", 502, 1024, 1000), 0),
    (("x", 131, 512, 256), 1), (("x", 131, 512, 4), 0), (("z", 197, 512, 100), 0), (("z", 155, 512, 0.1), 1),
    (("x", 501, 1024, 1959), 1), (("z", 501, 1024, 125), 1), (("x", 632, 2048, 3118), 1), (("z", 632, 2048, 197), 1),
    (("x", 501, 1024, 1), 0), (("z", 501, 1024, 1), 0), (("x", 753, 2048, 16), 1), (("x", 1004, 2048, 16), 0),
    # general kernels: few long rows
    (("x", 384, 0, 320), 1), (("x", 32, 0, 1), 1), (("x", 1536, 0, 1), 0), (("x", 1536, 0, 4), 1), (("z", 320, 0, 40), 1),
    # assembled right-hand side: full tiles of the general kernel, few rows, odd lengths, direct sums
    (("div", 96, 0, 1), 1), (("div", 320, 0, 64), 0), (("div", 640, 0, 256), 0), (("div", 300, 0, 64), 1),
    (("div", 300, 0, 16), 0), (("div", 720, 0, 4), 0), (("div", 720, 0, 16), 1), (("div", 375, 0, 16), 1),
    (("div", 502, 1, 1), 1)]


def test_measured_sides(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "choice.cpp", tmp_path / "choice"
    src.write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), os.path.join(CSRC, "ibp_host.cpp"), "-o", str(exe)],
                   check=True)
    lines = "".join(" ".join(map(str, c)) + "\n" for c, _ in CASES)
    out = subprocess.run([str(exe)], input=lines, check=True, capture_output=True, text=True).stdout
    wrong = [c for (c, want), got in zip(CASES, out) if int(got) != want]
    assert len(out) == len(CASES) and not wrong, wrong
