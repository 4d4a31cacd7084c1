"""Factorisations n = S P of the matrix-product transforms (host logic, CPU)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_19130_amd", "csrc")

SRC = r"""
#include <cstdio>
#include "ibp_host.hpp"
int main() {
  for (int n = 1; n <= 4096; ++n) {
    const ibp::MdftShape m = ibp::mdft_shape(n);
    printf("%d %d %d %d %d\n", n, m.S, m.P, m.MT, m.KT);
  }
}
"""


def test_shapes_of_every_length(tmp_path):
    """Every length: S P = n with S <= 16 and 4 <= P <= 256, the 16-row and
    4-deep steps cover P/2 + 1 (the depth in an even number of steps, none to
    spare), no other divisor takes fewer products, and lengths are left to the
    other kernels exactly when no divisor qualifies."""
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "shapes.cpp", tmp_path / "shapes"
    src.write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), os.path.join(CSRC, "ibp_host.cpp"), "-o", str(exe)],
                   check=True)
    rows = [tuple(map(int, l.split())) for l in subprocess.run([str(exe)], check=True, capture_output=True,
                                                               text=True).stdout.splitlines()]
    assert len(rows) == 4096

    def steps(P):
        L = P // 2 + 1
        return -(-L // 16), 2 * -(-L // 8)

    def cost(P):
        mt, kt = steps(P)
        return mt * kt / P

    for n, S, P, MT, KT in rows:
        ok = [s for s in range(1, 17) if n % s == 0 and 4 <= n // s <= 256] if n >= 16 else []
        if not ok:
            assert S == 0, n
            continue
        assert S in ok and S * P == n and (MT, KT) == steps(P), (n, S, P)
        assert 16 * MT >= P // 2 + 1 and 4 * KT >= P // 2 + 1 and KT % 2 == 0
        assert cost(P) <= min(cost(n // s) for s in ok) * (1 + 1e-12), (n, S, P)
