"""FP64 line solves with the columns in registers (513..768 and 1025..1536
rows): both ends of every row count that has its own shape, both kinds of
wall, against the oracle at the tolerance of the other parity tests and
against the staged solve (columns given) at twice that."""

import numpy as np
import pytest

import oracle
from paper_2609_19130_amd import ibpoisson as ibp
from paper_2609_19130_amd import synth

from gpu_helpers import gpu_solve, rel, require_gpu

pytestmark = pytest.mark.gpu
TOL64 = 1e-12


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


@pytest.mark.parametrize("bc", [("neumann", "neumann"), ("dirichlet", "neumann"), ("dirichlet", "dirichlet")])
@pytest.mark.parametrize("ny", [513, 640, 641, 768, 1025, 1280, 1281, 1536])
def test_rows_at_the_edges_of_every_shape(monkeypatch, ny, bc):
    nx, nz = (18, 10) if ny % 2 else (32, 7)   # kx padding with and without a last line of its own
    yf = synth.tanh_faces(ny, 2.0)
    f = np.random.default_rng(ny).uniform(-1, 1, (ny, nz, nx))
    got, info = gpu_solve(f, 2 * np.pi, 1.7, yf, bc=bc)
    again, _ = gpu_solve(f, 2 * np.pi, 1.7, yf, bc=bc)
    assert np.array_equal(got, again)
    monkeypatch.setenv("IBP_YCOLS", "4")
    staged, _ = gpu_solve(f, 2 * np.pi, 1.7, yf, bc=bc)
    ref, m = oracle.solve(f, 2 * np.pi, 1.7, yf, bc=bc)
    assert rel(got, ref) <= TOL64
    assert rel(got, staged) <= 2 * TOL64
    assert abs(info["removed_mean"] - m) <= 1e-14
