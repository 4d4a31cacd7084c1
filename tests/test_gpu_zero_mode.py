"""The (0,0) mode of FP64 singular solves, from the spectrum's (0,0) column
after direct transforms and from the row sums after Bluestein ones, and
batches of more grids than one load of the grid search covers (64)."""

import numpy as np
import pytest
import torch

import oracle
from paper_2609_19130_amd import ibpoisson as ibp
from paper_2609_19130_amd import synth

from gpu_helpers import gpu_solve, rel, require_gpu, to_dev

pytestmark = pytest.mark.gpu
TOL64 = 1e-12


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def field(nx, ny, nz):
    """Plane means of up to 5, so that the (0,0) mode carries most of the solution."""
    f = np.random.default_rng(nx + 7 * ny + 13 * nz).uniform(-1, 1, (ny, nz, nx))
    return f + 5 * np.cos(np.arange(ny) + 0.3)[:, None, None]


# register lengths, matrix products, mixed radix (too short for products), Bluestein in z and in x, nz = 1, tall columns
@pytest.mark.parametrize("nx,ny,nz", [(64, 9, 32), (48, 200, 40), (12, 33, 10), (34, 5, 521), (1042, 5, 6), (40, 17, 1),
                                      (1, 17, 40), (20, 650, 6), (20, 1400, 6), (20, 900, 6)])
def test_plane_means(nx, ny, nz):
    yf = synth.tanh_faces(ny, 2.0)
    f = field(nx, ny, nz)
    got, info = gpu_solve(f, 2 * np.pi, 1.7, yf)
    ref, m = oracle.solve(f, 2 * np.pi, 1.7, yf)
    assert rel(got, ref) <= TOL64
    assert abs(info["removed_mean"] - m) <= 3e-14   # log2(n) = 15 additions of values up to 6, rounded to 1.1e-16
    f[ny // 2, 0, 0] = np.inf
    _, info = gpu_solve(f, 2 * np.pi, 1.7, yf)
    assert info["nonfinite_input"] == 1


@pytest.mark.parametrize("count", [1, 63, 64, 65, 130])
def test_batches_past_one_load_of_the_search(count):
    shapes = [(32 + 4 * (i % 5), 4 + 3 * (i % 7), 24 + 8 * (i % 3)) for i in range(count)]
    plans, rhs, refs = [], [], []
    for i, (nx, ny, nz) in enumerate(shapes):
        yf = synth.tanh_faces(ny, 1.5)
        f = field(nx, ny, nz) + i
        plans.append(ibp.Plan(nx, ny, nz, 2 * np.pi, 1.7, yf))
        rhs.append(to_dev(f))
        refs.append(oracle.solve(f, 2 * np.pi, 1.7, yf)[0])
    phi = ibp.solve_batched(plans, rhs, [torch.empty_like(r) for r in rhs])
    for p, ref in zip(phi, refs):
        assert rel(p.cpu().numpy(), ref) <= TOL64
    for p in plans:
        p.close()
