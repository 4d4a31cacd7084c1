"""FP64 transforms as register DFTs times matrix products (lengths n = S P).

Each case is held to the oracle at the FP64 tolerance of the other parity
tests (1e-12 relative, the whole field) and to the general transforms on the
same input (IBP_MDFT=0) at twice that.  Lengths cover every S, the edges of
the 16-row and 4-deep steps (P/2 + 1 = 15, 16, 17; P even and odd, smallest
and largest), tiles with idle threads, columns past the spectrum and a last
row without a partner."""

import numpy as np
import pytest

import oracle
from oracle.grid import geometry
from oracle.operators import divergence
from paper_2609_19130_amd import ibpoisson as ibp
from paper_2609_19130_amd import synth

from gpu_helpers import rel, require_gpu, to_dev

pytestmark = pytest.mark.gpu
TOL64 = 1e-12

# x lengths by S: 16: 320, 15: 375, 14: 350, 13: 377, 12: 348, 11: 319, 10: 290, 9: 261, 8: 240, 7: 203, 6: 186,
# 5: 155, 4: 116, 3: 87, 2: 62, 1: 31
SHAPES = [(320, 5, 375), (350, 4, 377), (348, 3, 319), (290, 3, 261), (240, 5, 203), (186, 3, 155), (116, 5, 87),
          (62, 7, 31), (375, 3, 320), (377, 3, 350), (319, 3, 348), (261, 5, 290), (203, 3, 240), (155, 5, 186),
          (87, 3, 116), (31, 5, 62),
          # P/2 + 1 = 15, 16, 17 at one S; the largest P; the smallest lengths
          (28 * 8, 2, 30 * 8), (31 * 8, 3, 32 * 9), (256, 2, 251), (502, 2, 753), (1004, 2, 995), (18, 3, 16), (17, 2, 19)]


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def field(nx, ny, nz):
    return np.random.default_rng(nx + 7 * ny + 13 * nz).uniform(-1, 1, (ny, nz, nx))


def solve(monkeypatch, on, f, yf, **kw):
    monkeypatch.setenv("IBP_MDFT", "1" if on else "0")
    ny, nz, nx = f.shape
    plan = ibp.Plan(nx, ny, nz, 2 * np.pi, 1.7, yf, **kw)
    try:
        return plan.solve(to_dev(f)).cpu().numpy(), plan.info()
    finally:
        plan.close()


@pytest.mark.parametrize("nx,ny,nz", SHAPES)
def test_every_length_class(monkeypatch, nx, ny, nz):
    yf = synth.tanh_faces(ny, 2.0)
    f = field(nx, ny, nz)
    got, info = solve(monkeypatch, True, f, yf)
    general, ginfo = solve(monkeypatch, False, f, yf)
    ref, m = oracle.solve(f, 2 * np.pi, 1.7, yf)
    assert rel(got, ref) <= TOL64
    assert rel(got, general) <= 2 * TOL64
    assert abs(info["removed_mean"] - m) <= 1e-14


def test_many_tiles_per_block(monkeypatch):
    """More tiles than resident blocks, so that blocks loop (the next tile's
    loads run under the current one's products), with ragged last tiles."""
    for nx, ny, nz in [(96, 301, 80), (45, 203, 176)]:
        yf = synth.tanh_faces(ny, 1.5)
        f = field(nx, ny, nz)
        got, _ = solve(monkeypatch, True, f, yf, bc=("neumann", "dirichlet"))
        ref, _ = oracle.solve(f, 2 * np.pi, 1.7, yf, bc=("neumann", "dirichlet"))
        assert rel(got, ref) <= TOL64, (nx, ny, nz)


@pytest.mark.parametrize("nx,ny,nz,sources", [(96, 6, 80, True), (75, 5, 48, False)])
def test_assembled_right_hand_side(monkeypatch, nx, ny, nz, sources):
    monkeypatch.setenv("IBP_MDFT", "1")
    yf = synth.tanh_faces(ny, 2.0)
    u, v, w = synth.uniform_velocity(nx, ny, nz, seed=3)
    q = field(nx, ny, nz) if sources else None
    adt = 0.3
    rhs = divergence(u, v, w, geometry(nx, ny, nz, 2 * np.pi, 1.7, yf))
    rhs = (rhs - q if sources else rhs) / adt
    plan = ibp.Plan(nx, ny, nz, 2 * np.pi, 1.7, yf)
    phi = plan.solve_divergence(to_dev(u), to_dev(v), to_dev(w), adt, q=to_dev(q) if sources else None)
    ref, _ = oracle.solve(rhs, 2 * np.pi, 1.7, yf)
    assert rel(phi.cpu().numpy(), ref) <= TOL64
    plan.close()


def test_update_of_the_mixed_form(monkeypatch):
    """mixed_f64inv on general lengths: its FP64 inverse passes (the update
    adds to the iterate) run the products."""
    nx, ny, nz = 96, 24, 80
    yf = synth.tanh_faces(ny, 2.0)
    u, v, w = synth.uniform_velocity(nx, ny, nz, seed=5)
    f = divergence(u, v, w, geometry(nx, ny, nz, 2 * np.pi, 1.7, yf))
    got, info = solve(monkeypatch, True, f, yf, precision="mixed_f64inv")
    ref, _ = oracle.solve(f, 2 * np.pi, 1.7, yf)
    assert info["converged"] == 1 and info["rel_residual"] <= 1e-10 and info["iterations"] >= 1
    assert rel(got, ref) <= 1e-10   # the mixed forms' tolerance on this residual


def test_non_finite_input_is_flagged(monkeypatch):
    nx, ny, nz = 96, 6, 48
    f = field(nx, ny, nz)
    f[3, 17, 40] = np.nan
    _, info = solve(monkeypatch, True, f, synth.tanh_faces(ny, 2.0))
    assert info["nonfinite_input"] == 1


@pytest.mark.parametrize("nx,ny,nz", [(640, 3, 5), (1536, 2, 7), (1000, 9, 64), (320, 64, 64), (18, 40, 33), (31, 16, 64)])
def test_few_tiles_per_compute_unit(monkeypatch, nx, ny, nz):
    """Rows from below one to sixteen per compute unit: blocks of more waves
    than their tasks need, tiles chosen for even rounds, ragged last ones."""
    yf = synth.tanh_faces(ny, 2.0)
    f = field(nx, ny, nz)
    got, _ = solve(monkeypatch, True, f, yf)
    ref, _ = oracle.solve(f, 2 * np.pi, 1.7, yf)
    assert rel(got, ref) <= TOL64


@pytest.mark.parametrize("nx,ny,nz", [(320, 3, 7), (350, 4, 5), (348, 3, 5), (290, 3, 4), (240, 5, 4), (186, 3, 5),
                                      (116, 5, 6), (62, 7, 8), (375, 3, 5), (377, 3, 4), (319, 3, 6), (261, 5, 4),
                                      (203, 3, 5), (155, 5, 4), (87, 3, 6), (31, 5, 8), (96, 301, 80), (720, 40, 31)])
def test_assembled_right_hand_side_of_every_length_class(monkeypatch, nx, ny, nz):
    """Every S, row pairs across planes (odd nz), blocks that loop."""
    monkeypatch.setenv("IBP_MDFT", "1")
    yf = synth.tanh_faces(ny, 2.0)
    u, v, w = synth.uniform_velocity(nx, ny, nz, seed=nx)
    q = field(nx, ny, nz) if nx % 2 else None
    rhs = divergence(u, v, w, geometry(nx, ny, nz, 2 * np.pi, 1.7, yf))
    rhs = (rhs - q if q is not None else rhs) / 0.3
    plan = ibp.Plan(nx, ny, nz, 2 * np.pi, 1.7, yf)
    phi = plan.solve_divergence(to_dev(u), to_dev(v), to_dev(w), 0.3, q=to_dev(q) if q is not None else None)
    ref, _ = oracle.solve(rhs, 2 * np.pi, 1.7, yf)
    assert rel(phi.cpu().numpy(), ref) <= TOL64
    plan.close()


@pytest.mark.parametrize("nx,ny,nz", [(251, 3, 64), (502, 4, 251), (64, 5, 501), (1536, 2, 7), (334, 40, 64)])
def test_lengths_that_choose_their_kernels_by_size(monkeypatch, nx, ny, nz):
    """Without a request the solve and the solve of an assembled right-hand
    side choose their kernels on their own (products, register Bluestein,
    general), and with them where the (0,0) mode's sums come from."""
    monkeypatch.delenv("IBP_MDFT", raising=False)
    yf = synth.tanh_faces(ny, 2.0)
    u, v, w = synth.uniform_velocity(nx, ny, nz, seed=7)
    rhs = divergence(u, v, w, geometry(nx, ny, nz, 2 * np.pi, 1.7, yf)) / 0.3
    for bc in (("neumann", "neumann"), ("neumann", "dirichlet")):
        plan = ibp.Plan(nx, ny, nz, 2 * np.pi, 1.7, yf, bc=bc)
        f = field(nx, ny, nz)
        ref, m = oracle.solve(f, 2 * np.pi, 1.7, yf, bc=bc)
        assert rel(plan.solve(to_dev(f)).cpu().numpy(), ref) <= TOL64
        assert abs(plan.info()["removed_mean"] - m) <= 1e-14
        phi = plan.solve_divergence(to_dev(u), to_dev(v), to_dev(w), 0.3)
        ref, _ = oracle.solve(rhs, 2 * np.pi, 1.7, yf, bc=bc)
        assert rel(phi.cpu().numpy(), ref) <= TOL64
        plan.close()
