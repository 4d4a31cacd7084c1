"""Tuned configurations against the solve without one: whatever a tuning cache
line asks for, the solution's bits are the same."""

import json

import numpy as np
import pytest
import torch

from paper_2609_19130_amd import ibpoisson as ibp
from paper_2609_19130_amd import synth

from gpu_helpers import require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def plan_of(nx, ny, nz, precision):
    return ibp.Plan(nx, ny, nz, 2 * np.pi, 1.3, synth.tanh_faces(ny, 2.0), precision=precision, max_iters=3)


# rows with a line-solve kernel of their own in FP64 (513..768, 1025..1536) and a staged one; products, general
# and register transforms
@pytest.mark.parametrize("nx,ny,nz,precision", [(32, 600, 7, "fp64"), (18, 1100, 10, "fp64"), (64, 770, 32, "fp64"),
                                                (96, 40, 80, "fp64"), (502, 24, 251, "fp64"), (96, 40, 80, "mixed"),
                                                (96, 40, 80, "mixed_f64sweep"), (100, 30, 60, "mixed_f64inv")])
def test_cached_choices_keep_the_bits(monkeypatch, tmp_path, nx, ny, nz, precision):
    cache = tmp_path / "tune.jsonl"
    f = to_dev(np.random.default_rng(ny).standard_normal((ny, nz, nx)))
    monkeypatch.delenv("IBP_TUNE_CACHE", raising=False)
    p = plan_of(nx, ny, nz, precision)
    ref = p.solve(f)
    monkeypatch.setenv("IBP_TUNE_CACHE", str(cache))
    p.autotune(f)
    assert torch.equal(p.solve(f), ref)
    p.close()
    line = json.loads(cache.read_text().splitlines()[-1])
    for ycols in (0, 2, 4, 8, 16):
        for zdiv in (1, 2, 4):
            for small in (0, 1):
                line.update(ycols=ycols, zdiv=zdiv, xsmall=small, zsmall=small)
                cache.write_text(json.dumps(line) + "\n")
                p = plan_of(nx, ny, nz, precision)
                assert torch.equal(p.solve(f), ref), line
                p.close()


def test_choice_tuned_for_fp64_does_not_follow_into_a_mixed_form(monkeypatch, tmp_path):
    """A plan whose precision is changed after an FP64 configuration with the
    large x tile was applied solves as a plan created in that form."""
    nx, ny, nz = 96, 40, 80
    cache = tmp_path / "tune.jsonl"
    f = to_dev(np.random.default_rng(3).standard_normal((ny, nz, nx)))
    monkeypatch.delenv("IBP_TUNE_CACHE", raising=False)
    p = plan_of(nx, ny, nz, "mixed")
    ref = p.solve(f)
    p.close()
    monkeypatch.setenv("IBP_TUNE_CACHE", str(cache))
    p = plan_of(nx, ny, nz, "fp64")
    p.autotune(f)
    line = json.loads(cache.read_text().splitlines()[-1])
    cache.write_text(json.dumps(dict(line, xsmall=0)) + "\n")
    p.close()
    p = plan_of(nx, ny, nz, "fp64")
    p.set_precision("mixed", max_iters=3)
    assert torch.equal(p.solve(f), ref)
    p.close()


def test_lines_of_other_kernels_are_not_applied(monkeypatch, tmp_path):
    """A cache line timed before the kernels it chooses between changed (no
    revision in its key) leaves a plan to its defaults and to a new search."""
    nx, ny, nz = 96, 40, 80
    cache = tmp_path / "tune.jsonl"
    old = {"key": f"gfx950/plan/{nx}x{ny}x{nz}/0", "xdiv": 1, "zdiv": 4, "ycols": 2, "xsmall": 0, "zsmall": 0,
           "persistent": 0, "lag": 1, "chunk": 8, "ms": 0.1}
    cache.write_text(json.dumps(old) + "\n")
    monkeypatch.setenv("IBP_TUNE_CACHE", str(cache))
    f = to_dev(np.random.default_rng(4).standard_normal((ny, nz, nx)))
    p = plan_of(nx, ny, nz, "fp64")
    assert p.autotune(f)["tried"] > 0
    again = plan_of(nx, ny, nz, "fp64")
    assert again.autotune(f)["tried"] == 0
    for q in (p, again):
        q.close()


@pytest.mark.parametrize("nx,ny,nz,most", [(32, 600, 32, 1), (96, 600, 80, 2), (96, 40, 80, 9)])
def test_only_configurations_that_differ_are_timed(monkeypatch, nx, ny, nz, most):
    """FP64: register transforms with the register line solve have one
    configuration, products two z tiles, the staged line solve four column
    counts."""
    monkeypatch.delenv("IBP_TUNE_CACHE", raising=False)
    f = to_dev(np.random.default_rng(5).standard_normal((ny, nz, nx)))
    p = plan_of(nx, ny, nz, "fp64")
    assert 1 <= p.autotune(f)["tried"] <= most
    p.close()
