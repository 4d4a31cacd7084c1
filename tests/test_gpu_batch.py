"""Batched solves of many uneven grids: one launch per solve stage covering
every grid (ibp_batch_* and ibp_solve_batched).  GPU only."""

import numpy as np
import pytest
import torch

import oracle
from oracle.grid import geometry
from oracle.operators import divergence
from paper_2609_19130_amd import ibpoisson as ibp
from paper_2609_19130_amd import synth

from gpu_helpers import rel, require_gpu, to_dev
from test_gpu_parity import TOL_MIXED_VS_FP64, residual

pytestmark = pytest.mark.gpu

TOL64 = 1e-12
REG_LENGTHS = {32, 64, 128, 256, 512, 1024}   # lengths the single-grid path transforms in registers


def line_solve_shape(ny):
    """(lanes, rows per lane) of a single grid's line solve: 32 lanes up to
    ny = 384, then 64; rows from 2, 4, 8, 12, 16, 24."""
    lanes = 64 if ny > 384 else 32
    need = -(-ny // lanes)
    return lanes, next(k for k in (2, 4, 8, 12, 16, 24) if k >= need)


def batch_rows(ny, lanes, kmax):
    """Rows per lane of one grid inside a batch whose largest ny gives
    (lanes, kmax): kmax/4 or kmax/2 where that holds ny, else kmax."""
    need = -(-ny // lanes)
    if kmax % 4 == 0 and need <= kmax // 4:
        return kmax // 4
    if kmax % 2 == 0 and need <= kmax // 2:
        return kmax // 2
    return kmax


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def batch_case(count=64, seed=4, precision="fp64", max_iters=4):
    grids = synth.batch_grids(seed=seed, count=count)
    plans, rhs, fs = [], [], []
    for gd in grids:
        yf = synth.tanh_faces(gd["ny"], gd["beta"])
        g = geometry(gd["nx"], gd["ny"], gd["nz"], gd["Lx"], gd["Lz"], yf)
        u, v, w = synth.uniform_velocity(gd["nx"], gd["ny"], gd["nz"], seed=gd["seed"])
        f = divergence(u, v, w, g)
        fs.append((f, yf))
        plans.append(ibp.Plan(gd["nx"], gd["ny"], gd["nz"], gd["Lx"], gd["Lz"], yf,
                              precision=precision, max_iters=max_iters))
        rhs.append(to_dev(f))
    return grids, plans, rhs, fs


@pytest.fixture(scope="module")
def c4():
    return batch_case()


def test_batched_fp64_matches_single_and_oracle(c4):
    """64 uneven grids in one launch per stage: every grid within 1e-12 of
    its single solve, bitwise where the single solve uses the same
    arithmetic (mixed-radix transforms and the batch's rows per lane), and
    within 1e-12 of the oracle on 8 grids."""
    grids, plans, rhs, fs = c4
    phis = [torch.empty_like(r) for r in rhs]
    ibp.solve_batched(plans, rhs, phis)
    torch.cuda.synchronize()
    lanes, kmax = line_solve_shape(max(gd["ny"] for gd in grids))
    same = 0
    for i, (p, r) in enumerate(zip(plans, rhs)):
        single = p.solve(r)
        gd = grids[i]
        assert float(torch.linalg.vector_norm(single - phis[i]) / torch.linalg.vector_norm(single)) <= TOL64, i
        if (gd["nx"] // 2 not in REG_LENGTHS and gd["nz"] not in REG_LENGTHS
                and line_solve_shape(gd["ny"]) == (lanes, batch_rows(gd["ny"], lanes, kmax))):
            same += 1
            assert torch.equal(single, phis[i]), f"grid {i}: batched differs from single"
    assert same >= 3
    for i in range(0, 64, 8):
        f, yf = fs[i]
        gd = grids[i]
        ref, _ = oracle.solve(f, gd["Lx"], gd["Lz"], yf)
        assert rel(phis[i].cpu().numpy(), ref) <= TOL64, (i, gd)


def test_batch_object_graph_and_ycols(c4):
    """The explicit batch gives the cached path's bits, under graph capture
    (every replay) and for every line-solve column count."""
    grids, plans, rhs, _ = c4
    ref = [torch.empty_like(r) for r in rhs]
    ibp.solve_batched(plans, rhs, ref)
    b = ibp.Batch(plans)
    out = b.solve(rhs)
    torch.cuda.synchronize()
    assert all(torch.equal(a, c) for a, c in zip(ref, out))
    for cols in (2, 4, 16, 8):
        b.set_ycols(cols)
        out = b.solve(rhs)
        torch.cuda.synchronize()
        assert all(torch.equal(a, c) for a, c in zip(ref, out)), cols
    inp = [r.clone() for r in rhs]
    outg = [torch.empty_like(r) for r in rhs]
    b.solve(inp, outg)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.solve(inp, outg)
    for k in range(3):
        scale = float(2 ** (k + 1))   # powers of two scale every intermediate exactly
        for a, r in zip(inp, rhs):
            a.copy_(r * scale)
        for o in outg:
            o.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i in range(len(rhs)):
            assert torch.equal(outg[i], ref[i] * scale), (k, i)
    b.close()


def test_batched_mixed_converges_per_grid():
    """Every grid of a mixed batch: converged, its residual recomputed here
    with the oracle's operator (<= 1e-10 and equal to the reported one), and
    its solution against the oracle within the mixed error bound."""
    grids, plans, rhs, fs = batch_case(count=24, seed=9, precision="mixed", max_iters=6)
    phis = [torch.empty_like(r) for r in rhs]
    ibp.solve_batched(plans, rhs, phis)
    torch.cuda.synchronize()
    for i, p in enumerate(plans):
        info = p.info()
        assert info["converged"] == 1 and info["rel_residual"] <= 1e-10, (i, info)
        f, yf = fs[i]
        gd = grids[i]
        phi = phis[i].cpu().numpy()
        r = residual(f, phi, gd["Lx"], gd["Lz"], yf)
        assert r <= 1e-10, (i, r)
        assert abs(info["rel_residual"] - r) <= 0.05 * r + 1e-15, (i, r, info["rel_residual"])
        ref, _ = oracle.solve(f, gd["Lx"], gd["Lz"], yf)
        assert rel(phi, ref) <= TOL_MIXED_VS_FP64, (i, gd, rel(phi, ref), r)


def test_batched_more_than_max_and_stale_batch():
    """70 grids run as a batch of 64 and a batch of 6; a batch whose plan
    changed precision refuses to run; a mixed-precision sequence falls back
    to one solve after another."""
    grids, plans, rhs, _ = batch_case(count=70, seed=11)
    phis = ibp.solve_batched(plans, rhs, [torch.empty_like(r) for r in rhs])
    torch.cuda.synchronize()
    for i in (0, 63, 64, 69):
        single = plans[i].solve(rhs[i])
        assert float(torch.linalg.vector_norm(single - phis[i]) / torch.linalg.vector_norm(single)) <= TOL64
    b = ibp.Batch(plans[:4])
    plans[1].set_precision("mixed", 1e-10, 4)
    with pytest.raises(ibp.IbpError) as e:
        b.solve(rhs[:4])
    assert e.value.status == ibp.INVALID_VALUE
    b.close()
    out = ibp.solve_batched(plans[:4], rhs[:4], [torch.empty_like(r) for r in rhs[:4]])   # loop fallback
    torch.cuda.synchronize()
    for i in range(4):
        assert plans[i].info()["converged"] == 1
        assert torch.isfinite(out[i]).all()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_autotune_is_bitwise_neutral(precision):
    """Autotuning picks work splits by timing; the solution bits do not
    depend on the choice (single plans and batches)."""
    grids, plans, rhs, _ = batch_case(count=12, seed=13, precision=precision)
    ref = [p.solve(r) for p, r in zip(plans, rhs)]
    torch.cuda.synchronize()
    for p, r, a in zip(plans[:4], rhs[:4], ref[:4]):
        t = p.autotune(r)
        assert t["tried"] >= 5 and t["ms"] > 0 and t["ycols"] in (0, 2, 4, 8, 16)   # 0: default shape kept
        assert torch.equal(p.solve(r), a)
    b = ibp.Batch(plans)
    before = b.solve(rhs)
    t = b.autotune(rhs)
    assert t["tried"] >= 13 and t["ms"] <= t["ms_before"] * 1.5
    if precision == "mixed":
        assert t["xdiv"] == 1
    after = b.solve(rhs)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(before, after))
    b.close()


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_batch_with_a_tall_grid_runs_every_line_solve_class(precision):
    """One grid taller than 384 rows puts the whole batch on 64-lane line
    solves (8 rows per lane); the others run 4 or 2 rows per lane in launches
    of their own, and a grid of 6 rows takes fewer (0,0)-mode blocks than the
    default.  Every grid against its single solve and the oracle."""
    dims = [(48, 400, 40), (40, 130, 24), (32, 40, 48), (24, 6, 16), (30, 250, 20)]
    assert line_solve_shape(max(d[1] for d in dims)) == (64, 8)
    assert sorted({batch_rows(d[1], 64, 8) for d in dims}) == [2, 4, 8]
    plans, rhs, fs = [], [], []
    try:
        for i, (nx, ny, nz) in enumerate(dims):
            yf = synth.tanh_faces(ny, 2.0)
            g = geometry(nx, ny, nz, 2 * np.pi, 1.3, yf)
            u, v, w = synth.uniform_velocity(nx, ny, nz, seed=60 + i)
            f = divergence(u, v, w, g)
            fs.append((f, yf))
            plans.append(ibp.Plan(nx, ny, nz, 2 * np.pi, 1.3, yf, precision=precision, max_iters=6))
            rhs.append(to_dev(f))
        outs = ibp.solve_batched(plans, rhs, [torch.empty_like(r) for r in rhs])
        torch.cuda.synchronize()
        tol = TOL64 if precision == "fp64" else 1e-8
        for i, (p, r) in enumerate(zip(plans, rhs)):
            if precision == "mixed":
                assert p.info()["converged"] == 1
            single = p.solve(r)
            assert float(torch.linalg.vector_norm(single - outs[i]) / torch.linalg.vector_norm(single)) <= tol, i
            f, yf = fs[i]
            ref, _ = oracle.solve(f, 2 * np.pi, 1.3, yf)
            assert rel(outs[i].cpu().numpy(), ref) <= tol, (i, dims[i])
    finally:
        for p in plans:
            p.close()


TALL_DIMS = [(48, 400, 40), (40, 130, 24), (32, 40, 48), (24, 6, 16), (30, 250, 20), (64, 20, 1)]


def tall_case(precision):
    plans, rhs = [], []
    for i, (nx, ny, nz) in enumerate(TALL_DIMS):
        yf = synth.tanh_faces(ny, 2.0)
        f = np.random.default_rng(80 + i).standard_normal((ny, nz, nx))
        plans.append(ibp.Plan(nx, ny, nz, 2 * np.pi, 1.3, yf, precision=precision, max_iters=4))
        rhs.append(to_dev(f))
    return plans, rhs


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("case", ["c4", "tall"])
def test_persistent_schedule_matches_staged(precision, case):
    """The whole batched solve as one persistent launch (grids pinned to XCD
    queues, stages overlapped across grids) gives bitwise the results of one
    launch per stage, on every grid, on repeated solves (the queue counters
    re-arm at the end of each launch) and under graph capture: the 64-grid
    workload (32-lane line solves, 8 rows) and a batch with a 400-row grid
    (64 lanes, the K, K/2 and K/4 classes, a 6-row grid, one nz = 1 grid)."""
    if case == "c4":
        _, plans, rhs, _ = batch_case(count=64 if precision == "fp64" else 24, seed=4 if precision == "fp64" else 9,
                                      precision=precision, max_iters=4)
    else:
        plans, rhs = tall_case(precision)
    b = ibp.Batch(plans)
    b.set_persistent(False)
    staged = b.solve(rhs)
    torch.cuda.synchronize()
    b.set_persistent(True)
    for rep in range(3):
        out = b.solve(rhs)
        torch.cuda.synchronize()
        for i in range(len(rhs)):
            assert torch.equal(out[i], staged[i]), (rep, i)
        for p in plans:
            info = p.info()   # raises if a queue wait gave up
            if precision == "mixed":
                assert info["converged"] == 1, info
    inp = [r.clone() for r in rhs]
    outg = [torch.empty_like(r) for r in rhs]
    b.solve(inp, outg)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b.solve(inp, outg)
    for k in range(3):
        scale = float(2 ** (k + 1))
        for a, r in zip(inp, rhs):
            a.copy_(r * scale)
        for o in outg:
            o.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i in range(len(rhs)):
            assert torch.equal(outg[i], staged[i] * scale), (k, i)
    b.close()
    for p in plans:
        p.close()


def test_tuning_cache(monkeypatch, tmp_path):
    """Tuned choices persist in the IBP_TUNE_CACHE file (one JSON line per
    key: architecture, dimensions, precision): a second plan or batch of the
    same dimensions takes the cached choice without a search, plans pick it
    up when created, and the bits do not change."""
    import json
    cache = tmp_path / "tune.jsonl"
    monkeypatch.setenv("IBP_TUNE_CACHE", str(cache))
    nx, ny, nz = 96, 40, 48   # general (LDS) x and z transforms: the tile choice applies
    yf = synth.tanh_faces(ny, 2.0)
    f = to_dev(np.random.default_rng(21).standard_normal((ny, nz, nx)))
    a = ibp.Plan(nx, ny, nz, 2 * np.pi, 1.0, yf)
    ref = a.solve(f).clone()
    t1 = a.autotune(f)
    assert t1["tried"] >= 8 and t1["xsmall"] in (0, 1) and t1["zsmall"] in (0, 1), t1
    lines = [json.loads(l) for l in cache.read_text().splitlines()]
    assert len(lines) == 1 and lines[0]["key"].endswith(f"/plan/{nx}x{ny}x{nz}/0"), lines
    assert lines[0]["ycols"] == t1["ycols"] and lines[0]["zdiv"] == t1["zdiv"]
    b = ibp.Plan(nx, ny, nz, 2 * np.pi, 1.0, yf)   # created with the cached choice
    assert torch.equal(b.solve(f), ref)
    t2 = b.autotune(f)
    assert t2["tried"] == 0 and all(t2[k] == t1[k] for k in ("zdiv", "ycols", "xsmall", "zsmall")), (t1, t2)
    assert torch.equal(b.solve(f), ref)
    # batches
    grids, plans, rhs, _ = batch_case(count=6, seed=17)
    bt = ibp.Batch(plans)
    base = bt.solve(rhs)
    t3 = bt.autotune(rhs)
    assert t3["tried"] >= 13
    bt2 = ibp.Batch(plans)
    t4 = bt2.autotune(rhs)
    assert t4["tried"] == 0 and all(t4[k] == t3[k] for k in ("xdiv", "zdiv", "persistent")), (t3, t4)
    out = bt2.solve(rhs)
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(base, out))
    assert len(cache.read_text().splitlines()) == 2
    for o in (bt, bt2):
        o.close()
    for p in plans + [a, b]:
        p.close()


@pytest.mark.parametrize("dims", [[(126, 70, 132)], [(126, 70, 132), (256, 80, 10)],
                                  [(8 + 2 * i, 66 + i, 10 + i % 3) for i in range(4)] + [(154, 90, 121)] * 3,
                                  [(20 + 4 * i, 70 - i, (16, 18, 20, 22)[i % 4]) for i in range(8)],
                                  [(20 + 4 * i, 70 - i, (16, 18, 20, 22)[i % 4]) for i in range(8)] + [(56, 100, 48)]],
                         ids=["1", "2-general", "7-general", "8-products", "9-products"])
def test_batch_sizes_on_both_sides_of_the_grid_search(dims):
    """Grid search by scalar loads (up to 8 grids) and by ballot; batches
    without and with matrix-product lines (a persistent kernel each): staged
    and persistent alike to the bit, and every grid against its single solve."""
    plans, rhs = [], []
    for i, (nx, ny, nz) in enumerate(dims):
        f = np.random.default_rng(90 + i).standard_normal((ny, nz, nx))
        plans.append(ibp.Plan(nx, ny, nz, 2 * np.pi, 1.3, synth.tanh_faces(ny, 2.0)))
        rhs.append(to_dev(f))
    b = ibp.Batch(plans)
    b.set_persistent(False)
    staged = b.solve(rhs)
    b.set_persistent(True)
    out = b.solve(rhs)
    torch.cuda.synchronize()
    for i, (p, r) in enumerate(zip(plans, rhs)):
        assert torch.equal(out[i], staged[i]), dims[i]
        single = p.solve(r)
        assert float(torch.linalg.vector_norm(single - out[i]) / torch.linalg.vector_norm(single)) <= TOL64, dims[i]
    b.close()
    for p in plans:
        p.close()
