"""Edges of the fused smoothing passes' tiles, through the C ABI: lattices whose
width leaves 0 to 3 cells in the last strip of four, tile seams in x and y,
heights around the r.z partials' groups of eight planes, and coarser levels
with ragged last cells smoothed by the fused passes (a low coarse-solve
threshold), against one kernel per sweep.  The two compute the same V-cycle up
to FP32 rounding and the solves stop at a relative residual of 1e-10 (1e-8 in
precision 32), so the fields agree to 1e-12 (1e-6) and the iteration counts are
equal, as in the sweep-by-sweep comparison.  The depth of the tiles in z must
not change a bit of any result."""
import numpy as np
import pytest

from paper_2105_00448_amd import hca, synth

pytestmark = pytest.mark.gpu

SHAPES = [(9, 30, 57), (8, 63, 114), (17, 21, 62), (7, 70, 35), (33, 12, 121), (20, 100, 4), (10, 47, 3)]


def replicate(shape, seed):
    tis = synth.make_tissue(shape, 4, seed=seed)
    sched = synth.bolus_schedule([0, 2])
    return (tis.cell, tis.w, tis.seed, (sched.times, sched.amts))


def fields(reps, steps=3, **over):
    with hca.Simulation(reps, hca.default_params(x0_extrapolate=2, **over)) as sim:
        sim.step(steps)
        return ([{k: sim.field(k, r) for k in ("K", "G1", "G2", "L")} for r in range(len(reps))],
                list(sim.stats()["cg_iters"]))


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("coarse", [4096, 64])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_tile_edges_match_the_per_sweep_kernels(shape, coarse, precision):
    print(f"\n[fused tiles] {shape} coarse {coarse} precision {precision}", flush=True)
    rep = replicate(shape, sum(shape))
    (f0,), i0 = fields([rep], mg_fuse=0, mg_coarse_max=coarse, precision=precision)
    (f1,), i1 = fields([rep], mg_fuse=1, mg_coarse_max=coarse, precision=precision)
    assert i0 == i1
    tol = 1e-12 if precision == 64 else 1e-6
    for k in ("K", "G1", "G2"):
        assert np.abs(f1[k] - f0[k]).max() <= tol * np.abs(f0[k]).max(), k
    assert np.array_equal(f1["L"], f0["L"])


def test_tile_depth_does_not_change_a_bit(monkeypatch):
    """The r.z partials cover eight planes of a tile column at any depth."""
    reps = [replicate(s, 40 + i) for i, s in enumerate([(37, 30, 61), (16, 20, 33), (1, 50, 41)])]
    out = []
    for depth in (8, 16, 40):
        monkeypatch.setenv("HCA_FUSED_DEPTH", str(depth))
        out.append(fields(reps, mg_coarse_max=512)[0])
    monkeypatch.setenv("HCA_FUSED_DEPTH", "0")
    out.append(fields(reps, mg_coarse_max=512)[0])
    for other in out[1:]:
        for a, b in zip(out[0], other):
            for k in a:
                assert np.array_equal(a[k], b[k]), k


def test_shallow_tiles_do_not_change_a_bit(monkeypatch):
    """Lattices of up to 64^3 voxels: partials of four planes, tiles of four or
    more on every level, alone or beside a larger lattice (partials of eight)."""
    small = [replicate(s, 60 + i) for i, s in enumerate([(37, 30, 61), (16, 64, 64), (64, 64, 64), (3, 9, 20)])]
    alone = [fields([r], mg_coarse_max=512)[0][0] for r in small]
    batch = fields(small, mg_coarse_max=512)[0]
    mixed = fields(small + [replicate((65, 64, 64), 70)], mg_coarse_max=512)[0]
    monkeypatch.setenv("HCA_FUSED_DEPTH", "16")
    deep = fields(small, mg_coarse_max=512)[0]
    for i in range(len(small)):
        for other in (batch[i], mixed[i], deep[i]):
            for k in alone[i]:
                assert np.array_equal(alone[i][k], other[k]), (i, k)
