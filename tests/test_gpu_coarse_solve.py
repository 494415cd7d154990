"""The one-workgroup coarse solve at the edges of its forms, through the C ABI:
one to six cells a thread of its first level, whole and ragged cells, lattices
of one plane, rows and columns (more than 1024 cells on its second level), the
one-cell level alone.  The reference is the same V-cycle with one kernel per
sweep on every level down to the last (coarse threshold 1).  The two agree up
to FP32 rounding and the solves stop at a relative residual of 1e-10, so the
fields agree to 1e-12 and the iteration counts are equal, as in the
sweep-by-sweep comparison."""
import numpy as np
import pytest

from paper_2105_00448_amd import hca, synth

pytestmark = pytest.mark.gpu

# first level of the coarse solve: cells a thread
SHAPES = [
    (9, 14, 19), (24, 24, 24), (26, 30, 28), (32, 30, 33), (34, 34, 33),          # 1, 2, 3, 4, 6
    (1, 40, 50), (1, 70, 100), (1, 100, 100), (1, 128, 126), (1, 131, 129),       # the same, one plane
    (1, 1, 5600), (5600, 1, 1), (1, 3000, 2),                                     # rows and columns
    (2, 2, 2), (3, 2, 1), (70, 40, 64),
]


def solve(shape, coarse_max):
    tis = synth.make_tissue(shape, 4, seed=sum(shape))
    sched = synth.bolus_schedule([0, 1])
    with hca.Simulation([(tis.cell, tis.w, tis.seed, (sched.times, sched.amts))],
                        hca.default_params(x0_extrapolate=0, mg_fuse=0, mg_coarse_max=coarse_max)) as sim:
        sim.step(2)
        return {k: sim.field(k) for k in ("K", "G1", "G2", "L")}, list(sim.stats()["cg_iters"])


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_coarse_solve_matches_the_per_sweep_kernels(shape):
    print(f"\n[coarse solve] {shape}", flush=True)
    ref, it_ref = solve(shape, 1)
    out, it = solve(shape, 8192)
    assert it == it_ref
    for k in ("K", "G1", "G2"):
        assert np.abs(out[k] - ref[k]).max() <= 1e-12 * np.abs(ref[k]).max(), k
    assert np.array_equal(out["L"], ref["L"])
