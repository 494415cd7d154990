"""The solves' ends from the kept z (precision 64): no iteration's z kept,
those of the first two, of the first four, in solves of fewer iterations and of
more than are kept.  From one state the forms differ by the order of the sums x_0 + sum alpha_k p_k alone, with terms that
shrink from iteration to iteration, so the fields agree to 1e-13 of their
largest value after one step and the iteration counts are equal."""
import numpy as np
import pytest

from paper_2105_00448_amd import hca, synth

pytestmark = pytest.mark.gpu


def replicates(shape):
    reps = []
    for i in range(2):
        tis = synth.make_tissue(shape, 4, seed=5 + i)
        sched = synth.bolus_schedule([0, 1])
        reps.append((tis.cell, tis.w, tis.seed, (sched.times, sched.amts)))
    return reps


def solve(keep, monkeypatch, reps, steps, states=None, **over):
    monkeypatch.setenv("HCA_CG_KEEP", str(keep))
    with hca.Simulation(reps, hca.default_params(**over), states=states) as sim:
        sim.step(steps)
        return [sim.field(k, r) for r in range(2) for k in ("K", "G1", "G2")], list(sim.stats(0)["cg_iters"])


@pytest.mark.parametrize("rtol", [1e-3, 1e-7, 1e-10, 1e-12])
@pytest.mark.parametrize("shape", [(9, 21, 34), (1, 40, 33), (3, 5, 7)], ids=str)
def test_kept_z_matches_the_updates_in_every_apply(shape, rtol, monkeypatch):
    """One step from one state: every solve starts from the same bits."""
    print(f"\n[kept z] {shape} {rtol}", flush=True)
    reps = replicates(shape)
    with hca.Simulation(reps, hca.default_params()) as sim:
        states = [sim.export_state(r) for r in range(2)]
    reps = [(None, None, seed, sched) for _, _, seed, sched in reps]
    ref, it_ref = solve(0, monkeypatch, reps, 1, states, cg_rtol=rtol, x0_extrapolate=0)
    for keep in (2, 4):
        out, it = solve(keep, monkeypatch, reps, 1, states, cg_rtol=rtol, x0_extrapolate=0)
        assert it == it_ref
        for a, b in zip(ref, out):
            assert np.abs(a - b).max() <= 1e-13 * np.abs(a).max()


def test_kept_z_with_substeps_and_newton(monkeypatch):
    """Solve after solve (theta-scheme substeps, Newton oxygen, fitted guesses),
    each of which starts from the last one's rounding: to 1e-12 at a relative
    residual of 1e-10, as in the sweep-by-sweep comparison."""
    for over in (dict(pde_substeps=4, pde_theta=0.5), dict(o2_newton=3)):
        ref, it_ref = solve(0, monkeypatch, replicates((8, 20, 30)), 3, **over)
        out, it = solve(4, monkeypatch, replicates((8, 20, 30)), 3, **over)
        assert it == it_ref
        for a, b in zip(ref, out):
            assert np.abs(a - b).max() <= 1e-12 * np.abs(a).max()
