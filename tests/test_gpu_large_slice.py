"""Precision 32 on a slice whose r.z column sums (one per voxel and field on one
plane) number more than 2^31.  The slice is made of mirrored copies of one
block, so that with no flux through its edges every block's fields are the
small slice's.  Both solves stop at a relative residual of 1e-8; the operators'
diagonals span less than four orders of magnitude, so the fields agree to 1e-4 of
their largest value."""
import numpy as np
import pytest
import torch

from paper_2105_00448_amd import hca, synth

pytestmark = pytest.mark.gpu

BLOCK, COPIES, FIELDS = 128, 162, 5


def mirrored(a, copies):
    """copies x copies blocks, each the mirror image of its neighbours."""
    two = np.concatenate([a, a[:, ::-1]], axis=1)
    two = np.concatenate([two, two[::-1]], axis=0)
    return np.tile(two, (copies // 2, copies // 2))


def test_more_than_2_31_column_sums():
    edge = BLOCK * COPIES
    assert FIELDS * edge * edge > 2 ** 31
    if torch.cuda.mem_get_info()[0] < 250 << 30:   # the FP64 initialisation of 4.3e8 voxels
        pytest.skip("needs 250 GiB of device memory")
    tis = synth.make_tissue((1, BLOCK, BLOCK), 4, seed=9)
    sched = synth.bolus_schedule([0, 1])

    def fields(copies):
        cell, w = mirrored(tis.cell[0], copies)[None], mirrored(tis.w[0], copies)[None]
        prm = hca.default_params(precision=32, vegf=1, drug3=1, x0_extrapolate=0)
        with hca.Simulation([(cell, w, tis.seed, (sched.times, sched.amts))], prm) as sim:
            print(f"\n[large slice] {cell.shape} initialised", flush=True)
            sim.run_phases(hca.PH_O2 | hca.PH_DRUGS | hca.PH_VEGF)
            print("[large slice] solved", flush=True)
            for k in ("K", "G1", "V"):
                yield k, sim.field(k)[0]

    small = dict(fields(2))
    for k, big in fields(COPIES):
        tile = 2 * BLOCK
        d = np.abs(big.reshape(COPIES // 2, tile, COPIES // 2, tile) - small[k][None, :, None, :]).max()
        assert d <= 1e-4 * np.abs(small[k]).max(), (k, d)
