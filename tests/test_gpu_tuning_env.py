"""A tuning variable of the environment holds for the contexts made while it is
set and for no later one: the stencil tiles' depth by hca_tile_shape, the fused
smoothing passes' by their kernels' times (a 128^3 lattice in one slab of 128
planes leaves most of the chip idle: more than twice the default's time)."""
import pytest

from paper_2105_00448_amd import hca, synth

pytestmark = pytest.mark.gpu


def replicate(shape):
    tis = synth.make_tissue(shape, 4, seed=sum(shape))
    sched = synth.bolus_schedule([0, 1])
    return (tis.cell, tis.w, tis.seed, (sched.times, sched.amts))


# (shape, default depth in precision 64): either side of both lines of the rule
DEPTHS = [((20, 30, 27), 4), ((16, 32, 32), 4), ((17, 32, 32), 8), ((64, 32, 32), 8), ((65, 32, 32), 16)]


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("shape,depth", DEPTHS, ids=str)
def test_tile_depth_holds_while_it_is_set(shape, depth, precision, monkeypatch):
    def tz():
        with hca.Simulation([replicate(shape)], hca.default_params(precision=precision)) as sim:
            return sim.tile_shape()[2]
    default = min(depth if precision == 64 else 16, shape[0])
    assert tz() == default
    for knob in (2, 12, 16):
        monkeypatch.setenv("HCA_TILE_DEPTH", str(knob))
        assert tz() == min(knob, shape[0])
        monkeypatch.delenv("HCA_TILE_DEPTH")
        assert tz() == default


def fused_us(rep, **over):
    """Microseconds of level 0's pre- and post-smoothing."""
    with hca.Simulation([rep], hca.default_params(profile=1, **over)) as sim:
        sim.step(1)
        sim.reset_kernel_times()
        sim.step(2)
        kt = sim.kernel_times()
        return sum(kt[k]["ms"] / kt[k]["launches"] * 1e3 for k in ("k_mg_prefused<L0>", "k_mg_postfused<L0>"))


def test_fused_depth_holds_while_it_is_set(monkeypatch):
    rep = replicate((128, 128, 128))
    us = lambda: fused_us(rep)
    us()
    before = us()
    monkeypatch.setenv("HCA_FUSED_DEPTH", "1024")
    forced = us()
    monkeypatch.delenv("HCA_FUSED_DEPTH")
    after = us()
    print(f"\n[fused depth] default {before:.1f} us, one slab {forced:.1f}, default again {after:.1f}", flush=True)
    assert forced >= 1.5 * before
    assert after <= 1.25 * before


@pytest.mark.parametrize("precision", [64, 32])
@pytest.mark.parametrize("knob,value", [("HCA_FUSED_MIN", "64"), ("HCA_FUSED_TARGET", "1")])
def test_fused_tiles_aimed_at(knob, value, precision, monkeypatch):
    """Both give tiles of 64 planes (16 by default): half the chip and more idle."""
    rep = replicate((128, 128, 128))
    fused_us(rep, precision=precision)
    before = fused_us(rep, precision=precision)
    monkeypatch.setenv(knob, value)
    forced = fused_us(rep, precision=precision)
    monkeypatch.delenv(knob)
    after = fused_us(rep, precision=precision)
    print(f"\n[{knob}] precision {precision}: default {before:.1f} us, 64 planes {forced:.1f}, default again {after:.1f}",
          flush=True)
    assert forced >= 1.5 * before
    assert after <= 1.25 * before
