"""The traffic records price each dispatch of the CG's apply by what its
iteration moves (a solve's first, z kept, x updated too) and each solve's end by
the iterations that it sums, over the voxels still iterating: counters of
known bytes give back those bytes, and the committed records' counted traffic
exceeds the algorithmic bytes by halo reads alone (for a stencil over planes of
tiles at most a third, for the pointwise end a tenth)."""
import json
import os

import pytest

from paper_2105_00448_amd import profile_summary as ps

PROFILES = os.path.join(ps.ROOT, "profiles")


def solve(iters, e, kept, noop):
    """Dispatches of one solve of systems that stop after `iters` iterations
    (of one size each), with `noop` launches that find every system finished."""
    fetch, write = [("k_cg_start", 0.0)], [("k_cg_start", 0.0)]
    n = len(iters)
    for it in range(max(iters) + noop):
        act = sum(i > it for i in iters) / n
        read = 4 + e if it == 0 else 4 + 2 * e
        x = e if it > kept else 0
        fetch += [("k_cg_apply", act * (read + x)), ("k_cg_update", act * 2 * e)]
        write += [("k_cg_apply", act * (2 * e + x)), ("k_cg_update", act * (e + 4))]
    fetch.append(("k_cg_finish", sum((e + 4 * min(i, kept) + (e if i > kept else 0)) for i in iters) / n))
    write.append(("k_cg_finish", float(e)))
    return fetch, write


@pytest.mark.parametrize("e,kept", [(8, 3), (8, 2), (8, 0), (4, 0)])
def test_counters_of_known_bytes(e, kept):
    fetch, write = [], []
    for iters, noop in (((6, 2, 3), 1), ((1, 1, 1), 0), ((4, 4, 9), 2), ((3, 1, 1), 3)):
        f, w = solve(iters, e, kept, noop)
        fetch += f
        write += w
    forms = ps.cg_forms(fetch, write, e, kept)
    assert set(forms) == ({"first", "kept", "x", "finish"} if kept else {"first", "x", "finish"})
    for form, (n, share, f, w, bpv) in forms.items():
        assert n > 0 and 0 < share <= n
        assert f + w == pytest.approx(bpv, rel=1e-12), form
    assert forms["first"][4] == pytest.approx(forms["first"][1] * (4 + 3 * e))
    assert forms["x"][4] == pytest.approx(forms["x"][1] * (4 + 6 * e))


@pytest.mark.parametrize("kernel,tag,lo,hi,most", [
    ("k_cg_apply", "config5", 28, 52, 4 / 3), ("k_cg_apply", "plain128", 28, 52, 4 / 3),
    ("k_cg_apply", "config5_fp32", 16, 28, 4 / 3), ("k_cg_finish", "config5", 20, 36, 1.1),
    ("k_cg_finish", "plain128", 20, 36, 1.1)])
def test_committed_records(kernel, tag, lo, hi, most):
    rec = json.load(open(os.path.join(PROFILES, f"{kernel}_{tag}_traffic.json")))
    assert lo <= rec["algorithmic_bytes_per_voxel"] <= hi
    assert 1 / most <= rec["traffic_bytes_per_voxel"] / rec["algorithmic_bytes_per_voxel"] <= most
