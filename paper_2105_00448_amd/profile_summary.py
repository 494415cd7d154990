"""Summaries of rocprofv3 runs of a bench workload, written under profiles/.

Reads three rocprofv3 output folders of the same `bench.py --profile-only`
command (a kernel trace, a FETCH_SIZE pass and a WRITE_SIZE pass, each
started with `--copy-calibration 256` so that the runtime's copy of 256 MiB
calibrates the counters) and writes:

  <workload>_kernel_stats.md              per-kernel durations of the stepped context
  <kernel>_<workload>_traffic.{json,md}   HBM bytes per voxel of the solver's
                                          streaming kernels (CG and level-0
                                          multigrid), against their algorithmic bytes

Usage: python -m paper_2105_00448_amd.profile_summary WORKLOAD PRECISION KT_DIR FETCH_DIR WRITE_DIR COMMAND
"""
import collections
import csv
import glob
import hashlib
import json
import os
import re
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCES = ["paper_2105_00448_amd/csrc/k_solver.hip", "paper_2105_00448_amd/csrc/k_mg.hip",
           "paper_2105_00448_amd/csrc/dev_util.h", "paper_2105_00448_amd/csrc/hca_internal.h"]
COPY_KIB = 256 * 1024
# the counter passes collect only these dispatches (--kernel-include-regex)
PMC_REGEX = ("k_cg_start|k_cg_update|k_cg_apply|k_cg_finish|k_mg_pre|k_mg_sweep|k_mg_restrict|k_mg_post1|k_mg_post2|"
             "k_mg_postfused|k_mg_coarse|k_init_cells|copyBuffer")
# kernels priced per launch (levels below level 0, the one-workgroup coarse solve)
PER_LAUNCH = ["k_mg_prefused<2, true, false>", "k_mg_postfused<2, true, false, false, double>",
              "k_mg_prefused<2, true, true>", "k_mg_postfused<2, true, false, true, float>", "k_mg_pre<false, float>",
              "k_mg_restrict<false, float>", "k_mg_post1<false, float>",
              "k_mg_post2<false, float, double>", "k_mg_post2<false, float, float>", "k_mg_coarse"]
# voxels (of one system) of each workload, and its systems per solve
WORKLOADS = {"config5": (384 ** 3, 4), "plain128": (128 ** 3, 1)}


def kernels(e):
    """Streaming kernels of the solve (demangled-name prefix -> (short name,
    algorithmic bytes per active voxel)); e = bytes of a stored field value.
    Level 0 of the multigrid is the <true, ...> instance, or the fused
    three-stage passes k_mg_prefused<3, ...> / k_mg_postfused<3, ...> (the default).
    The apply and the solves' end move different bytes from iteration to iteration
    and are priced by cg_forms instead."""
    fp = "double" if e == 8 else "float"
    p32 = "false" if e == 8 else "true"   # the fused passes' precision flag
    return {
        f"k_cg_update<false, {fp}>": ("k_cg_update", 3 * e),
        "k_mg_pre<true, float>": ("k_mg_pre_L0", 12.0),
        "k_mg_sweep<true, float>": ("k_mg_sweep_L0", 16.0),
        "k_mg_restrict<true, float>": ("k_mg_restrict_L0", 12.5),
        "k_mg_post1<true, float>": ("k_mg_post1_L0", 16.5),
        f"k_mg_post2<true, {fp}, {fp}>": ("k_mg_post2_L0", 12 + e),
        f"k_mg_prefused<3, true, {p32}>": ("k_mg_prefused_L0", 12.5),
        f"k_mg_postfused<3, true, true, {p32}, {fp}>": ("k_mg_postfused_L0", 24.5 if e == 8 else 16.5),
    }


def kept_z():
    """Iterations whose z a precision-64 solve keeps (CgRing)."""
    src = open(os.path.join(ROOT, "paper_2105_00448_amd/csrc/hca_internal.h")).read()
    return int(re.search(r"constexpr int kZRing = (\d+);", src).group(1))


def cg_forms(fetch, write, e, kept):
    """Counted and algorithmic bytes of the apply's forms and of the solves' ends.

    ``fetch`` and ``write``: (kernel, bytes) of the same dispatches of
    k_cg_start, k_cg_apply, k_cg_update and k_cg_finish in launch order, one
    counter each; ``e`` bytes of a stored value, ``kept`` iterations of a solve
    keep z.  An iteration's update reads the same bytes per active voxel
    whatever its number, so its FETCH over the largest is the share of voxels
    still iterating.  Returns {form: [dispatches, share, FETCH, WRITE, algorithmic
    bytes x share]}, sums over the dispatches, the bytes per voxel of all systems:
    "first" (p = z), "kept" (x untouched), "x" (x += alpha p made too), "finish"."""
    price = {"first": 4 + 3 * e, "kept": 4 + 4 * e, "x": 4 + 6 * e}
    if [k for k, _ in fetch] != [k for k, _ in write]:
        raise SystemExit("the two counter passes launched different kernels")
    top = max(v for k, v in fetch if k == "k_cg_update")
    out, shares, pending = collections.defaultdict(lambda: [0, 0.0, 0.0, 0.0, 0.0]), [], None

    def add(form, share, f, w, bpv):
        o = out[form]
        for i, v in enumerate((1, share, f, w, bpv)):
            o[i] += v
    for (k, f), (_, w) in zip(fetch, write):
        if k == "k_cg_start":
            shares = []
        elif k == "k_cg_apply":
            pending = (f, w)
        elif k == "k_cg_update":
            share, it = f / top, len(shares)
            if share >= 0.02:   # (launches that found every system finished: left out)
                form = "first" if it == 0 else "kept" if it <= kept else "x"
                add(form, share, *pending, price[form] * share)
            shares.append(share)
        elif k == "k_cg_finish":
            at = shares + [0.0] * (kept + 1)
            add("finish", at[0], f, w, 2 * e * at[0] + 4 * sum(at[:kept]) + e * at[kept])
    return out


def name(r):
    return r["Kernel_Name"].split("(")[0].replace("void ", "").replace("hca::", "")


def one_csv(folder, suffix):
    hits = glob.glob(os.path.join(folder, "**", f"*{suffix}"), recursive=True)
    if len(hits) != 1:
        raise SystemExit(f"expected one *{suffix} under {folder}, found {hits}")
    return list(csv.DictReader(open(hits[0])))


def stepped_context(rows, key):
    """Dispatches after the last context initialisation (k_init_cells)."""
    rows = sorted(rows, key=lambda r: int(r[key]))
    last = max(i for i, r in enumerate(rows) if "k_init_cells" in r["Kernel_Name"])
    return rows, rows[last + 1:]


def pmc_command(command, counter):
    """The counter pass of the kernel-trace command `command`."""
    return (command.replace("--kernel-trace --stats",
                            f"--pmc {counter} --kernel-include-regex '{PMC_REGEX}'")
            .replace("P_kt", "P_f" if counter == "FETCH_SIZE" else "P_w"))


def main(workload, precision, kt_dir, f_dir, w_dir, command):
    e = 8 if int(precision) == 64 else 4
    ks = kernels(e)
    nvox, nrep = WORKLOADS[workload]
    tag = workload if e == 8 else f"{workload}_fp32"
    _, kt = stepped_context(one_csv(kt_dir, "kernel_trace.csv"), "Start_Timestamp")
    dur = collections.defaultdict(list)
    for r in kt:
        dur[name(r)].append((int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) / 1e3)
    total = sum(sum(v) for v in dur.values())
    span = (int(kt[-1]["End_Timestamp"]) - int(kt[0]["Start_Timestamp"])) / 1e6
    out = [f"# Kernel statistics: {tag} (multigrid-preconditioned CG, precision {precision})", "",
           "Command (repository root, one MI355X):", "", f"    {command}", "",
           "One context of the workload after its initialisation (warm-up and timed steps,",
           "captured CG iterations replayed as HIP graphs, then the profiled windows, kernels",
           "launched directly); durations are rocprofv3's",
           f"dispatch timestamps ({len(kt)} dispatches, span {span:.2f} ms, kernel time "
           f"{total / 1e3:.2f} ms).", "",
           "| kernel | calls | total ms | mean us | % |", "|---|---:|---:|---:|---:|"]
    for k, v in sorted(dur.items(), key=lambda kv: -sum(kv[1]))[:30]:
        out.append(f"| {k} | {len(v)} | {sum(v) / 1e3:.2f} | {sum(v) / len(v):.1f} | "
                   f"{100 * sum(v) / total:.1f} |")
    if workload == "config5":
        # bench.py's profiled windows close the run: every kernel class, the
        # dominant class alone (its event-timed launches give the roofline's
        # mean_launch_us), the surrogate alone; 3 steps each, k_stats ending
        # every step
        ends = [i for i, r in enumerate(kt) if name(r).startswith("k_stats")]
        if len(ends) >= 7:
            win = kt[ends[-7] + 1:ends[-4] + 1]
            wd = collections.defaultdict(list)
            for r in win:
                wd[name(r)].append((int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) / 1e3)
            out += ["", "The dominant-class window (the 3 steps bench.py times the dominant kernel "
                        "in, with HIP events on its launches; other classes run untimed).  Launches "
                        "that found every system finished (a few us: the replayed iteration pairs' "
                        "no-ops) are left out, as the library's timing leaves them out:", "",
                    "| kernel | launches | mean us |", "|---|---:|---:|"]
            for k, v in sorted(wd.items(), key=lambda kv: -sum(kv[1]))[:6]:
                real = [x for x in v if x >= 0.02 * max(v)]
                out.append(f"| {k} | {len(real)} | {sum(real) / len(real):.1f} |")
    open(os.path.join(ROOT, "profiles", f"{tag}_kernel_stats.md"), "w").write("\n".join(out) + "\n")

    def counters(folder):
        allr, ctx = stepped_context(one_csv(folder, "counter_collection.csv"), "Dispatch_Id")
        first = min(i for i, r in enumerate(allr) if "k_init_cells" in r["Kernel_Name"])
        copies = [float(r["Counter_Value"]) for r in allr[:first]
                  if "copyBuffer" in r["Kernel_Name"] and int(r["Grid_Size"]) > 100000]
        return ctx, copies
    F, cf = counters(f_dir)
    W, cw = counters(w_dir)
    ffac, wfac = COPY_KIB / (sum(cf) / len(cf)), COPY_KIB / (sum(cw) / len(cw))
    h = hashlib.sha256()
    for f in SOURCES:
        h.update(open(os.path.join(ROOT, f), "rb").read())
    table = ["| kernel | dispatches (all systems iterating) | FETCH B/voxel | WRITE B/voxel | "
             "measured B/voxel | algorithmic B/voxel | ratio |", "|---|---:|---:|---:|---:|---:|---:|"]
    vox = 3 * nvox * nrep

    def record(short, dispatches, fetch, write, bpv):
        """fetch, write: bytes per voxel."""
        rec = {"kernel": short, "workload": workload, "precision": int(precision), "sources": SOURCES,
               "sources_sha256": h.hexdigest(), "fetch_factor": ffac, "write_factor": wfac,
               "voxels_all_systems": vox, "dispatches": dispatches,
               "fetch_bytes_per_voxel": fetch, "write_bytes_per_voxel": write,
               "traffic_bytes_per_voxel": fetch + write, "algorithmic_bytes_per_voxel": bpv,
               "commands": [pmc_command(command, "FETCH_SIZE"), pmc_command(command, "WRITE_SIZE")]}
        json.dump(rec, open(os.path.join(ROOT, "profiles", f"{short}_{tag}_traffic.json"), "w"), indent=1)

    def row(label, dispatches, fetch, write, bpv):
        return (f"| {label} | {dispatches} | {fetch:.2f} | {write:.2f} | {fetch + write:.2f} | "
                f"{bpv:.1f} | {(fetch + write) / bpv:.3f} |")
    for full, (short, bpv) in ks.items():
        fd = [float(r["Counter_Value"]) for r in F if name(r) == full]
        wd = [float(r["Counter_Value"]) for r in W if name(r) == full]
        if not fd:
            continue
        fall = [v for v in fd if v >= 0.9 * max(fd)]   # every system still iterating
        wall = sorted(wd, reverse=True)[:len(fall)]
        fetch = sum(fall) / len(fall) * 1024 * ffac / vox
        write = sum(wall) / len(wall) * 1024 * wfac / vox
        record(short, len(fall), fetch, write, bpv)
        table.append(row(full, len(fall), fetch, write, bpv))
    # the apply's forms and the solves' ends, per active voxel of every dispatch
    fp = "double" if e == 8 else "float"
    cg = {f"k_cg_start<{fp}>": "k_cg_start", f"k_cg_apply<false, {fp}>": "k_cg_apply",
          f"k_cg_update<false, {fp}>": "k_cg_update", f"k_cg_finish<{fp}>": "k_cg_finish"}
    forms = cg_forms(*[[(cg[name(r)], float(r["Counter_Value"]) * 1024 * fac) for r in rows if name(r) in cg]
                       for rows, fac in ((F, ffac), (W, wfac))], e, kept_z() if e == 8 else 0)
    ftable = [table[0].replace("dispatches (all systems iterating)", "dispatches").replace("voxel", "active voxel"),
              table[1]]

    def per_voxel(o):
        return o[0], o[2] / (o[1] * vox), o[3] / (o[1] * vox), o[4] / o[1]
    for form in ("first", "kept", "x"):
        if form in forms:
            ftable.append(row(f"k_cg_apply, {form}", *per_voxel(forms[form])))
    apply_all = [sum(v) for v in zip(*(forms[k] for k in ("first", "kept", "x") if k in forms))]
    ftable.append(row("k_cg_apply, all", *per_voxel(apply_all)))
    record("k_cg_apply", *per_voxel(apply_all))
    if "finish" in forms:
        ftable.append(row("k_cg_finish", *per_voxel(forms["finish"])))
        record("k_cg_finish", *per_voxel(forms["finish"]))
    small = ["| kernel | dispatches | mean us | FETCH KiB/dispatch | WRITE KiB/dispatch | GB/s |",
             "|---|---:|---:|---:|---:|---:|"]
    for full in PER_LAUNCH:
        fd = [float(r["Counter_Value"]) for r in F if name(r) == full]
        wd = [float(r["Counter_Value"]) for r in W if name(r) == full]
        du = dur.get(full, [])
        if not fd or not wd or not du:
            continue
        fk, wk, us = sum(fd) / len(fd) * ffac, sum(wd) / len(wd) * wfac, sum(du) / len(du)
        small.append(f"| {full} | {len(fd)} | {us:.1f} | {fk:.0f} | {wk:.0f} | "
                     f"{(fk + wk) * 1024 / (us * 1e-6) / 1e9:.0f} |")
    md = [f"# HBM traffic of the solver's streaming kernels: {tag}", "",
          "Commands (repository root, one MI355X), one counter per run:", "",
          "    " + pmc_command(command, "FETCH_SIZE"),
          "    " + pmc_command(command, "WRITE_SIZE"), "",
          "Calibration: `--copy-calibration 256` first copies 256 MiB device to device (the",
          f"runtime's blit kernel); per copy FETCH_SIZE reads {sum(cf) / len(cf):.0f} KiB and WRITE_SIZE",
          f"{sum(cw) / len(cw):.0f} KiB for {COPY_KIB} KiB moved each way: scale factors",
          f"{ffac:.3f} (fetch) and {wfac:.3f} (write).", "",
          f"Per voxel of all {3 * nrep} systems ({3 * nvox * nrep} voxels), on the dispatches where every",
          "system still iterates (counter within 10 % of the kernel's largest; later",
          "dispatches skip finished systems):", ""] + table + [
          "", "The CG's apply by its forms (a solve's first: p = z; x untouched, z kept; x += alpha p",
          "made too) and the solves' ends, per active voxel of every dispatch that had one (the",
          "share of voxels still iterating from the update of the same iteration; the end's",
          "algorithmic bytes from the solve's own iterations):", ""] + ftable + [
          "", "Kernels below level 0 (latency-bound: bytes per dispatch over all systems, mean",
          "duration from the kernel trace, effective rate):", ""] + small + [
          "", "`profiles/<kernel>_" + tag + "_traffic.json` hold these numbers with the SHA-256 of the",
          "solver's sources; `bench.py` reports them as `roofline.traffic` only while those",
          "sources are unchanged."]
    open(os.path.join(ROOT, "profiles", f"solver_{tag}_traffic.md"), "w").write("\n".join(md) + "\n")
    print(f"wrote profiles/{tag}_kernel_stats.md, profiles/solver_{tag}_traffic.md and the json records")


if __name__ == "__main__":
    if len(sys.argv) != 7:
        raise SystemExit(__doc__)
    main(*sys.argv[1:])
