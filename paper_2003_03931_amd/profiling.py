"""Turn rocprofv3 output into the short text summaries kept under profiles/.

* ``stats``: per-kernel call counts and mean durations from a
  ``rocprofv3 --kernel-trace --stats --output-format csv`` run.
* ``traffic``: HBM bytes of one execution of every step stage (all of its
  kernels together) from two ``--pmc FETCH_SIZE`` / ``--pmc WRITE_SIZE`` runs, each counter scaled by what
  it reads for a plain device copy of known size in the same run (the bench's
  ``--calibrate-copy`` step), so the numbers are bytes, not counter units.

bench.py reads the newest traffic summary for its dominant kernel when the
summary's source digest matches the current kernels (otherwise traffic is
reported as null).

Usage:
  python -m paper_2003_03931_amd.profiling stats <kernel_stats.csv> <out.txt> <command...>
  python -m paper_2003_03931_amd.profiling traffic <fetch_dir> <write_dir> <copy_bytes> <out.txt> <command...>
"""

import csv
import glob
import hashlib
import os
import re
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
PROFILES = os.path.join(ROOT, "profiles")

# step stage (cube_profile_read name) -> patterns of the kernel that begins an
# execution of it, of the kernels that may follow, and of one that must be among
# them.  P(k) and the sort launch transforms and scans of their own, without
# the kernel that must be there.
STAGE_KERNELS = {
    "coarse_deposit": (r"k_coarse_deposit", None, None),
    "coarse_fft_green": (r"k_fft<\d+, 0, 0>|k_fft_xy<\d+, false, false>", r"k_fft<|k_fft_xy<", r"k_fft<\d+, 2, 2>"),
    "fine_deposit": (r"k_deposit_zm<|k_deposit<\d+, false", None, None),
    "fine_r2c_xy": (r"k_r2c_plane", None, None),
    "fine_z_green": (r"k_zconv_half", None, None),
    "fine_c2r_xy": (r"k_c2r_plane", None, None),
    "gather_kick_drift": (r"k_gather<0,", None, None),
    "scan_counts": (r"k_cell_stats", r"k_tile_sums|k_tile_scan|k_decide", r"k_tile_scan"),
    "compact": (r"k_compact_brick", None, None),
    "velocity_encode": (r"k_vc_mean", r"k_vc_sigma|k_vc_encode", r"k_vc_encode"),
    "pp_force": (r"k_pp", None, None),
}
COPY_KERNELS = ("elementwise", "copyBuffer")


# sources whose kernels the profiled plain step never launches: the
# extended PP force (pp_range > 0), the cell-mean velocity codec
# (vel_codec = 1), the request server and the ensemble runner
NOT_IN_STEP = ("pp.hip", "vcodec.hip", "server.cpp", "ensemble.cpp")


_COMMENT = re.compile(r"//[^\n]*|/\*.*?\*/", re.S)


def _code_of(text):
    """Source text without comments and blank lines: what the compiler sees,
    so that a comment edit does not invalidate a summary."""
    lines = (ln.rstrip() for ln in _COMMENT.sub("", text).splitlines())
    return "\n".join(ln for ln in lines if ln)


def source_digest(root=None):
    """Digest of the code of the profiled step's kernels (comments ignored): a
    traffic summary is valid only for them."""
    h = hashlib.sha256()
    for f in sorted(glob.glob(os.path.join(root or HERE, "csrc", "*"))):
        if os.path.basename(f) in NOT_IN_STEP:
            continue
        with open(f, encoding="utf-8") as fh:
            h.update(os.path.basename(f).encode())
            h.update(_code_of(fh.read()).encode())
    return h.hexdigest()[:16]


def short_name(k):
    return k.replace("cube::(anonymous namespace)::", "").replace("void ", "").split("(")[0]


def stats_summary(csv_path, out_path, command):
    rows = list(csv.DictReader(open(csv_path)))
    rows.sort(key=lambda r: -float(r["TotalDurationNs"]))
    lines = [f"# rocprofv3 kernel stats", f"# command: {command}", f"# source digest: {source_digest()}",
             f"{'kernel':44s} {'calls':>7s} {'avg_us':>11s} {'total_ms':>10s} {'pct':>6s}"]
    for r in rows[:25]:
        lines.append(f"{short_name(r['Name'])[:44]:44s} {int(r['Calls']):7d} {float(r['AverageNs']) / 1e3:11.2f} "
                     f"{float(r['TotalDurationNs']) / 1e6:10.3f} {float(r['Percentage']):6.2f}")
    with open(out_path, "w") as f:
        f.write("\n".join(lines) + "\n")


def _counter_rows(d, counter):
    out = []
    for f in glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True):
        for r in csv.DictReader(open(f)):
            if r["Counter_Name"] == counter:
                out.append((int(r["Dispatch_Id"]), short_name(r["Kernel_Name"]), float(r["Counter_Value"])))
    return out


def stage_mean(rows, stage):
    """Mean sum of the counter over the executions of a stage, or None without
    one.  rows: (dispatch, kernel, value) of all dispatches of a run.  An
    execution is a dispatch of the stage's first kernel and the dispatches of
    its other kernels that follow it directly."""
    first, others, must = (re.compile(p) if p else None for p in STAGE_KERNELS[stage])
    runs, cur = [], None
    for _, k, v in sorted(rows):
        if first.match(k):
            cur = [0.0, must is None]
            runs.append(cur)
        elif not (others and others.match(k)):
            cur = None
        if cur is not None:
            cur[0] += v
            cur[1] = cur[1] or bool(must.match(k))
    sums = [v for v, whole in runs if whole]
    return sum(sums) / len(sums) if sums else None


def traffic_summary(fetch_dir, write_dir, copy_bytes, out_path, command):
    frows = _counter_rows(fetch_dir, "FETCH_SIZE")
    wrows = _counter_rows(write_dir, "WRITE_SIZE")
    # the calibration dispatch: a copy-like kernel whose write count is the
    # known size and which also reads (the buffer's fill writes the same
    # size but reads nothing); the same dispatch id in the fetch run gives
    # its read count
    fetch_of = {d: v for d, _, v in frows}
    cands = [(fetch_of.get(did, 0.0), did) for did, k, v in wrows
             if any(c in k for c in COPY_KERNELS) and abs(v * 1024.0 - copy_bytes) < 0.05 * copy_bytes]
    if not cands:
        raise SystemExit("no copy kernel in the WRITE_SIZE run: run the bench with --calibrate-copy")
    _, did = max(cands)
    wv = [v for d, _, v in wrows if d == did][0]
    fv = [v for d, _, v in frows if d == did][0]
    f_scale = copy_bytes / (fv * 1024.0)
    w_scale = copy_bytes / (wv * 1024.0)
    lines = ["# HBM traffic of one execution of each stage from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE (KiB),",
             f"# scaled by a {copy_bytes} B device copy in the same runs: read x{f_scale:.4f}, write x{w_scale:.4f}",
             f"# command: {command}", f"# source digest: {source_digest()}",
             f"{'stage':40s} {'read_MB':>10s} {'write_MB':>10s} {'traffic_MB':>11s}"]
    for stage in STAGE_KERNELS:
        rd, wr = stage_mean(frows, stage), stage_mean(wrows, stage)
        if rd is None or wr is None:
            continue
        rd *= 1024.0 * f_scale
        wr *= 1024.0 * w_scale
        lines.append(f"{stage:40s} {rd / 1e6:10.3f} {wr / 1e6:10.3f} {(rd + wr) / 1e6:11.3f}")
    with open(out_path, "w") as f:
        f.write("\n".join(lines) + "\n")


def lookup_traffic(stage, workload):
    """Traffic (bytes per execution) of a stage from profiles/, or None when the
    summary is missing or was taken on different kernel sources."""
    path = os.path.join(PROFILES, f"traffic_{workload}.txt")
    if not os.path.exists(path):
        return None
    digest = None
    for line in open(path):
        if line.startswith("# source digest:"):
            digest = line.split(":", 1)[1].strip()
        elif not line.startswith("#") and line.split() and line.split()[0] == stage:
            if digest != source_digest():
                return None
            return float(line.split()[3]) * 1e6
    return None


if __name__ == "__main__":
    if sys.argv[1] == "stats":
        stats_summary(sys.argv[2], sys.argv[3], " ".join(sys.argv[4:]))
    elif sys.argv[1] == "traffic":
        traffic_summary(sys.argv[2], sys.argv[3], int(sys.argv[4]), sys.argv[5], " ".join(sys.argv[6:]))
