"""Summaries of rocprofv3 CSV output for this library's kernels.

    python -m paper_2007_12273_amd.profsum trace  <kernel_trace.csv>
    python -m paper_2007_12273_amd.profsum bytes  <FETCH counter csv> <WRITE counter csv>
    python -m paper_2007_12273_amd.profsum insts  <visits.npz> <call>:<cold|warm> <counter csv> [...]

trace: per-kernel dispatch counts and durations, and per gm_compress call
(a call starts with the k_moments dispatch) the span of its EM phase, first
start to last end of its EM dispatches (k_em_span, k_em, k_em_big; they run
concurrently on several streams, so the phase span, not a single dispatch,
is the unit the EM roofline is quoted on), and with a queue column each
dispatch's start, duration and queue.

bytes: per gm_compress call the FETCH_SIZE and WRITE_SIZE counter totals
(KiB) over its EM dispatches, and the same counters for the largest
device copy in the run (a plain copy of known size calibrates them).

insts: instruction counters (any SQ_ counters, one or more csv files of
runs with the same launch sequence) of the EM dispatches of one
gm_compress call with FP32 iterations, per wave-update: a component update
executed by one wave of the cell's workgroup.  A cell's waves are those of
its length bucket, which holds the cells of up to 64 * per_thread * waves
particles (above the next smaller bucket's bound): of the k_em dispatches,
or of the plan's codes where the built-in launches ran; visits.npz
(bench.py --visits-out) gives the per-cell counts and updates of the cold
and the warm fit.
"""
from __future__ import annotations

import csv
import sys
from collections import OrderedDict


def _rows(path):
    with open(path) as f:
        return list(csv.DictReader(f))


CALL_START = "k_moments<"
EM_KERNELS = ("k_em_span<", "k_em<", "k_em_big<")


def _calls(rows, key_start):
    """Split dispatches (in dispatch order) into gm_compress calls."""
    rows = sorted(rows, key=lambda r: int(r["Dispatch_Id"]))
    calls, cur, last = [], None, None
    for r in rows:
        name = r["Kernel_Name"]
        # counter files hold one row per (dispatch, counter)
        first = r["Dispatch_Id"] != last
        last = r["Dispatch_Id"]
        if key_start in name and first:
            cur = []
            calls.append(cur)
        if cur is not None and any(k in name for k in EM_KERNELS):
            cur.append(r)
        if "k_finish<" in name:
            cur = None
    return calls


def trace(path):
    rows = _rows(path)
    agg = OrderedDict()
    for r in rows:
        d = (int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) * 1e-6
        name = r["Kernel_Name"].split("(")[0][:70]
        a = agg.setdefault(name, [0, 0.0])
        a[0] += 1
        a[1] += d
    print("%-72s %6s %12s %10s" % ("kernel", "calls", "total ms", "avg ms"))
    for name, (n, t) in sorted(agg.items(), key=lambda kv: -kv[1][1]):
        print("%-72s %6d %12.3f %10.4f" % (name, n, t, t / n))
    print()
    print("EM phase span per gm_compress call (first start to last end of its EM dispatches):")
    for i, c in enumerate(_calls(rows, CALL_START)):
        if not c:
            continue
        t0 = min(int(r["Start_Timestamp"]) for r in c)
        t1 = max(int(r["End_Timestamp"]) for r in c)
        busy = sum(int(r["End_Timestamp"]) - int(r["Start_Timestamp"]) for r in c)
        print("  call %2d: %2d EM dispatches, span %8.3f ms, sum of dispatch durations %8.3f ms"
              % (i, len(c), (t1 - t0) * 1e-6, busy * 1e-6))
        if "Queue_Id" in c[0]:
            print("           " + "  ".join(
                "%s +%.2f %.2f q%s" % (r["Kernel_Name"].split("(")[0].split("gm::")[-1].replace(" ", ""),
                                       (int(r["Start_Timestamp"]) - t0) * 1e-6,
                                       (int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) * 1e-6, r["Queue_Id"])
                for r in sorted(c, key=lambda r: int(r["Start_Timestamp"]))))


def _counter_calls(path):
    rows = _rows(path)
    calls = _calls(rows, CALL_START)
    totals = [sum(float(r["Counter_Value"]) for r in c) for c in calls]
    copies = [float(r["Counter_Value"]) for r in rows if "copyBuffer" in r["Kernel_Name"]]
    return totals, (max(copies) if copies else 0.0)


def bytes_(fetch_path, write_path):
    f_tot, f_copy = _counter_calls(fetch_path)
    w_tot, w_copy = _counter_calls(write_path)
    print("largest device copy: FETCH_SIZE %.0f KiB, WRITE_SIZE %.0f KiB" % (f_copy, w_copy))
    print("per gm_compress call, EM dispatches summed (KiB):")
    for i, (f, w) in enumerate(zip(f_tot, w_tot)):
        print("  call %2d: FETCH_SIZE %12.0f  WRITE_SIZE %12.0f" % (i, f, w))


def _shapes(names):
    """Sorted (largest cell, waves) of the buckets that the dispatches
    [(kernel name, workgroup size)] of a call with FP32 iterations cover."""
    shapes = set()
    for name, size in names:
        args = name.split("<", 1)[1].split(">", 1)[0].split(",")
        if "k_em_span<" in name:
            import ctypes
            from . import _lib
            if "double" in name:
                raise ValueError("FP64 iterations: the plan's codes do not give the built-in launches' waves")
            v = (ctypes.c_int32 * 12)()
            lib = _lib.load()
            lib.gm_autotune_reset()
            _lib.check(lib.gm_autotune_get(int(args[0]), int(args[1]), 0, 0, v, None, None), "gm_autotune_get")
            shapes |= {(64 * (c // 1000) * (c // 10 % 100), c // 10 % 100) for c in v}
        elif "k_em<" in name:
            shapes.add((64 * int(args[2]) * (size // 64), size // 64))
    return sorted(shapes)


def insts(visits_path, spec, paths):
    import numpy as np
    z = np.load(visits_path)
    n = z["n"]
    call, which = spec.split(":")
    visits = z["visits_" + which]
    tot, wave_updates, updates = OrderedDict(), 0, 0
    for path in paths:
        disp = OrderedDict()
        for r in _calls(_rows(path), CALL_START)[int(call)]:
            d = disp.setdefault(r["Dispatch_Id"], {"row": r, "c": {}})
            d["c"][r["Counter_Name"]] = d["c"].get(r["Counter_Name"], 0.0) + float(r["Counter_Value"])
        shapes = _shapes([(d["row"]["Kernel_Name"], int(d["row"]["Workgroup_Size"])) for d in disp.values()])
        wu, up, lo = 0, 0, 0
        for hi, W in shapes:
            sel = (n > lo) & (n <= hi)
            up += int(visits[sel].sum())
            wu += int(visits[sel].sum()) * W
            lo = hi
        wave_updates, updates = wu, up
        for d in disp.values():
            for k, v in d["c"].items():
                tot[k] = tot.get(k, 0.0) + v
    print("call %s (%s fit): %d component updates, %d wave-updates" % (call, which, updates, wave_updates))
    for k, v in tot.items():
        print("  %-32s %14.4g total %10.2f per wave-update" % (k, v, v / max(1, wave_updates)))


def main(argv):
    if len(argv) >= 2 and argv[0] == "trace":
        trace(argv[1])
    elif len(argv) >= 3 and argv[0] == "bytes":
        bytes_(argv[1], argv[2])
    elif len(argv) >= 4 and argv[0] == "insts":
        insts(argv[1], argv[2], argv[3:])
    else:
        print(__doc__)
        return 2
    return 0


if __name__ == "__main__":
    sys.exit(main(sys.argv[1:]))
