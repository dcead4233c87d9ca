#!/usr/bin/env python3
"""Throughput of the layer-case FDM transport hot path on one MI355X.

Headline workload (the single-instance configuration beyond the on-chip
cache): a 4096 x 4096 periodic grid of 64 diagonal density bands (widths
8-32 cells, amplitudes +-[0.5, 1], alternating signs, seed 3) under a
celerity field v0 = tanh(tau/0.5), tau a unit-RMS sum of 16 Fourier modes
with |k| <= 8; LAW Hamiltonian, minmod limiter, two-stage Heun steps at
Courant number 0.45, float32 state (synthetic input).  A step is one full
time step of every node: limited slopes, one-sided derivatives, speeds,
numerical Hamiltonian and conservative update, both stages.

Legs beside it: the same workload with float64 state; the 2048^2 expanding
loop; the 384-instance batched workload (batched vs one launch per
instance); the coupled 512^2 run; the paper's fully discrete scheme; the
64^2 colliding pulses at full length.  Every leg's result is compared with
the FP64 oracle on the same inputs (relative L1 and L-infinity over the
initial norms, and the drift of the conserved totals), inside the CPU
baseline leg, which times that oracle on the host cores.  Prints one JSON
line.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import struct
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "transport cell-updates/s and % HBM peak; batched vs plain speedup at ≤1e-5 rel L1"
HBM_PEAK_GBS = 8000.0            # MI355X HBM3E, GB/s
# VALU issue peak with packed FP32 off: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz
ISSUE_PEAK = 256 * 64 * 2.4e9
# algorithmic bytes per cell-update: read and write both density components
# once (float32: 16 B, float64: 32 B), plus 4 B to read a float32 celerity field
STATE_BYTES = {"fp32": 16, "fp64": 32}
FIELD_BYTES = 4

PROFILE_FILE = os.path.join(ROOT, "profiles", "fused_kernel_bands_field_4096_fp32_counters.json")
LIB_FILE = os.path.join(ROOT, "paper_1911_03225_amd", "libfdm.so")
HEADLINE_KERNEL = "fused_kernel<3, 0, true, false, false, float, float>"   # minmod, LAW, celerity field, Heun
HEADLINE_SYMBOL = "_ZN3fdm12_GLOBAL__N_112fused_kernelILi3ELi0ELb1ELb0ELb0EffEEvNS_7InstDevEliii"
# Repeated autotuner runs on one box order heights within about 3% of each
# other differently; within that the height the counters were taken at is kept.
PROFILED_HEIGHT_SLACK = 1.03
COPY_KERNEL = "copy_kernel<float>"
GOLDEN_C4 = os.path.join(ROOT, "tests", "golden", "coupled_c4_history.json")


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def _elf_sections(b):
    """[name, type, addr, offset, size, link] of each section of an ELF64 image."""
    shoff, = struct.unpack_from("<Q", b, 0x28)
    shentsize, shnum, shstrndx = struct.unpack_from("<HHH", b, 0x3A)
    secs = []
    for i in range(shnum):
        o = shoff + i * shentsize
        name, typ = struct.unpack_from("<II", b, o)
        addr, off, size = struct.unpack_from("<QQQ", b, o + 16)
        link, = struct.unpack_from("<I", b, o + 40)
        secs.append([name, typ, addr, off, size, link])
    names = secs[shstrndx][3]
    for s in secs:
        s[0] = b[names + s[0]:b.index(b"\0", names + s[0])].decode()
    return secs


def kernel_code_hash(path=LIB_FILE, symbol=HEADLINE_SYMBOL, arch="gfx950"):
    """SHA-256 of a kernel as built: its machine code and its kernel
    descriptor (registers, LDS, launch settings; without the entry offset,
    which moves with the rest of the code object), read from the library's
    offload bundles.  None when the library or the kernel is not there.  The
    counter summary is keyed by it, so the counters stay valid across edits
    that leave the headline kernel's code unchanged, and only those."""
    try:
        with open(path, "rb") as fh:
            b = fh.read()
        fat = [s for s in _elf_sections(b) if s[0] == ".hip_fatbin"]
        if not fat:
            return None
        data = b[fat[0][3]:fat[0][3] + fat[0][4]]
        magic = b"__CLANG_OFFLOAD_BUNDLE__"
        base = data.find(magic)
        while base >= 0:
            n, = struct.unpack_from("<Q", data, base + len(magic))
            p = base + len(magic) + 8
            for _ in range(n):
                off, size, tl = struct.unpack_from("<QQQ", data, p)
                triple = data[p + 24:p + 24 + tl].decode()
                p += 24 + tl
                if not triple.endswith("--" + arch):
                    continue
                elf = data[base + off:base + off + size]
                secs = _elf_sections(elf)
                found = {}
                for st in (s for s in secs if s[1] == 2):          # SHT_SYMTAB
                    strtab = secs[st[5]][3]
                    for k in range(st[4] // 24):
                        o = st[3] + 24 * k
                        nm, _info, _other, shndx = struct.unpack_from("<IBBH", elf, o)
                        val, sz = struct.unpack_from("<QQ", elf, o + 8)
                        name = elf[strtab + nm:elf.index(b"\0", strtab + nm)].decode()
                        if name in (symbol, symbol + ".kd") and shndx < len(secs):
                            sec = secs[shndx]
                            start = sec[3] + val - sec[2]
                            found[name] = elf[start:start + sz]
                if symbol in found and len(found.get(symbol + ".kd", b"")) == 64:
                    kd = found[symbol + ".kd"]
                    return hashlib.sha256(found[symbol] + kd[:16] + kd[24:]).hexdigest()
            base = data.find(magic, base + 1)
    except (OSError, ValueError, struct.error, IndexError, UnicodeDecodeError):
        return None
    return None


# ------------------------------------------------------------ counter summary

def _counter_rows(directories, counters):
    """{kernel name: {counter: [values per dispatch]}} and grid sizes from
    rocprofv3 counter CSVs under the given directories."""
    import collections
    import csv
    import glob
    vals = collections.defaultdict(lambda: collections.defaultdict(list))
    grids = collections.defaultdict(set)
    for d in directories:
        for f in glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True):
            for r in csv.DictReader(open(f)):
                if r["Counter_Name"] in counters:
                    vals[r["Kernel_Name"]][r["Counter_Name"]].append(float(r["Counter_Value"]))
                    grids[r["Kernel_Name"]].add(int(r["Grid_Size"]))
    return vals, grids


def write_profile_summary(fetch_dir, write_dir, sq_dir, out, copy_n, tile_rows):
    """Per-launch counters of the headline kernel at one tile height from
    three rocprofv3 passes (FETCH_SIZE, WRITE_SIZE, SQ): HBM-side bytes, each
    counter calibrated by what it reads for a copy kernel of 4 copy_n^2 bytes
    each way, and the VALU and MFMA instructions issued.  Stored in `out`
    under by_rows[tile_rows], beside the entries of other heights taken on
    the same kernel sources (a summary of other sources is replaced)."""
    def pick(vals, pat, counter):
        for name, cs in vals.items():
            if pat in name and counter in cs:
                return sum(cs[counter]) / len(cs[counter])
        raise SystemExit("no %s samples of %s" % (counter, pat))
    fv, _ = _counter_rows([fetch_dir], {"FETCH_SIZE"})
    wv, _ = _counter_rows([write_dir], {"WRITE_SIZE"})
    sv, _ = _counter_rows([sq_dir], {"SQ_WAVES", "SQ_INSTS_VALU", "SQ_INSTS_MFMA", "SQ_ACTIVE_INST_VALU",
                                     "SQ_BUSY_CYCLES", "SQ_WAVE_CYCLES", "SQ_WAIT_INST_ANY", "GRBM_GUI_ACTIVE"})
    copy_kib = 4.0 * copy_n * copy_n / 1024.0
    ff = copy_kib / pick(fv, COPY_KERNEL, "FETCH_SIZE")
    wf = copy_kib / pick(wv, COPY_KERNEL, "WRITE_SIZE")
    fk, wk = pick(fv, HEADLINE_KERNEL, "FETCH_SIZE"), pick(wv, HEADLINE_KERNEL, "WRITE_SIZE")
    sq = {c: pick(sv, HEADLINE_KERNEL, c) for c in ("SQ_WAVES", "SQ_INSTS_VALU", "SQ_INSTS_MFMA",
                                                     "SQ_ACTIVE_INST_VALU", "SQ_WAVE_CYCLES", "SQ_WAIT_INST_ANY")
          if any(HEADLINE_KERNEL in n and c in cs for n, cs in sv.items())}
    entry = {"copy_probe_n": copy_n, "fetch_factor": round(ff, 4), "write_factor": round(wf, 4),
             "fetch_kib": round(fk, 1), "write_kib": round(wk, 1),
             "bytes_per_launch": round((fk * ff + wk * wf) * 1024.0),
             "sq_per_launch": {k: round(v, 1) for k, v in sq.items()}}
    summary = {"kernel": HEADLINE_KERNEL, "kernel_code_sha256": kernel_code_hash(), "grid": 4096,
               "by_rows": {}}
    try:
        with open(out) as fh:
            old = json.load(fh)
        if summary["kernel_code_sha256"] and old.get("kernel_code_sha256") == summary["kernel_code_sha256"] and \
                isinstance(old.get("by_rows"), dict):
            summary["by_rows"] = old["by_rows"]
    except (OSError, ValueError):
        pass
    summary["by_rows"][str(int(tile_rows))] = entry
    summary["by_rows"] = {k: summary["by_rows"][k] for k in sorted(summary["by_rows"], key=int)}
    with open(out, "w") as fh:
        json.dump(summary, fh, indent=1)
    print(json.dumps(summary))


def _profile_entries():
    """{tile rows: counter entry} of the committed summary when it was taken
    on the headline kernel's current machine code, else {}."""
    try:
        with open(PROFILE_FILE) as fh:
            p = json.load(fh)
    except (OSError, ValueError):
        return {}
    code = kernel_code_hash()
    if not code or p.get("kernel_code_sha256") != code or not isinstance(p.get("by_rows"), dict):
        return {}
    return {int(k): v for k, v in p["by_rows"].items()}


def profiled_heights():
    """Tile heights the committed counter summary covers (current kernel code)."""
    return sorted(_profile_entries())


def load_profile(tile_rows):
    """The headline kernel's counters at this tile height, measured on its
    current machine code, else None."""
    e = _profile_entries().get(int(tile_rows))
    return dict(e, tile_rows=int(tile_rows)) if e else None


# ------------------------------------------------------------------ helpers

def host_arrays(t11, t12):
    import numpy as np
    return t11.cpu().numpy().astype(np.float64), t12.cpu().numpy().astype(np.float64)


def timed_steps(fdm, ctx, t11, t12, K, repeats, stream):
    """Median wall time of K steps enqueued back to back on the library's
    stream, between HIP events on that stream."""
    import torch
    times = []
    for _ in range(repeats):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        torch.cuda.synchronize()
        e0.record(stream)
        fdm.fdm_transport_step(ctx, t11, t12, K)
        e1.record(stream)
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1) / 1000.0)
    return sorted(times)[len(times) // 2], times


def single_instance(fdm, a11, a12, K, W, repeats, stream, desc_kw, options, autotune, field=None,
                    prefer_rows=(), sustained=0):
    """Autotune, a K-step run from the inputs (kept for parity), W warmup
    steps, then the timed K-step repeats.  Returns timing and the state
    after the first K steps.  prefer_rows: fused tile heights the counter
    passes were taken at; when the autotuner's best is none of them, the
    fastest of them it timed within 3% of its best is kept instead."""
    import numpy as np
    import torch
    dev = torch.device("cuda:0")
    sdt = torch.float64 if options.get("precision") == "fp64" else torch.float32
    ny, nx = a11.shape
    t11 = torch.from_numpy(a11).to(dev).to(sdt)
    t12 = torch.from_numpy(a12).to(dev).to(sdt)
    ctx = fdm.fdm_transport_init(fdm.desc(nx, ny, v0_field=field, **desc_kw), options=options, stream=stream,
                                 keep=[field] if field is not None else [])
    sched = options.get("schedule", "auto")
    if sched == "auto":   # the library's own choice, when not tuned
        sched = "fused" if fdm.load_library().fdm_debug_fused(ctx.handle) else "plain"
    trials, choice = None, "fixed" if options.get("tile_rows") else "default rule"
    if autotune:
        trials = fdm.fdm_autotune(ctx, [t11], [t12], trial_steps=20)
        best = min(trials, key=lambda t: t["seconds_per_step"])
        sched, choice = best["schedule"], "autotuned"
        near = [t for t in trials if t["schedule"] == "fused" and t["tile_rows"] in prefer_rows and
                t["seconds_per_step"] <= PROFILED_HEIGHT_SLACK * best["seconds_per_step"]]
        if near and not (best["schedule"] == "fused" and best["tile_rows"] in prefer_rows):
            rows = min(near, key=lambda t: t["seconds_per_step"])["tile_rows"]
            fdm.fdm_destroy(ctx)
            ctx = fdm.fdm_transport_init(fdm.desc(nx, ny, v0_field=field, **desc_kw),
                                         options=dict(options, schedule="fused", tile_rows=rows),
                                         stream=stream, keep=[field] if field is not None else [])
            sched, choice = "fused", "profiled height, within 3% of the autotuned best"
    rows = fdm.fdm_tile_rows(ctx, 0)
    dt = fdm.fdm_transport_dt(ctx)
    # Warmup right before the timed regions, with no host work between: an
    # idle GPU lowers its clock, and a few milliseconds of load ramp it back
    # (a 20-step region after a 100 ms host pause measured 17% slower than
    # the steady rate of 200- and 2000-step regions).
    fdm.fdm_transport_step(ctx, t11, t12, W)
    t_med, times = timed_steps(fdm, ctx, t11, t12, K, repeats, stream)
    # Beside the K-step regions, one region of `sustained` steps: a short
    # region right after the warmup runs at the burst clock, a long one at
    # the clock the board's power limit holds.
    sus = timed_steps(fdm, ctx, t11, t12, sustained, 1, stream)[0] / sustained if sustained else None
    # then K steps from the inputs again: the result the oracle checks
    t11.copy_(torch.from_numpy(a11).to(dev).to(sdt))
    t12.copy_(torch.from_numpy(a12).to(dev).to(sdt))
    fdm.fdm_transport_step(ctx, t11, t12, K)
    torch.cuda.synchronize()
    after = host_arrays(t11, t12)
    fdm.fdm_destroy(ctx)
    del t11, t12
    return {"seconds": t_med, "times": times, "schedule": sched, "tile_rows": rows, "dt": dt,
            "trials": trials, "tile_choice": choice, "after": after, "cells": int(np.prod(a11.shape)),
            "sustained_seconds_per_step": sus, "sustained_steps": sustained}


# ---------------------------------------------------------------- the legs

def headline_leg(fdm, W_, K, warm, repeats, autotune, tile_rows, schedule, log):
    import torch
    a11, a12, v0 = W_.bands_and_celerity(4096, seed=3)
    stream = torch.cuda.current_stream()
    tv = torch.from_numpy(v0).to("cuda:0")
    prefer = profiled_heights()
    r = single_instance(fdm, a11, a12, K, warm, repeats, stream, dict(limiter="minmod", cfl=0.45),
                        {"schedule": schedule, "tile_rows": tile_rows}, autotune, field=tv, prefer_rows=prefer,
                        sustained=max(200, 10 * K))
    cells = r["cells"]
    value = cells * K / r["seconds"]
    fused = r["schedule"] == "fused"
    launches = K if fused else 2 * K
    kernel_s = r["seconds"] / launches
    alg_bytes = (STATE_BYTES["fp32"] + FIELD_BYTES) * cells * K // launches
    achieved = alg_bytes / kernel_s / 1e9
    prof = load_profile(r["tile_rows"]) if fused else None
    valu = None
    if prof and "SQ_INSTS_VALU" in prof["sq_per_launch"]:
        issued = prof["sq_per_launch"]["SQ_INSTS_VALU"] * 64
        valu = {"issued_lane_instr_per_launch": round(issued),
                "achieved_T_per_s": round(issued / kernel_s / 1e12, 3),
                "issue_peak_T_per_s": round(ISSUE_PEAK / 1e12, 2),
                "frac": round(issued / kernel_s / ISSUE_PEAK, 4),
                "issued_per_node_stage": round(issued / (2 * cells), 2),
                "mfma_instructions": prof["sq_per_launch"].get("SQ_INSTS_MFMA"),
                "source": "SQ_INSTS_VALU x 64 lanes per launch, " + os.path.relpath(PROFILE_FILE, ROOT)}
    roofline = {"bound": "hbm", "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": round(achieved / HBM_PEAK_GBS, 4),
                "traffic": prof["bytes_per_launch"] if prof else None,
                "traffic_vs_algorithmic": round(prof["bytes_per_launch"] / alg_bytes, 3) if prof else None,
                "kernel": (HEADLINE_KERNEL + " (both Heun stages; minmod, LAW, celerity field)") if fused
                else "stage_kernel (first and second Heun stage)",
                "kernel_avg_us": round(1e6 * kernel_s, 2), "launches_per_step": launches // K,
                "algorithmic_bytes_per_launch": alg_bytes,
                "bytes_per_cell_update": STATE_BYTES["fp32"] + FIELD_BYTES,
                "timing": "HIP events on the library's stream around K back-to-back steps, median of %d" % repeats,
                "sustained": {"steps": r["sustained_steps"],
                              "kernel_avg_us": round(1e6 * r["sustained_seconds_per_step"] * K / launches, 2),
                              "frac": round(alg_bytes / (r["sustained_seconds_per_step"] * K / launches) / 1e9
                                            / HBM_PEAK_GBS, 4),
                              "note": "one region of that many steps after the K-step ones: the clock the "
                                      "power limit holds, against the burst clock of short regions"},
                "valu": valu}
    log("bench[c3]: %.4e cell-updates/s, %.2f us per %s launch, %.0f GB/s algorithmic (%.3f of HBM peak), "
        "%d-row tiles; %d-step region %.2f us per launch" % (
            value, 1e6 * kernel_s, r["schedule"], achieved, achieved / HBM_PEAK_GBS, r["tile_rows"],
            r["sustained_steps"], roofline["sustained"]["kernel_avg_us"]))
    return r, value, roofline, (a11, a12, v0)


def fp64_state_leg(fdm, K, warm, repeats, inputs, log):
    import torch
    a11, a12, v0 = inputs
    stream = torch.cuda.current_stream()
    tv = torch.from_numpy(v0).to("cuda:0")
    r = single_instance(fdm, a11, a12, K, warm, repeats, stream, dict(limiter="minmod", cfl=0.45),
                        {"precision": "fp64", "schedule": "plain"}, False, field=tv)
    value = r["cells"] * K / r["seconds"]
    b = STATE_BYTES["fp64"] + FIELD_BYTES
    log("bench[c3 fp64]: %.4e cell-updates/s (float64 state, two stage launches per step)" % value)
    return r, {"cell_updates_per_s": round(value, 1), "ms_per_step": round(1e3 * r["seconds"] / K, 4),
               "schedule": "plain", "tile_rows": r["tile_rows"], "bytes_per_cell_update": b,
               "hbm_frac_algorithmic": round(value * b / 1e9 / HBM_PEAK_GBS, 4),
               "timing": "HIP events around K back-to-back steps, median of %d" % repeats}


def loop_leg(fdm, W_, K, warm, repeats, autotune, log, schedule="auto", tile_rows=0):
    import torch
    a11, a12 = W_.ring(2048, 2048, R=300.0, sigma=6.0)
    stream = torch.cuda.current_stream()
    r = single_instance(fdm, a11, a12, K, warm, repeats, stream, dict(limiter="superbee", cfl=0.4, v0=-1.0),
                        {"schedule": schedule, "tile_rows": tile_rows}, autotune)
    value = r["cells"] * K / r["seconds"]
    log("bench[c2]: %.4e cell-updates/s (%s, %d rows)" % (value, r["schedule"], r["tile_rows"]))
    return r, {"grid": [2048, 2048], "limiter": "superbee", "cfl": 0.4, "steps": K,
               "cell_updates_per_s": round(value, 1), "ms_per_step": round(1e3 * r["seconds"] / K, 5),
               "schedule": r["schedule"], "tile_rows": r["tile_rows"],
               "hbm_frac_algorithmic": round(value * STATE_BYTES["fp32"] / 1e9 / HBM_PEAK_GBS, 4),
               "note": "state and stage buffer (64 MiB) fit in the 256 MB MALL"}, (a11, a12)


def fully_discrete_leg(fdm, W_, K, warm, repeats, autotune, log):
    import torch
    a11, a12 = W_.ring(2048, 2048, R=300.0, sigma=6.0)
    stream = torch.cuda.current_stream()
    kw = dict(limiter="superbee", cfl=0.25, v0=-1.0, time_order=1, scheme="fully_discrete")
    r = single_instance(fdm, a11, a12, K, warm, repeats, stream, kw, {"schedule": "plain"}, autotune)
    value = r["cells"] * K / r["seconds"]
    log("bench[fd]: %.4e cell-updates/s, %.2f us/step" % (value, 1e6 * r["seconds"] / K))
    return r, {"grid": [2048, 2048], "limiter": "superbee", "cfl": 0.25, "steps": K,
               "cell_updates_per_s": round(value, 1), "ms_per_step": round(1e3 * r["seconds"] / K, 5),
               "tile_rows": r["tile_rows"]}, (a11, a12)


def c1_leg(fdm, W_, log):
    """The small plain case at full length: 64^2 colliding pulses, LAW
    v0 = -1, minmod, Heun, Courant 0.5, 400 steps."""
    import numpy as np
    import torch
    a11, a12 = (np.ascontiguousarray(a) for a in W_.colliding_pulses(64))
    stream = torch.cuda.current_stream()
    t11, t12 = torch.from_numpy(a11).to("cuda:0"), torch.from_numpy(a12).to("cuda:0")
    ctx = fdm.fdm_transport_init(fdm.desc(64, 64, limiter="minmod", cfl=0.5, v0=-1.0), stream=stream)
    dt = fdm.fdm_transport_dt(ctx)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    fdm.fdm_transport_step(ctx, t11, t12, 400)
    e1.record(stream)
    torch.cuda.synchronize()
    sec = e0.elapsed_time(e1) / 1000.0
    after = host_arrays(t11, t12)
    fdm.fdm_destroy(ctx)
    log("bench[c1]: 400 steps of 64^2 in %.2f ms" % (1e3 * sec))
    return {"a11": a11, "a12": a12, "after": after, "dt": dt}, {
        "grid": [64, 64], "steps": 400, "limiter": "minmod", "cfl": 0.5, "dt": dt,
        "us_per_step": round(1e6 * sec / 400, 2), "cell_updates_per_s": round(64 * 64 * 400 / sec, 1),
        "note": "launch-bound at this size"}


def _make_instance(inst):
    return inst.make()


def batched_leg(fdm, W_, K, log, autotune=True, schedules=("batched", "plain", "fused")):
    """The 384-instance workload: one K-step chunk as one graph of batched
    launches, as one graph of batched fused launches, and as one launch per
    instance per stage; then the stratified subset again with float64 state
    (batched).  Keeps the subset's results for parity."""
    import concurrent.futures as cf
    import multiprocessing as mp
    import torch
    insts = W_.batched_instances()
    subset = W_.stratified_subset(insts, large_nodes=512 * 512)
    idx = [insts.index(s) for s in subset]
    t0 = time.perf_counter()
    workers = max(1, min(16, os.cpu_count() or 1))
    with cf.ProcessPoolExecutor(max_workers=workers, mp_context=mp.get_context("spawn")) as ex:
        arrays = list(ex.map(_make_instance, insts, chunksize=4))
    log("bench[batched]: generated %d instances in %.1f s" % (len(insts), time.perf_counter() - t0))
    dev = torch.device("cuda:0")
    fields = [torch.from_numpy(a[2]).to(dev) if a[2] is not None else None for a in arrays]
    descs = [fdm.desc(i.nx, i.ny, limiter=i.limiter, cfl=0.4, v0=i.v0, v0_field=f) for i, f in zip(insts, fields)]
    nodes = sum(i.nx * i.ny for i in insts)
    stream = torch.cuda.current_stream()
    out, finals = {}, {}
    # the inputs stay on the device: resetting the state before the timed
    # run is a device copy, not 1.4 GB over the host link with the GPU idle
    d11 = [torch.from_numpy(a[0]).to(dev) for a in arrays]
    d12 = [torch.from_numpy(a[1]).to(dev) for a in arrays]
    for sched in schedules:
        s11 = [x.clone() for x in d11]
        s12 = [x.clone() for x in d12]
        ctx = fdm.fdm_transport_init(descs, options={"schedule": sched}, stream=stream, keep=fields)
        if autotune:
            fdm.fdm_autotune(ctx, s11, s12, trial_steps=2)
        rows = fdm.fdm_tile_rows(ctx, 0)
        if sched != "plain":
            fdm.fdm_run(ctx, s11, s12, K, K, history=False)      # capture + warm
        else:
            fdm.fdm_transport_step(ctx, s11, s12, 2)
        for a, b in zip(s11, d11):
            a.copy_(b)
        for a, b in zip(s12, d12):
            a.copy_(b)
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        if sched != "plain":
            fdm.fdm_run(ctx, s11, s12, K, K, history=False)
        else:
            fdm.fdm_transport_step(ctx, s11, s12, K)
        e1.record(stream)
        torch.cuda.synchronize()
        sec = e0.elapsed_time(e1) / 1000.0
        stats = fdm.fdm_transport_stats(ctx, s11, s12, allow_nonfinite=True)
        fdm.fdm_destroy(ctx)
        out[sched] = {"seconds": round(sec, 4), "cell_updates_per_s": round(nodes * K / sec, 1), "tile_rows": rows,
                      "nonfinite_instances": sum(1 for st in stats if st["nonfinite"])}
        finals[sched] = (s11, s12)
        log("bench[batched]: %s %d steps in %.3f s (%.3e cell-updates/s)" % (sched, K, sec, nodes * K / sec))

    def same(a, b):
        if a not in finals or b not in finals:
            return None
        return bool(all(torch.equal(x, y) for x, y in zip(finals[a][0], finals[b][0])) and
                    all(torch.equal(x, y) for x, y in zip(finals[a][1], finals[b][1])))
    eq, feq = same("batched", "plain"), same("fused", "plain") if "plain" in finals else same("fused", "batched")
    ref = finals["batched"] if "batched" in finals else next(iter(finals.values()))
    sub32 = [host_arrays(ref[0][i], ref[1][i]) for i in idx]
    del finals
    # float64 state, batched, on the subset
    t11 = [torch.from_numpy(arrays[i][0]).to(dev).double() for i in idx]
    t12 = [torch.from_numpy(arrays[i][1]).to(dev).double() for i in idx]
    ctx = fdm.fdm_transport_init([descs[i] for i in idx], options={"schedule": "batched", "precision": "fp64"},
                                 stream=stream, keep=fields)
    fdm.fdm_run(ctx, t11, t12, K, K, history=False)
    torch.cuda.synchronize()
    fdm.fdm_destroy(ctx)
    sub64 = [host_arrays(a, b) for a, b in zip(t11, t12)]
    ratio = lambda a, b: round(out[a]["seconds"] / out[b]["seconds"], 3) if a in out and b in out else None  # noqa: E731
    res = {"instances": len(insts), "nodes": nodes, "chunk_steps": K,
           "batched": out.get("batched"), "plain": out.get("plain"), "fused_batched": out.get("fused"),
           "speedup": ratio("plain", "batched"), "fused_speedup_vs_plain": ratio("plain", "fused"),
           "bitwise_equal": eq, "fused_bitwise_equal": feq}
    keep = {"subset": subset, "inputs": [arrays[i] for i in idx], "fp32": sub32, "fp64": sub64}
    return res, keep


def coupled_leg(fdm, W_, n_steps, log, n=512):
    """The coupled workload: a 512^2 layer with 20 seeded loops (plateaus
    +-0.2, erfc edges sigma 2, radii 20-80), a 4-voxel layer in a 512-voxel
    cell, mu = 1, nu = 0.3, threshold 0.01, mobility 1, strain rate 1e-3,
    Courant 0.4 with the step capped at 0.02; n_steps coupled steps (static
    solve, velocity law, adaptive step, transport, mean slip), a stats record
    every 100 steps."""
    import torch
    phi, a11, a12 = W_.plateau_rings(n, n, seed=4)
    dev = torch.device("cuda:0")
    t11, t12 = torch.from_numpy(a11).to(dev), torch.from_numpy(a12).to(dev)
    stream = torch.cuda.current_stream()
    ctx = fdm.fdm_transport_init(fdm.desc(n, n, limiter="minmod", cfl=0.4, v0=-1.0), stream=stream)
    L = fdm.loading(strain_rate13=1e-3, tau0=0.01, mobility=1.0, mu=1.0, lam=1.5, layer_h=4.0, cell_l3=512.0,
                    dt_max=0.02, eps13=0.0, phi_mean=float(phi.mean()))
    fdm.fdm_run(ctx, t11.clone(), t12.clone(), 20, 20, loading=L)    # plans, workspace, warm-up
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    hist = fdm.fdm_run(ctx, t11, t12, n_steps, 100, loading=L)
    torch.cuda.synchronize()
    sec = time.perf_counter() - t0
    fdm.fdm_destroy(ctx)
    hist = [h[0] for h in hist]
    log("bench[coupled]: %d coupled steps in %.3f s (%.1f us/step)" % (n_steps, sec, 1e6 * sec / n_steps))
    pick = hist[9::10] if len(hist) >= 10 else hist
    res = {"grid": [n, n], "steps": n_steps, "seconds": round(sec, 4), "ms_per_step": round(1e3 * sec / n_steps, 4),
           "cell_updates_per_s": round(n * n * n_steps / sec, 1),
           "timing": "host wall clock over the call (step scalars stay on the device; one sync per 100 steps)",
           "stress_strain": [[round(r["eps13"], 7), round(r["sigma13"], 8), round(r["phi_mean"], 8),
                              round(r["vmax"], 6)] for r in pick],
           "stress_strain_columns": ["eps13", "sigma13", "phi_mean", "vmax"]}
    return res, {"hist": hist, "s0": float(abs(a11.astype("float64")).sum() + abs(a12.astype("float64")).sum()),
                 "steps": n_steps}


# ------------------------------------------------------ oracle: cpu baseline

def _rel(g, o, a):
    import numpy as np
    a11, a12 = a
    d1 = np.abs(a11.astype(np.float64)).sum() + np.abs(a12.astype(np.float64)).sum()
    di = max(np.abs(a11).max(), np.abs(a12).max())
    return (float((np.abs(g[0] - o[0]).sum() + np.abs(g[1] - o[1]).sum()) / d1),
            float(max(np.abs(g[0] - o[0]).max(), np.abs(g[1] - o[1]).max()) / di))


def _drift(x, a):
    """Change of the conserved totals (sum alpha_11, sum alpha_12) over the
    initial sum |alpha|."""
    import numpy as np
    a11, a12 = (v.astype(np.float64) for v in a)
    d = np.abs(a11).sum() + np.abs(a12).sum()
    return float((abs(x[0].sum() - a11.sum()) + abs(x[1].sum() - a12.sum())) / d)


def parity_record(g, o, a, steps, bound_l1=None):
    e1, ei = _rel(g, o, a)
    rec = {"steps": steps, "rel_l1": e1, "rel_linf": ei, "drift": _drift(g, a), "oracle_drift": _drift(o, a)}
    if bound_l1 is not None:
        rec["bar_rel_l1"] = bound_l1
    return rec


def host_description():
    model = None
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        affinity = len(os.sched_getaffinity(0))
    except AttributeError:
        affinity = None
    return {"nproc": os.cpu_count(), "affinity_cpus": affinity, "cpu_model": model,
            "OMP_NUM_THREADS": os.environ.get("OMP_NUM_THREADS")}


def cpu_baseline_leg(K, head, loop, fd, c1, fp64, batched, coupled, min_seconds, log):
    """The FP64 oracle on the host cores: timed on the headline workload (all
    threads, and one thread) and at full length on the small case; every
    leg's GPU result is compared with it on the same inputs."""
    import numpy as np
    import oracle
    oracle.build(force=False)
    threads = oracle.max_threads()
    parity = {}
    # headline: K steps from the inputs (the parity reference), continued
    # until min_seconds have been timed
    r, (a11, a12, v0) = head
    P = oracle.Problem(4096, 4096, limiter="minmod", v0=v0.astype(np.float64), dt=r["dt"])
    assert oracle.cfl_dt(P, 0.45) == r["dt"]
    t0 = time.perf_counter()
    o = oracle.run(P, a11, a12, K)
    steps, el = K, time.perf_counter() - t0
    parity["c3_fp32"] = parity_record(r["after"], o, (a11, a12), K, max(1e-5, 1e-6 * K))
    if fp64 is not None:
        parity["c3_fp64"] = parity_record(fp64["after"], o, (a11, a12), K, 1e-5)
    x = o
    while el < min_seconds:
        t1 = time.perf_counter()
        x = oracle.run(P, x[0], x[1], K)
        el += time.perf_counter() - t1
        steps += K
    all_cores = 4096 * 4096 * steps / el
    log("bench[cpu]: oracle %d steps of 4096^2 in %.1f s on %d threads" % (steps, el, threads))
    oracle.set_threads(1)
    t1 = time.perf_counter()
    oracle.run(P, a11, a12, 1)
    single = 4096 * 4096 / (time.perf_counter() - t1)
    # the small case at full length, one thread and all threads
    Pc = oracle.Problem(64, 64, limiter="minmod", v0=-1.0, dt=c1["dt"]) if c1 else None
    full = None
    if c1:
        t1 = time.perf_counter()
        oc = oracle.run(Pc, c1["a11"], c1["a12"], 400)
        c1_single = 64 * 64 * 400 / (time.perf_counter() - t1)
    oracle.set_threads(threads)
    if c1:
        t1 = time.perf_counter()
        oracle.run(Pc, c1["a11"], c1["a12"], 400)
        c1_all = 64 * 64 * 400 / (time.perf_counter() - t1)
        full = {"workload": "64x64 colliding pulses, minmod, Heun, CFL 0.5, 400 steps (full length)",
                "single_thread": round(c1_single, 1), "all_threads": round(c1_all, 1)}
        parity["c1_fp32_full_length"] = parity_record(c1["after"], oc, (c1["a11"], c1["a12"]), 400, 1e-5)
    cpu = {"value": round(all_cores, 1), "unit": "cell-updates/s", "cores": threads, "kind": "oracle",
           "sample": "first %d steps of the 4096x4096 bands + celerity field workload (FP64, OpenMP over rows, "
                     "%d threads), %.1f s" % (steps, threads, el),
           "single_thread": {"value": round(single, 1), "unit": "cell-updates/s",
                             "sample": "first step of the same workload on one thread"},
           "full_length": full, "host": host_description()}
    if loop:
        r2, (b11, b12) = loop
        P2 = oracle.Problem(2048, 2048, limiter="superbee", v0=-1.0, dt=r2["dt"])
        parity["c2_fp32"] = parity_record(r2["after"], oracle.run(P2, b11, b12, K), (b11, b12), K,
                                          max(1e-5, 1e-6 * K))
    if fd:
        r3, (b11, b12) = fd
        P3 = oracle.Problem(2048, 2048, limiter="superbee", v0=-1.0, dt=r3["dt"], time_order=1,
                            scheme="fully_discrete")
        parity["fully_discrete_fp32"] = parity_record(r3["after"], oracle.run(P3, b11, b12, K), (b11, b12), K)
    if batched:
        t1 = time.perf_counter()
        rows = []
        steps_b = batched["K"]
        for inst, inp, g32, g64 in zip(batched["subset"], batched["inputs"], batched["fp32"], batched["fp64"]):
            a11b, a12b, vb = inp
            Pb = oracle.Problem(inst.nx, inst.ny, limiter=inst.limiter,
                                v0=inst.v0 if vb is None else vb.astype(np.float64))
            Pb.dt = oracle.cfl_dt(Pb, 0.4)
            ob = oracle.run(Pb, a11b, a12b, steps_b)
            e32, i32 = _rel(g32, ob, (a11b, a12b))
            e64, i64 = _rel(g64, ob, (a11b, a12b))
            rows.append({"size": [inst.nx, inst.ny], "velocity": inst.velocity, "limiter": inst.limiter,
                         "init": inst.init, "fp32_rel_l1": e32, "fp32_rel_linf": i32, "fp64_rel_l1": e64,
                         "fp64_rel_linf": i64, "fp32_drift": _drift(g32, (a11b, a12b))})
        worst = lambda k: max(x[k] for x in rows)   # noqa: E731
        parity["batched_subset"] = {
            "instances": len(rows), "steps": steps_b,
            "fp32_rel_l1_max": worst("fp32_rel_l1"), "fp32_rel_linf_max": worst("fp32_rel_linf"),
            "fp64_rel_l1_max": worst("fp64_rel_l1"), "fp64_rel_linf_max": worst("fp64_rel_linf"),
            "fp32_within_1e-5": sum(1 for x in rows if x["fp32_rel_l1"] <= 1e-5),
            "fp64_within_1e-5": sum(1 for x in rows if x["fp64_rel_l1"] <= 1e-5),
            "per_instance": rows}
        log("bench[cpu]: oracle over the %d-instance subset, %d steps, in %.1f s" %
            (len(rows), steps_b, time.perf_counter() - t1))
    if coupled:
        parity["coupled_c4"] = coupled_curve_parity(coupled)
    return cpu, parity


def coupled_curve_parity(coupled):
    """The coupled run's stress-strain history against the oracle's history
    stored in tests/golden/coupled_c4_history.json (written from oracle/
    only); deviations over each quantity's largest magnitude on the curve."""
    if not os.path.exists(GOLDEN_C4) or coupled["steps"] != 5000:
        return None
    g = json.load(open(GOLDEN_C4))
    ref = [dict(zip(g["columns"], r)) for r in g["history"]]
    hist = coupled["hist"]
    if len(hist) != len(ref):
        return None
    out = {}
    for k in ("eps13", "sigma13", "phi_mean"):
        scale = max(abs(r[k]) for r in ref)
        out[k + "_max_dev"] = max(abs(h[k] - r[k]) for h, r in zip(hist, ref)) / scale
    out["sum_abs_max_dev"] = max(abs(h["sum_abs"] - r["sum_abs"]) for h, r in zip(hist, ref)) / coupled["s0"]
    out["records"] = len(ref)
    out["reference"] = os.path.relpath(GOLDEN_C4, ROOT)
    return out


# ------------------------------------------------------------------- main

def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--repeats", type=int, default=5)
    ap.add_argument("--tile-rows", type=int, default=0, help="0: the library's default rule")
    ap.add_argument("--no-autotune", action="store_true",
                    help="keep --tile-rows and --schedule instead of timing the candidates (fdm_autotune)")
    ap.add_argument("--schedule", default="auto", choices=["auto", "plain", "fused"])
    ap.add_argument("--only-headline", action="store_true", help="skip every leg but the headline")
    ap.add_argument("--no-fp64", action="store_true")
    ap.add_argument("--no-loop", action="store_true")
    ap.add_argument("--loop-schedule", default="auto", choices=["auto", "plain", "fused"],
                    help="schedule of the 2048^2 loop leg (with --no-autotune: the one timed)")
    ap.add_argument("--loop-rows", type=int, default=0, help="tile rows of the loop leg (0: the default rule)")
    ap.add_argument("--no-batched", action="store_true")
    ap.add_argument("--batched-steps", type=int, default=500)
    ap.add_argument("--batched-schedules", default="batched,plain,fused",
                    help="schedules of the batched leg, comma-separated (plain: one launch per instance)")
    ap.add_argument("--no-coupled", action="store_true")
    ap.add_argument("--coupled-steps", type=int, default=5000)
    ap.add_argument("--no-fd", action="store_true")
    ap.add_argument("--no-c1", action="store_true")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=10.0, help="least oracle time on the headline workload")
    ap.add_argument("--copy-probe", type=int, default=0, metavar="N",
                    help="also run one Euler step on an N x N zero state: its copy-back is a plain copy kernel "
                         "of 4*N*N bytes per array each way, the byte reference for the memory counters")
    ap.add_argument("--profile-from", nargs=3, metavar=("FETCH_DIR", "WRITE_DIR", "SQ_DIR"),
                    help="no run: summarise rocprofv3 FETCH_SIZE, WRITE_SIZE and SQ counter CSVs of a profiled "
                         "headline run (with --copy-probe) into the counter file")
    ap.add_argument("--profile-out", default=PROFILE_FILE)
    args = ap.parse_args()

    if args.profile_from:
        write_profile_summary(*args.profile_from, args.profile_out, args.copy_probe or 16384, args.tile_rows)
        return

    world = int(os.environ.get("WORLD_SIZE", "1"))
    if args.gpus != 1 or world != 1:
        print("bench.py measures one GPU only: the library has no multi-GPU path "
              "(--gpus %d, WORLD_SIZE %d requested)" % (args.gpus, world), file=sys.stderr)
        sys.exit(2)
    if args.only_headline:
        args.no_fp64 = args.no_loop = args.no_batched = args.no_coupled = args.no_fd = args.no_c1 = True

    import torch
    from paper_1911_03225_amd import fdm, workloads as W_

    K, warm = args.steps, args.warmup
    autotune = not args.no_autotune
    log("bench: headline workload, 4096^2 bands + celerity field")
    head_r, value, roofline, inputs = headline_leg(fdm, W_, K, warm, args.repeats, autotune, args.tile_rows,
                                                   args.schedule, log)
    fp64 = loop = fd = c1 = batched = coupled = None
    extra = {}
    if not args.no_fp64:
        fp64, extra["fp64_state"] = fp64_state_leg(fdm, K, warm, args.repeats, inputs, log)
    if not args.no_loop:
        r2, extra["loop_2048"], ins = loop_leg(fdm, W_, K, warm, args.repeats, autotune, log,
                                               args.loop_schedule, args.loop_rows)
        loop = (r2, ins)
    if not args.no_fd:
        r3, extra["fully_discrete"], ins = fully_discrete_leg(fdm, W_, K, warm, args.repeats, autotune, log)
        fd = (r3, ins)
    if not args.no_c1:
        c1, extra["c1_full_length"] = c1_leg(fdm, W_, log)
    if args.copy_probe:
        m = args.copy_probe
        z11 = torch.zeros((m, m), dtype=torch.float32, device="cuda:0")
        z12 = torch.zeros((m, m), dtype=torch.float32, device="cuda:0")
        ctx1 = fdm.fdm_transport_init(fdm.desc(m, m, limiter="minmod", cfl=0.25, v0=-1.0, time_order=1))
        fdm.fdm_transport_step(ctx1, z11, z12, 1)
        torch.cuda.synchronize()
        fdm.fdm_destroy(ctx1)
        del z11, z12
        log("bench: copy probe: one Euler step on %dx%d, copy kernel of %d bytes per array" % (m, m, 4 * m * m))
    if not args.no_batched:
        extra["batched_vs_plain"], keep = batched_leg(fdm, W_, args.batched_steps, log, autotune=autotune,
                                                      schedules=tuple(args.batched_schedules.split(",")))
        batched = dict(keep, K=args.batched_steps)
    if not args.no_coupled:
        extra["coupled"], coupled = coupled_leg(fdm, W_, args.coupled_steps, log)

    cpu, parity = None, None
    if not args.no_cpu_baseline:
        cpu, parity = cpu_baseline_leg(K, (head_r, inputs), loop, fd, c1, fp64, batched, coupled,
                                       args.cpu_seconds, log)
        for key, leg in (("c3_fp64", "fp64_state"), ("c2_fp32", "loop_2048"), ("fully_discrete_fp32",
                                                                               "fully_discrete"),
                         ("c1_fp32_full_length", "c1_full_length"), ("batched_subset", "batched_vs_plain"),
                         ("coupled_c4", "coupled")):
            if key in parity and leg in extra:
                extra[leg]["parity"] = parity[key]

    out = {
        "metric": METRIC, "value": round(value, 1), "unit": "cell-updates/s",
        "n_gpus": 1, "steps": K, "warmup": warm, "ms_per_step": round(1e3 * head_r["seconds"] / K, 5),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "bands + celerity field 4096x4096: 64 diagonal bands (seed 3) under a 16-mode "
                               "Fourier celerity tanh(tau/0.5), LAW, minmod, Heun, CFL 0.45",
                   "grid": [4096, 4096], "limiter": "minmod", "cfl": 0.45, "dt": head_r["dt"], "time_order": 2,
                   "schedule": head_r["schedule"], "tile_rows": head_r["tile_rows"],
                   "tiling": head_r["tile_choice"],
                   "precision": "fp32"},
        "hbm_frac_algorithmic": roofline["frac"],
        "roofline": roofline,
        "parity": parity["c3_fp32"] if parity else None,
        "cpu_baseline": cpu,
    }
    out.update(extra)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
