#!/usr/bin/env python3
"""Benchmark: NNP energy + force throughput (atom-steps/s) on one MI355X.

One step is one full energy + force evaluation through the C ABI
(``nnp_compute``): cell list, neighbour lists, descriptors, per-species
networks (forward + backward), FP64 energy sum, descriptor adjoint and FP64
force gather.  The neighbour search reruns every step; inputs stay resident
in device memory.  The timed steps use the library's production path (direct
launches, one HIP-graph replay for few atoms); a second pass of the same length with per-stage
HIP events gives the kernel durations used for the roofline entry.

Default workload: the largest configuration, a periodic water box of 87,000
molecules (261,000 atoms, L = 137.7 A), FP32 form as ``value``; the BF16 form
is timed on the same input, and both are checked against the FP64 oracle over
every atom (force relative and absolute RMSE, energy error per atom).  The line
also carries the NVE check on the 4,096-molecule box (1,000 velocity-Verlet
steps of 0.5 fs and 2,000 of 0.25 fs over the same 0.5 ps: energy drift and
deviation).  ``--workload`` also accepts the 192-, 12,288- and 98,304-atom
boxes, the batch of 256 open H/C/N/O molecules and the solute in MM charges.

Prints one JSON line on stdout; progress goes to stderr.
"""
from __future__ import annotations

import argparse
import gc
import json
import math
import os
import statistics
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

METRIC = "NNP energy+force atom-steps/s (BF16 vs FP32 form) at stated force RMSE"

WORKLOADS = {
    "c1": dict(kind="water", n_mol=64, L=12.42, desc="periodic water box, 64 molecules (192 atoms), L=12.42 A"),
    "c2": dict(kind="water", n_mol=4096, L=49.7, desc="periodic water box, 4,096 molecules (12,288 atoms), L=49.7 A"),
    "c3": dict(kind="water", n_mol=32768, L=99.4, desc="periodic water box, 32,768 molecules (98,304 atoms), L=99.4 A"),
    "c5a": dict(kind="water", n_mol=87000, L=137.7,
                desc="periodic water box, 87,000 molecules (261,000 atoms), L=137.7 A"),
    "c2e8": dict(kind="water", n_mol=4096, L=49.7, n_members=8,
                 desc="periodic water box, 4,096 molecules (12,288 atoms), L=49.7 A, 8-member ensemble of "
                      "networks sharing one descriptor (energy and forces are the member means)"),
    "c4": dict(kind="batch", n_sys=256, desc="256 open H/C/N/O walk molecules of 24-300 atoms, one batched call"),
    "c5b": dict(kind="solute_mm",
                desc="60-atom H/C/N/O walk solute in 10,000 fixed-charge MM waters (30,000 point charges "
                     "entering as the extra input channel, 12 A), periodic L=68.3 A"),
    "c5e": dict(kind="solute_ee",
                desc="60-atom H/C/N/O walk solute in 10,000 fixed-charge MM waters, electrostatic embedding "
                     "with network-predicted atomic charges (E_i = e_i + q_i phi_i), periodic L=68.3 A"),
}

# Peaks (MI355X, published): HBM 8 TB/s; dense MFMA BF16 and FP16 2.5 PFLOP/s.
# VALU: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz = 3.93e13 lane-operations/s (unpacked FP32
# and FP64 issue at that rate; transcendentals at a quarter of it, counted as 4 operations).
PEAK_HBM_GBS = 8000.0
# The FP32 network form runs on FP16 operand pairs ("split"): four FP16 products per FP32 one in
# the forward pass, three in the backward pass.
PEAK_MFMA_TFLOPS = {"split": 2500.0 / 3.5, "bf16": 2500.0}
PEAK_VALU_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12

# Algorithmic VALU lane-operations per unit of work (transcendental = 4): the arithmetic the
# method needs per radial pair and per angular triplet, forward and adjoint.
OPS_FWD_RAD_PAIR = 155
OPS_FWD_TRIPLET = 150
OPS_BWD_RAD_PAIR = 200
OPS_BWD_TRIPLET = 300
# MM potential channel, per (NNP atom, MM charge) pair tested: minimum-image
# displacement and r^2 (16), inside the cutoff rsq, cos and the charge term (13),
# the wavefront sum over MM lanes (12); the adjoint adds sin, d(fc/r)/dr, the
# pair vector and three wavefront sums (80 in all).  Transcendentals count 4.
OPS_MM_FWD_PAIR = 40
OPS_MM_BWD_PAIR = 80


# rocprofv3 summaries committed under profiles/ (written by --summarize-profiles).
PROFILE_TAGS = {"c1": "water192", "c2": "water12288", "c3": "water98304", "c5a": "water261000",
                "c2e8": "water12288_ensemble8",
                "c4": "hcno_batch256", "c5b": "hcno60_mm30000", "c5e": "hcno60_mm30000_charges"}
CSRC = os.path.join(ROOT, "paper_2604_21441_amd", "csrc")
CALIB_BYTES = 1 << 30   # --calib-copy: one device copy of this many bytes (read + write)
# Shader-sequencer counters, two passes of at most eight SQ counters (whole-GPU sums per dispatch).
SQ_PASSES = (("SQ_WAVES", "SQ_INSTS_VALU", "SQ_INSTS_MFMA", "SQ_VALU_MFMA_BUSY_CYCLES", "SQ_INSTS_LDS",
              "SQ_LDS_BANK_CONFLICT", "SQ_ACTIVE_INST_LDS", "SQ_WAIT_INST_LDS"),
             ("SQ_WAVE_CYCLES", "SQ_WAIT_ANY", "SQ_WAIT_INST_ANY", "SQ_ACTIVE_INST_VALU", "SQ_INSTS_SALU",
              "SQ_INSTS_VMEM_RD", "SQ_INSTS_VMEM_WR", "SQ_BUSY_CU_CYCLES"))
N_SIMD = 256 * 4
CLOCK_HZ = 2.4e9


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_sources():
    """Kernel base name -> defining source file and a digest of that file, the shared
    header and the build script (a profile's counters are stale once these change).
    Comments and the layout of whitespace are left out of the digest: editing them
    changes no kernel."""
    import glob
    import hashlib
    import re

    def code(path):
        text = open(path, "rb").read()
        if path.endswith((".hip", ".h")):
            text = re.sub(rb"/\*.*?\*/", b"", text, flags=re.S)
            text = re.sub(rb"//[^\n]*", b"", text)
            text = re.sub(rb"\s+", b" ", text)
        return text

    common = b"".join(code(f) for f in (os.path.join(CSRC, "nnp_internal.h"),
                                        os.path.join(ROOT, "paper_2604_21441_amd", "build.py")))
    out = {}
    for f in sorted(glob.glob(os.path.join(CSRC, "*.hip"))):
        src = code(f)
        dig = hashlib.sha256(src + common).hexdigest()[:16]
        for m in re.finditer(rb"__global__\s+(?:__launch_bounds__\((?:[^()]|\([^()]*\))*\)\s+)?void\s+(k_\w+)\s*\(", src):
            out[m.group(1).decode()] = {"file": os.path.basename(f), "digest": dig}
    return out


def network_form(prec):
    """How the network's products run (a key of PEAK_MFMA_TFLOPS)."""
    return "bf16" if prec == "bf16" else "split"


def stage_kernel(stage, variants, prec, cfg, periodic=True, n=0):
    """Name (as the profiler prints it, without namespaces and arguments) of the kernel
    that runs a stage, given the variants the library reports."""
    widths = list(cfg["widths"])
    k0 = (widths[0] + 31) // 32 * 32
    op = {"bf16": 1, "split": 2}[network_form(prec)]
    v = variants or {}
    if stage == "neighbours":
        return "k_neighbours" if v.get("neighbours", 0) == 0 else "k_neighbours_cell"
    if stage == "descriptor":
        small = "k_desc_fwd_pool<1>" if 0 < n <= 8 * 256 else "k_desc_fwd_pool<2>"   # eight atoms per CU
        return ["k_desc_fwd", "k_desc_fwd_rows<16>", "k_desc_fwd_rows<8>", small,
                "k_desc_fwd_pool<4>"][v.get("descriptor", 1)]
    if stage == "network":
        nv = v.get("network", 2)
        dims = f"{k0}, {widths[1]}, {widths[2]}, {widths[3]}, {op}"
        if widths[-1] == 2:   # charge output: one kernel template, (columns, mixed, wavefronts) per variant
            c, mixed, nw = {2: (2, False, 4), 3: (2, False, 4), 4: (2, True, 4), 5: (1, False, 8),
                            6: (2, True, 8), 7: (2, False, 8)}.get(nv, (1, False, 4))
            return f"k_mlp_split_q<{dims}, {c}, {'true' if mixed else 'false'}, {nw}>"
        if nv in (8, 9) and prec == "bf16" and k0 <= 128:
            return f"k_mlp_lds<{k0}, {widths[1]}, {widths[2]}, {widths[3]}, {'2, 8' if nv == 8 else '1, 16'}>"
        if nv in (8, 9):
            nv = 2
        cols = {1: 1, 2: 2, 3: 4 if k0 <= 128 else 2}.get(nv)
        if nv == 3 and cols == 4 and op == 2:
            return f"k_mlp_split8<{dims}, 4, false>"
        if nv == 4:
            return f"k_mlp_mixed<{dims}>"
        if nv in (5, 6, 7):
            return f"k_mlp_split8<{dims}, {1 if nv == 5 else 2}, {'true' if nv == 6 else 'false'}>"
        return f"k_mlp_reg<{dims}>" if nv == 0 else f"k_mlp_split<{dims}, {cols}>"
    if stage == "adjoint":
        return f"k_desc_adj<{len(cfg['species'])}>"
    return {"gather": "k_force_gather", "energy": "k_force_gather", "mm": "k_mm_fwd",
            "mm_adjoint": "k_mm_bwd<1>"}.get(stage)   # (small ML regions: one MM atom per lane)


def profile_entry(workload, kernel):
    """A kernel's entry in the committed rocprofv3 summary of this workload (average
    duration, calibrated HBM bytes per dispatch), or None if absent or taken from
    other sources than the ones present now."""
    path = os.path.join(ROOT, "profiles", f"nnp_compute_{PROFILE_TAGS[workload]}_traffic.json")
    if kernel is None or not os.path.exists(path):
        return None
    k = json.load(open(path))["kernels"].get(kernel)
    src = kernel_sources().get(kernel.split("<")[0])
    if not k or src is None or src["digest"] != k.get("digest"):
        return None
    return k


def profile_traffic(workload, kernel):
    """HBM bytes per dispatch (calibrated FETCH_SIZE + WRITE_SIZE) of a kernel from the
    committed profile of this workload, or None."""
    k = profile_entry(workload, kernel)
    if not k or k.get("fetch_bytes") is None or k.get("write_bytes") is None:
        return None
    return k["fetch_bytes"] + k["write_bytes"]


def profile_commands(workload):
    """The commands that produce the rocprofv3 output --summarize-profiles reads
    ($ROOT = repository root, $OUT = output folder)."""
    b = "python3 $ROOT/bench.py"
    return [
        "cd /tmp && export TMPDIR=/tmp",
        f"rocprofv3 --kernel-trace --stats --output-format csv -d $OUT/kt_{workload} -o run -- "
        f"{b} --workload {workload} --steps 20 --warmup 5 --no-cpu --nve 0",
        f"rocprofv3 --pmc FETCH_SIZE --output-format csv -d $OUT/FETCH_SIZE_{workload} -o run -- "
        f"{b} --workload {workload} --steps 3 --warmup 1 --no-cpu --nve 0",
        f"rocprofv3 --pmc WRITE_SIZE --output-format csv -d $OUT/WRITE_SIZE_{workload} -o run -- "
        f"{b} --workload {workload} --steps 3 --warmup 1 --no-cpu --nve 0",
        f"rocprofv3 --pmc {' '.join(SQ_PASSES[0])} --output-format csv -d $OUT/SQA_{workload} -o run -- "
        f"{b} --workload {workload} --steps 3 --warmup 1 --no-cpu --nve 0",
        f"rocprofv3 --pmc {' '.join(SQ_PASSES[1])} --output-format csv -d $OUT/SQB_{workload} -o run -- "
        f"{b} --workload {workload} --steps 3 --warmup 1 --no-cpu --nve 0",
        f"rocprofv3 --pmc FETCH_SIZE --output-format csv -d $OUT/calib_FETCH_SIZE -o run -- {b} --calib-copy",
        f"rocprofv3 --pmc WRITE_SIZE --output-format csv -d $OUT/calib_WRITE_SIZE -o run -- {b} --calib-copy",
        f"python3 bench.py --summarize-profiles $OUT --workload {workload}",
    ]


def _short_name(name):
    s = name.replace("void ", "").replace("nnp::(anonymous namespace)::", "").strip()
    depth = 0
    for i, ch in enumerate(s):
        if ch == "<":
            depth += 1
        elif ch == ">":
            depth -= 1
        elif ch == "(" and depth == 0:
            return s[:i]
    return s


def _counter_means(path):
    """Mean counter value per kernel (over dispatches) from a counter_collection CSV."""
    import csv
    import collections
    acc = collections.defaultdict(list)
    for r in csv.DictReader(open(path)):
        acc[(_short_name(r["Kernel_Name"]), r["Counter_Name"])].append(float(r["Counter_Value"]))
    return {k: (sum(v) / len(v), len(v)) for k, v in acc.items()}


def summarize_profiles(out_dir, workload):
    """Write <out_dir>/profiles/nnp_compute_<tag>_kernels.md and _traffic.json from the
    rocprofv3 output under out_dir.  Run it on the tree that was profiled: the source
    digests it records are those of the files present when it runs."""
    import csv
    tag = PROFILE_TAGS[workload]
    stats = list(csv.DictReader(open(os.path.join(out_dir, f"kt_{workload}", "run_kernel_stats.csv"))))
    calib = {}
    for c in ("FETCH_SIZE", "WRITE_SIZE"):
        means = _counter_means(os.path.join(out_dir, f"calib_{c}", "run_counter_collection.csv"))
        kib = max(v for (k, cn), (v, _) in means.items() if "copyBuffer" in k and cn == c)
        calib[c] = CALIB_BYTES / (kib * 1024.0)       # bytes per counted byte
    counters = {}
    for c in ("FETCH_SIZE", "WRITE_SIZE"):
        for (k, cn), (v, nd) in _counter_means(os.path.join(out_dir, f"{c}_{workload}",
                                                            "run_counter_collection.csv")).items():
            counters.setdefault(k, {})[c] = v * 1024.0 * calib[c]
    srcs = kernel_sources()
    kernels = {}
    for r in stats:
        k = _short_name(r["Name"])
        if not k.startswith("k_"):
            continue
        src = srcs.get(k.split("<")[0], {})
        kernels[k] = {"calls": int(r["Calls"]), "avg_us": float(r["AverageNs"]) / 1e3,
                      "min_us": float(r["MinNs"]) / 1e3, "max_us": float(r["MaxNs"]) / 1e3,
                      "share_pct": float(r["Percentage"]),
                      "fetch_bytes": counters.get(k, {}).get("FETCH_SIZE"),
                      "write_bytes": counters.get(k, {}).get("WRITE_SIZE"),
                      "source": src.get("file"), "digest": src.get("digest")}
    cmds = profile_commands(workload)
    doc = {"workload": WORKLOADS[workload]["desc"], "calibration": calib, "commands": cmds, "kernels": kernels}
    dest = os.path.join(out_dir, "profiles")
    os.makedirs(dest, exist_ok=True)
    with open(os.path.join(dest, f"nnp_compute_{tag}_traffic.json"), "w") as f:
        json.dump(doc, f, indent=1)
    lines = [f"# Kernel durations and HBM traffic: {WORKLOADS[workload]['desc']}", "",
             "rocprofv3 kernel-trace statistics (every dispatch of the run: autotuning candidates, the",
             "FP32 and BF16 forms, the production calls and the event-timed pass) and per-dispatch HBM bytes",
             "from FETCH_SIZE / WRITE_SIZE, scaled by what the same counters read for a plain",
             f"{CALIB_BYTES >> 20} MiB device copy (fetch x{calib['FETCH_SIZE']:.3f}, "
             f"write x{calib['WRITE_SIZE']:.3f}).", "", "Commands ($ROOT = repository root, $OUT = output folder):",
             "", "```"] + cmds + ["```", "",
             "| kernel | calls | avg us | min us | max us | % time | fetch MB | write MB | source |",
             "|---|---:|---:|---:|---:|---:|---:|---:|---|"]
    for k, e in sorted(kernels.items(), key=lambda kv: -kv[1]["share_pct"]):
        fb = "" if e["fetch_bytes"] is None else f"{e['fetch_bytes'] / 1e6:.2f}"
        wb = "" if e["write_bytes"] is None else f"{e['write_bytes'] / 1e6:.2f}"
        lines.append(f"| `{k}` | {e['calls']} | {e['avg_us']:.2f} | {e['min_us']:.2f} | {e['max_us']:.2f} | "
                     f"{e['share_pct']:.2f} | {fb} | {wb} | {e['source']} |")
    with open(os.path.join(dest, f"nnp_compute_{tag}_kernels.md"), "w") as f:
        f.write("\n".join(lines) + "\n")
    log(f"[bench] wrote {dest}/nnp_compute_{tag}_kernels.md and _traffic.json ({len(kernels)} kernels)")
    # shader-sequencer counters, when their passes were collected
    sq = {}
    for pi, names in enumerate(SQ_PASSES):
        path = os.path.join(out_dir, f"SQ{'AB'[pi]}_{workload}", "run_counter_collection.csv")
        if not os.path.exists(path):
            continue
        for (k, cn), (v, nd) in _counter_means(path).items():
            if k.startswith("k_"):
                sq.setdefault(k, {})[cn] = v
    if not sq:
        return
    lines = [f"# Shader-sequencer counters: {WORKLOADS[workload]['desc']}", "",
             "Per-dispatch means of whole-GPU counter sums (rocprofv3 --pmc, two passes of eight SQ",
             "counters; commands in the kernels summary of this workload).  Derived columns:",
             f"* MFMA busy = SQ_VALU_MFMA_BUSY_CYCLES / ({N_SIMD} SIMDs x kernel duration x {CLOCK_HZ / 1e9} GHz),",
             "  the duration being the kernel-trace average above;",
             "* VALU/wave and MFMA/wave = SQ_INSTS_VALU / SQ_WAVES and SQ_INSTS_MFMA / SQ_WAVES",
             "  (VALU counts include the MFMA instructions);",
             "* LDS conflict share = SQ_LDS_BANK_CONFLICT / (SQ_ACTIVE_INST_LDS + SQ_LDS_BANK_CONFLICT);",
             "* wait share = SQ_WAIT_ANY / SQ_WAVE_CYCLES (waves waiting on memory counters).", "",
             "| kernel | waves | VALU/wave | MFMA/wave | MFMA busy | LDS instr/wave | LDS conflict share | "
             "wait share | VMEM rd/wave | VMEM wr/wave |",
             "|---|---:|---:|---:|---:|---:|---:|---:|---:|---:|"]
    for k, e in sorted(sq.items(), key=lambda kv: -kernels.get(kv[0], {}).get("share_pct", 0.0)):
        waves = e.get("SQ_WAVES", 0.0) or float("nan")
        dur = kernels.get(k, {}).get("avg_us")
        busy = e.get("SQ_VALU_MFMA_BUSY_CYCLES")
        mf = (busy / (N_SIMD * dur * 1e-6 * CLOCK_HZ)) if (busy is not None and dur) else None
        lds_a, lds_c = e.get("SQ_ACTIVE_INST_LDS", 0.0), e.get("SQ_LDS_BANK_CONFLICT", 0.0)
        conf = lds_c / (lds_a + lds_c) if lds_a + lds_c > 0 else None
        wc = e.get("SQ_WAVE_CYCLES")
        wait = e.get("SQ_WAIT_ANY", 0.0) / wc if wc else None
        fmt = lambda x, spec: "" if x is None else format(x, spec)
        lines.append(f"| `{k}` | {waves:.0f} | {fmt(e.get('SQ_INSTS_VALU', 0.0) / waves, '.0f')} | "
                     f"{fmt(e.get('SQ_INSTS_MFMA', 0.0) / waves, '.0f')} | {fmt(mf, '.3f')} | "
                     f"{fmt(e.get('SQ_INSTS_LDS', 0.0) / waves, '.0f')} | {fmt(conf, '.2f')} | {fmt(wait, '.2f')} | "
                     f"{fmt(e.get('SQ_INSTS_VMEM_RD', 0.0) / waves, '.1f')} | "
                     f"{fmt(e.get('SQ_INSTS_VMEM_WR', 0.0) / waves, '.1f')} |")
    with open(os.path.join(dest, f"nnp_compute_{tag}_sq.md"), "w") as f:
        f.write("\n".join(lines) + "\n")
    log(f"[bench] wrote {dest}/nnp_compute_{tag}_sq.md ({len(sq)} kernels)")


def network_flops_per_atom(widths):
    """2 x multiply-adds of the forward chain (one output row, or two with a charge
    output) plus the three backward products."""
    K0, N1, N2, N3 = widths[0], widths[1], widths[2], widths[3]
    fwd = K0 * N1 + N1 * N2 + N2 * N3 + N3 * widths[4]
    bwd = N3 * N2 + N2 * N1 + N1 * K0
    return 2 * (fwd + bwd)


def build_inputs(name):
    import numpy as np
    import synthetic as sy
    w = WORKLOADS[name]
    if w["kind"] == "water":
        cfg = sy.model_config("water")
        pos, Z, box = sy.water_box(w["n_mol"], w["L"], seed=0)
        return cfg, dict(pos=pos, Z=Z, box=box, offsets=None, mm_pos=None, mm_q=None,
                         n_members=w.get("n_members", 1))
    if w["kind"] in ("solute_mm", "solute_ee"):
        cfg = sy.model_config("hcno_mm" if w["kind"] == "solute_mm" else "hcno_ee")
        s = sy.solute_in_water(seed=0)
        return cfg, dict(pos=s["pos"], Z=s["Z"], box=s["box"], offsets=None, mm_pos=s["mm_pos"], mm_q=s["mm_q"])
    cfg = sy.model_config("hcno")
    pos, Z, off = sy.walk_batch(w["n_sys"], seed=0)
    return cfg, dict(pos=pos, Z=Z, box=None, offsets=np.asarray(off, np.int32), mm_pos=None, mm_q=None)


def run_form(P, cfg, flat, inp, prec, steps, warmup, autotune=True):
    """Time `steps` production calls (the library's own launches, preallocated outputs, topology
    reused), then the same number of calls with per-stage HIP-event timing."""
    import numpy as np
    import torch
    m = P.NNPModel(cfg, weights=flat, precision=prec, n_members=inp.get("n_members", 1))
    d = torch.from_numpy(inp["pos"]).cuda()
    n = d.shape[0]
    batched = inp["offsets"] is not None
    if batched:
        n_sys = len(inp["offsets"]) - 1
        m.reserve(n, n_sys)
        E = torch.empty(n_sys, dtype=torch.float64, device="cuda")
        F = torch.empty((n, 3), dtype=torch.float64, device="cuda")
        first = lambda: m.compute_batch(d, inp["Z"], inp["offsets"], out=(E, F))
        call = lambda: m.compute_batch(d, None, inp["offsets"], out=(E, F))
    elif inp["mm_pos"] is not None:   # MM charges through the extra input channel
        dm = torch.from_numpy(inp["mm_pos"]).cuda()
        dq = torch.from_numpy(inp["mm_q"]).cuda()
        m.reserve(n, 1, dm.shape[0])
        E = torch.empty(1, dtype=torch.float64, device="cuda")
        F = torch.empty((n, 3), dtype=torch.float64, device="cuda")
        Fmm = torch.empty((dm.shape[0], 3), dtype=torch.float64, device="cuda")
        first = lambda: m.compute(d, inp["Z"], inp["box"], mm_pos=dm, mm_q=dq, out=(E, F, Fmm))
        call = lambda: m.compute(d, None, inp["box"], mm_pos=dm, mm_q=dq, out=(E, F, Fmm))
    else:
        m.reserve(n)
        E = torch.empty(1, dtype=torch.float64, device="cuda")
        F = torch.empty((n, 3), dtype=torch.float64, device="cuda")
        first = lambda: m.compute(d, inp["Z"], inp["box"], out=(E, F, None))
        call = lambda: m.compute(d, None, inp["box"], out=(E, F, None))
    first()
    torch.cuda.synchronize()
    st = m.status()
    if st != 0:
        raise RuntimeError(f"device status {st} after the first call")
    E_first = E.detach().cpu().numpy().astype(float)
    F_first = F.detach().cpu().numpy()
    if inp.get("mm_pos") is not None:   # forces on NNP atoms, then on MM atoms
        F_first = np.concatenate([F_first, Fmm.detach().cpu().numpy()])
    if autotune:
        m.autotune(10)
    tuned = m.variants()
    gc.collect()
    gc.disable()   # a collector pause inside the timed loop would be charged to the library
    for _ in range(warmup):
        call()
    torch.cuda.synchronize()
    host_ms = []
    t0 = time.perf_counter()
    for _ in range(steps):
        tc = time.perf_counter()
        call()
        host_ms.append(time.perf_counter() - tc)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    gc.enable()
    if m.status() != 0:
        raise RuntimeError("device status flagged an error during the timed steps")
    # per-stage event timing (stage launches issued directly; same kernels)
    P.nnp_profile_enable(m.h, steps)
    torch.cuda.synchronize()
    tp0 = time.perf_counter()
    for _ in range(steps):
        call()
    torch.cuda.synchronize()
    tp1 = time.perf_counter()
    stage_ms, calls = P.nnp_profile_read(m.h)
    P.nnp_profile_enable(m.h, 0)
    cnt = m.read(P._lib.NNP_BUF_NBR_COUNT)
    out = {
        "ms_per_step": (t1 - t0) * 1e3 / steps,
        "host_call_ms": {"median": statistics.median(host_ms) * 1e3, "max": max(host_ms) * 1e3},
        "profiled_ms_per_step": (tp1 - tp0) * 1e3 / steps,
        "stage_ms": {k: v / max(calls, 1) for k, v in stage_ms.items()},
        "E": E_first,
        "F": F_first,
        "rad_pairs": int(cnt[:, 0].sum()),
        "triplets": int((cnt[:, 1].astype(np.int64) * (cnt[:, 1] - 1) // 2).sum()),
        "n": n,
        "n_mm": 0 if inp.get("mm_pos") is None else len(inp["mm_q"]),
        "tuned": tuned,
        "n_members": inp.get("n_members", 1),
    }
    m.close()
    return out


def oracle_reference(cfg, w, inp, sample_centres):
    """FP64 oracle energy/forces.  Full evaluation, or exact forces on sampled atoms."""
    import numpy as np
    import oracle as orc
    if inp["offsets"] is not None:
        E, F = orc.evaluate_batch(inp["pos"], inp["Z"], inp["offsets"], cfg, w)
        return {"E": E, "F": F, "atoms": np.arange(len(inp["Z"]))}
    if inp.get("mm_pos") is not None:
        r = orc.evaluate(inp["pos"], inp["Z"], cfg, w, box=inp["box"], mm_pos=inp["mm_pos"], mm_q=inp["mm_q"])
        F = np.concatenate([r["F"], r["F_mm"]])
        return {"E": np.array([r["E"]]), "F": F, "atoms": np.arange(len(F))}
    if sample_centres is None:
        r = orc.evaluate(inp["pos"], inp["Z"], cfg, w, box=inp["box"])
        return {"E": np.array([r["E"]]), "F": r["F"], "atoms": np.arange(len(inp["Z"]))}
    I, J = orc.neighbour_pairs(inp["pos"], float(cfg["rc_rad"]), inp["box"], centres=sample_centres)
    cs = np.unique(np.concatenate([sample_centres, J]))
    r = orc.evaluate(inp["pos"], inp["Z"], cfg, w, box=inp["box"], centres=cs)
    return {"E": None, "F": r["F"], "atoms": sample_centres}


def cpu_baseline(cfg, w, inp, reps):
    """The oracle as it stands, timed on the host cores on a bounded sample of the workload."""
    import numpy as np
    import torch
    import oracle as orc
    n = len(inp["Z"])
    if inp["offsets"] is not None:
        off = inp["offsets"]
        k = min(16, len(off) - 1)
        sub = slice(0, int(off[k]))
        sample = f"first {k} molecules ({int(off[k])} atoms) of the batch, E+F, median of {reps}"
        atoms = int(off[k])
        fn = lambda: orc.evaluate_batch(inp["pos"][sub], inp["Z"][sub], off[:k + 1], cfg, w)
    elif inp.get("mm_pos") is not None:
        sample = f"full {n}-atom solute with its {len(inp['mm_q'])} MM charges, E+F, median of {reps}"
        atoms = n
        fn = lambda: orc.evaluate(inp["pos"], inp["Z"], cfg, w, box=inp["box"], mm_pos=inp["mm_pos"],
                                  mm_q=inp["mm_q"])
    elif n <= 20000:
        sample = f"full {n}-atom system, E+F, median of {reps}"
        atoms = n
        fn = lambda: orc.evaluate(inp["pos"], inp["Z"], cfg, w, box=inp["box"])
    else:
        rng = np.random.default_rng(0)
        cs = np.sort(rng.choice(n, 8192, replace=False))
        sample = f"atomic energies of 8,192 random atoms of the {n}-atom box and their gradients, median of {reps}"
        atoms = cs.size
        fn = lambda: orc.evaluate(inp["pos"], inp["Z"], cfg, w, box=inp["box"], centres=cs)
    # about 10 s of CPU work: at least `reps` evaluations, more when one is short
    t = time.perf_counter()
    fn()
    times = [time.perf_counter() - t]
    total = max(reps, min(30, math.ceil(10.0 / max(times[0], 1e-3))))
    for _ in range(total - 1):
        t = time.perf_counter()
        fn()
        times.append(time.perf_counter() - t)
    sample = sample.replace(f"median of {reps}", f"median of {len(times)}")
    t = statistics.median(times)
    return {"value": atoms / t, "unit": "atom-steps/s", "cores": torch.get_num_threads(), "kind": "oracle",
            "sample": sample, "seconds_per_eval": t}


def roofline(res, cfg, prec, stage, workload, periodic):
    """Roofline entry for one stage from its live event time and its algorithmic work, with
    the committed rocprofv3 average of the same kernel beside it."""
    out = _roofline(res, cfg, prec, stage, workload, periodic)
    out["timing"] = ("HIP events on the call's stream around the stage's direct launches, averaged "
                     "over the profiled pass (without the events each kernel runs 1-3 us shorter)")
    out["event_us"] = res["stage_ms"][stage] * 1e3
    k = profile_entry(workload, out.get("kernel"))
    if k is not None and k.get("avg_us"):
        out["rocprof_avg_us"] = k["avg_us"]
        out["frac_at_rocprof_avg"] = out["frac"] * out["event_us"] / k["avg_us"]
    else:
        out["rocprof_avg_us"] = None
        out["frac_at_rocprof_avg"] = None
    return out


def _roofline(res, cfg, prec, stage, workload, periodic):
    widths = list(cfg["widths"])
    kernel = stage_kernel(stage, res["tuned"], prec, cfg, periodic, res["n"])
    traffic = profile_traffic(workload, kernel)
    n = res["n"]
    t = res["stage_ms"][stage] * 1e-3
    D = widths[0]
    if stage == "network":
        flops = network_flops_per_atom(widths) * n * res.get("n_members", 1)
        ach = flops / t / 1e12
        peak = PEAK_MFMA_TFLOPS[network_form(prec)]
        return {"kernel": kernel, "bound": "mfma", "achieved": ach, "peak": peak,
                "unit": "TFLOP/s", "frac": ach / peak, "traffic": traffic,
                "algorithmic_per_launch": flops}
    if stage in ("adjoint", "descriptor"):
        if stage == "adjoint":
            ops = OPS_BWD_RAD_PAIR * res["rad_pairs"] + OPS_BWD_TRIPLET * res["triplets"]
            byts = n * (4 * D + 16) + 24 * n
        else:
            ops = OPS_FWD_RAD_PAIR * res["rad_pairs"] + OPS_FWD_TRIPLET * res["triplets"]
            byts = n * (16 + 4 * D)
        ach = ops / t / 1e12
        return {"kernel": kernel, "bound": "alu",
                "achieved": ach, "peak": PEAK_VALU_TOPS, "unit": "TOP/s", "frac": ach / PEAK_VALU_TOPS,
                "traffic": traffic, "algorithmic_per_launch": ops, "hbm_GBs": byts / t / 1e9}
    if stage in ("mm", "mm_adjoint"):   # all (NNP atom, MM charge) pairs are tested
        ops = (OPS_MM_FWD_PAIR if stage == "mm" else OPS_MM_BWD_PAIR) * n * res["n_mm"]
        ach = ops / t / 1e12
        return {"kernel": kernel, "bound": "alu", "achieved": ach, "peak": PEAK_VALU_TOPS, "unit": "TOP/s",
                "frac": ach / PEAK_VALU_TOPS, "traffic": traffic, "algorithmic_per_launch": ops}
    # memory-bound stages
    byts = {"neighbours": n * 16 + 4 * res["rad_pairs"] + 8 * res["rad_pairs"],
            "gather": 12 * res["rad_pairs"] + 24 * n + 48 * n,
            "cells": 16 * n + 16 * n,
            "energy": 8 * (n // 16)}.get(stage, 16 * n)
    ach = byts / t / 1e9
    return {"kernel": kernel or stage, "bound": "hbm", "achieved": ach, "peak": PEAK_HBM_GBS, "unit": "GB/s",
            "frac": ach / PEAK_HBM_GBS, "traffic": traffic, "algorithmic_per_launch": byts}


def main(argv=None):
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--workload", default="c5a", choices=sorted(WORKLOADS))
    ap.add_argument("--form", default="fp32", choices=["fp32", "bf16"], help="form reported as `value`")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle (no RMSE, no cpu_baseline)")
    ap.add_argument("--cpu-reps", type=int, default=3)
    ap.add_argument("--no-autotune", action="store_true", help="use the built-in kernel variant choices")
    ap.add_argument("--nve", type=int, default=1000,
                    help="velocity-Verlet NVE steps of 0.5 fs on the 12,288-atom box at 300 K (with a companion "
                         "run of twice as many 0.25 fs steps); 0 skips the check")
    ap.add_argument("--summarize-profiles", metavar="DIR",
                    help="write DIR/profiles/ summaries for --workload from rocprofv3 output under DIR, then exit")
    ap.add_argument("--calib-copy", action="store_true",
                    help="only run a plain device copy of known size (HBM counter calibration)")
    args = ap.parse_args(argv)

    if args.summarize_profiles:
        summarize_profiles(args.summarize_profiles, args.workload)
        return 0
    if args.gpus != 1:
        print(f"bench.py: this build runs on one GPU only (got --gpus {args.gpus}); "
              "multi-GPU sharding is a design note, not an implemented path.", file=sys.stderr)
        return 2
    if int(os.environ.get("WORLD_SIZE", "1")) > 1:
        print("bench.py: launched with WORLD_SIZE > 1; this build runs on one GPU only.", file=sys.stderr)
        return 2

    import numpy as np
    import torch
    import synthetic as sy
    import paper_2604_21441_amd as P

    if args.calib_copy:
        nbytes = CALIB_BYTES
        a = torch.empty(nbytes // 4, dtype=torch.float32, device="cuda").fill_(1.0)
        b = torch.empty_like(a)
        for _ in range(5):
            b.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"calib_copy_bytes": nbytes, "launches": 5}))
        return 0

    torch.set_num_threads(len(os.sched_getaffinity(0)))
    cfg, inp = build_inputs(args.workload)
    w = sy.model_weights(cfg, seed=1, n_members=inp.get("n_members", 1))
    flat = sy.flat_weights(w)
    widths = list(cfg["widths"])
    n = len(inp["Z"])
    log(f"[bench] workload {args.workload}: {WORKLOADS[args.workload]['desc']} ({n} atoms)")

    forms = {}
    for prec in ("fp32", "bf16"):
        log(f"[bench] timing {prec}: {args.warmup} warmup + {args.steps} steps")
        forms[prec] = run_form(P, cfg, flat, inp, prec, args.steps, args.warmup, not args.no_autotune)
        log(f"[bench] {prec}: {forms[prec]['ms_per_step']:.4f} ms/step, "
            f"{n / forms[prec]['ms_per_step'] * 1e3:.4e} atom-steps/s")

    report_forms = {}
    ref = None
    if not args.no_cpu:
        log("[bench] oracle reference")
        ref = oracle_reference(cfg, w, inp, None)
    for prec, r in forms.items():
        entry = {"atom_steps_per_s": n / r["ms_per_step"] * 1e3, "ms_per_step": r["ms_per_step"],
                 "host_call_ms": r["host_call_ms"],
                 "profiled_ms_per_step": r["profiled_ms_per_step"], "stage_ms": r["stage_ms"],
                 "tuned_variants": r["tuned"]}
        if ref is not None:
            a = ref["atoms"]
            dF = r["F"][a] - ref["F"][a]
            entry["force_rel_rmse"] = float(np.linalg.norm(dF) / np.linalg.norm(ref["F"][a]))
            entry["force_rmse_eV_per_A"] = float(np.sqrt(np.mean(dF ** 2)))
            # worst NNP atom against the RMS NNP-atom force (MM atoms, whose forces are far
            # smaller, would make the ratio meaningless)
            nn = min(n, a.size)
            dFn, Fn = dF[:nn], ref["F"][a][:nn]
            entry["worst_atom_err_over_rms_force"] = float(
                np.linalg.norm(dFn, axis=1).max() / np.sqrt(np.mean(np.sum(Fn ** 2, axis=1))))
            if ref["E"] is not None:
                sizes = np.diff(inp["offsets"]) if inp["offsets"] is not None else np.array([n])
                entry["energy_err_per_atom_eV"] = float(np.max(np.abs(r["E"] - ref["E"]) / sizes))
            entry["rmse_over"] = ("all NNP and MM atoms" if inp.get("mm_pos") is not None else
                                  "all atoms" if a.size == n else f"{a.size} sampled atoms")
        report_forms[prec] = entry
    r32, r16 = forms["fp32"], forms["bf16"]
    report_forms["bf16"]["force_rel_rmse_vs_fp32"] = float(np.linalg.norm(r16["F"] - r32["F"]) /
                                                           np.linalg.norm(r32["F"]))
    report_forms["bf16"]["speedup_vs_fp32"] = r32["ms_per_step"] / r16["ms_per_step"]

    main_form = forms[args.form]
    dom = max(main_form["stage_ms"], key=lambda k: main_form["stage_ms"][k])
    periodic = inp["offsets"] is None
    roof = roofline(main_form, cfg, args.form, dom, args.workload, periodic)
    stage_roofs = {s: roofline(main_form, cfg, args.form, s, args.workload, periodic)
                   for s in ("descriptor", "network", "adjoint")}

    cpu = None
    if not args.no_cpu:
        log("[bench] cpu baseline (oracle on host cores)")
        cpu = cpu_baseline(cfg, w, inp, args.cpu_reps)
        log(f"[bench] cpu: {cpu['value']:.4e} atom-steps/s on {cpu['cores']} threads")

    nve = None
    if args.nve > 0:
        from paper_2604_21441_amd.md import run_nve
        c2 = WORKLOADS["c2"]
        wcfg = sy.model_config("water")
        wflat = sy.flat_weights(sy.model_weights(wcfg, seed=1))
        pos2, Z2, box2 = sy.water_box(c2["n_mol"], c2["L"], seed=0)
        masses = np.array([sy.WATER_MASS[int(z)] for z in Z2])
        v0 = sy.maxwell_boltzmann(Z2, 300.0, seed=2)
        runs = []
        for dt, steps in ((0.5, args.nve), (0.25, 2 * args.nve)):
            log(f"[bench] NVE on {c2['desc']}: {steps} steps of {dt} fs, {args.form}")
            mdl = P.NNPModel(wcfg, weights=wflat, precision=args.form)
            r = run_nve(mdl, pos2, Z2, box2, masses, v0, dt=dt, steps=steps)
            mdl.close()
            runs.append({"dt_fs": dt, "steps": steps, "drift_eV_per_atom_per_ps": r["drift_eV_per_atom_per_ps"],
                         "max_abs_dev_eV_per_atom": r["max_abs_dev_eV_per_atom"],
                         "ms_per_step": r["ms_per_step"]})
            log(f"[bench] NVE dt {dt}: drift {r['drift_eV_per_atom_per_ps']:.3e} eV/atom/ps, max |dE| "
                f"{r['max_abs_dev_eV_per_atom']:.3e} eV/atom, {r['ms_per_step']:.3f} ms/step")
        nve = {"workload": c2["desc"], "form": args.form, "T_start_K": 300.0,
               "masses_amu": {"O": 16.00, "H": 1.008}, "runs": runs,
               "max_dev_ratio_dt_over_dt_half": runs[0]["max_abs_dev_eV_per_atom"] /
               max(runs[1]["max_abs_dev_eV_per_atom"], 1e-300)}

    value = n / main_form["ms_per_step"] * 1e3
    out = {
        "metric": METRIC,
        "value": value,
        "unit": "atom-steps/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": main_form["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": args.form,
        "data": "synthetic",
        "config": {"workload": WORKLOADS[args.workload]["desc"] + f", {args.form.upper()} form",
                   "atoms": n, "form": args.form, "n_members": inp.get("n_members", 1),
                   "seeds": {"geometry": 0, "weights": 1}},
        "roofline": roof,
        "cpu_baseline": cpu,
        "forms": report_forms,
        "stage_roofline": stage_roofs,
        "nve": nve,
    }
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
