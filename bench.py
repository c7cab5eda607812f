#!/usr/bin/env python3
"""Benchmark: MHD cell-updates/s of the fused HIP path on a 256^3 periodic box.

Workload (synthetic, seeded): 256^3 periodic unit cube, gamma = 5/3, rho = 1,
p = 0.6, uniform B = (0.2, 0, 0), solenoidal Gaussian velocity with a shell
spectrum peaked at k = 4 and rms Mach 0.5; HLLD + PLM (van Leer) + E^c CT + RK2,
CFL 0.3.  A step is one full RK2 cycle (two fused stage launches and the
device-side cycle control) over the whole box; a cell-update is one cell
advanced one cycle.  Inputs are resident in HBM before timing starts.

The line reports FP64 as ``value`` (the paper's precision) and the FP32 run
under ``fp32``; each carries its own roofline for the stage kernel:
algorithmic HBM bytes per cell and cycle are 40 state words (stage 1 reads 8
and writes 8; stage 2 reads 8 + 8 and writes 8), i.e. 320 B (FP64) and 160 B
(FP32), against the 8 TB/s HBM3E peak of the MI355X.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import re
import sys
import tempfile
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# Vector-ALU lane-operations per second: 64 lanes on each of 256 x 4 SIMDs at 2.4 GHz, a
# wave instruction every 4 cycles in FP64 (measured 4.3 to 4.5 with two waves or more) and,
# in FP32, every 2.5, the least measured (independent multiply-adds; compare and select
# pairs take 3.1 to 3.5, selects and carries 4.3 to 4.5).  Packed FP32 is not used.
LANE_OPS_PER_S = {"fp64": 64 * 1024 * 2.4e9 / 4.0, "fp32": 64 * 1024 * 2.4e9 / 2.5}
# Flop ceilings of the two builds: FP64 is compiled without fused multiply-add
# (every flop is one lane-op: 39.3 TFLOP/s); FP32 contracts multiply-adds (an
# FMA is two flops: 126 TFLOP/s at most).
ALU_PEAK_TFLOPS = {"fp64": LANE_OPS_PER_S["fp64"] / 1e12, "fp32": 2 * LANE_OPS_PER_S["fp32"] / 1e12}
# Algorithmic floating-point operations (add/sub, mul, div, sqrt) per cell and
# stage of this method on this 256^3 input with HLLD, counted on the oracle by
# oracle/opcount.cpp ("method_flops": every difference, slope, face state,
# Riemann solve and update formed once; the oracle's repeated lower-face slope
# work, 131.2 per cell, is left out).
FLOPS_PER_CELL_STAGE = 1192.30
N = 256
METRIC = "MHD cell-updates/s at 256^3 (FP64 vs FP32, %HBM peak); batched p50/p99 latency"


def kernel_source_hash() -> str:
    h = hashlib.sha256()
    for f in ("mhd_device.h", "mhd_stage.inl", "mhd_brick.inl", "mhd_stage_launch.inl", "mhd_internal.h"):
        with open(os.path.join(ROOT, "paper_2304_13746_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _profile(precision: str):
    """The committed rocprofv3 counter summary of the stage kernel, or None if it
    is missing or was taken on other kernel sources."""
    path = os.path.join(ROOT, "profiles", f"stage_kernel_256_{precision}_counters.md")
    if not os.path.exists(path):
        return None
    txt = open(path).read()
    m = re.search(r"kernel source hash: ([0-9a-f]+)", txt)
    if not m or m.group(1) != kernel_source_hash():
        return None
    return txt


def counter_traffic(precision: str):
    """HBM bytes per stage launch from the counter summary (None if stale)."""
    txt = _profile(precision)
    m = re.search(r"HBM bytes per stage launch \(scaled\): ([0-9.eE+]+)", txt or "")
    return float(m.group(1)) if m else None


def valu_per_cell(precision: str):
    """VALU lane-instructions per cell and stage launch (mean of the RK2 stage-1
    and stage-2 kernels) from the counter summary (None if stale)."""
    txt = _profile(precision)
    rows = re.findall(r"^\| mode [01] \|[^|]*\|[^|]*\| ([0-9.]+) \|", txt or "", re.M)
    return sum(float(v) for v in rows) / len(rows) if len(rows) == 2 else None


def run_gpu(state, precision: str, steps: int, warmup: int, tile: int = 0, zchunk: int = 0,
            integrator: str = "rk2", emf: str = "ec", recon: str = "plm", n: int = N,
            riemann: str = "hlld", potential=None, diagnostics: bool = False):
    import torch

    from paper_2304_13746_amd.box import MHDBox

    ct, b0 = ("vecpot", potential["b0"]) if potential else ("face", (0.0, 0.0, 0.0))
    box = MHDBox(n, n, n, precision=precision, riemann=riemann, tile=tile, zchunk=zchunk,
                 integrator=integrator, emf=emf, recon=recon, ct=ct, b0=b0)
    if potential:
        state = dict(state, ax=potential["ax"], ay=potential["ay"], az=potential["az"])
    box.set_state(state)
    d0 = box.diagnostics() if diagnostics else None
    box.step(warmup)
    torch.cuda.synchronize()
    start = torch.cuda.Event(enable_timing=True)
    stop = torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    start.record(box.stream)
    box.step(steps)
    stop.record(box.stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms = start.elapsed_time(stop)
    _, t, dt, rc = box.get_state(check=False)
    out = {"ms_total": ms, "wall_s": wall, "t": t, "dt_next": dt, "rc": rc}
    if diagnostics:
        out["diagnostics"] = diag_drift(d0, box.diagnostics(), warmup + steps, t)
    box.close()
    return out


def diag_drift(d0, d1, cycles, t):
    """Conserved totals (compensated FP64 sums on the GPU) before and after the
    run: drift of mass and energy relative to their totals, of momentum and the
    mean field relative to the mass and field totals' scale, and div B."""
    bscale = max(float(np.max(np.abs(d0["bflux"]))), 1e-300)
    return {"cycles": cycles, "t": t,
            "mass_rel_drift": float(f"{(d1['mass'] - d0['mass']) / d0['mass']:.3e}"),
            "energy_rel_drift": float(f"{(d1['energy'] - d0['energy']) / d0['energy']:.3e}"),
            "momentum_drift": [float(f"{v:.3e}") for v in (d1["mom"] - d0["mom"])],
            "mean_field_rel_drift": float(f"{float(np.max(np.abs(d1['bflux'] - d0['bflux']))) / bscale:.3e}"),
            "divb_max_before": float(f"{d0['divb_max']:.3e}"),
            "divb_max_after": float(f"{d1['divb_max']:.3e}"),
            "divb_rms_after": float(f"{d1['divb_rms']:.3e}"), "status": d1["status"]}


def roofline(precision: str, launch_ms: float):
    """Roofline of the stage kernel from its measured average launch duration.
    The method's bound is HBM bandwidth: per cell a stage launch moves 20 state
    words on average (stage 1 reads 8 and writes 8, stage 2 reads 16 and writes
    8), i.e. 160 B (FP64) or 80 B (FP32) against 8 TB/s.  Beside it: the
    counter-measured traffic of the launch (copy-calibrated rocprofv3
    FETCH/WRITE), the algorithmic flop rate against the build's ALU ceiling,
    and the VALU issue floor from the counted lane-instructions."""
    word = 8 if precision == "fp64" else 4
    cells = N ** 3
    launch_s = launch_ms * 1e-3
    bytes_per_launch = 20 * word * cells
    gbs = bytes_per_launch / launch_s / 1e9
    traffic = counter_traffic(precision)
    flops = FLOPS_PER_CELL_STAGE * cells
    tflops = flops / launch_s / 1e12
    peak = ALU_PEAK_TFLOPS[precision]
    out = {"bound": "hbm", "achieved": round(gbs, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
           "frac": round(gbs / HBM_PEAK_GBS, 4),
           "traffic": None if traffic is None else round(traffic / 1e9, 4),
           "traffic_unit": "GB per stage launch (rocprofv3 FETCH_SIZE x2 + WRITE_SIZE, "
                           "copy-calibrated)",
           "traffic_ratio": None if traffic is None else round(traffic / bytes_per_launch, 3),
           "algorithmic_bytes_per_launch": bytes_per_launch,
           "launch_ms": round(launch_ms, 4),
           "alu": {"achieved": round(tflops, 2), "peak": round(peak, 1), "unit": "TFLOP/s",
                   "frac": round(tflops / peak, 4),
                   "algorithmic_flops_per_cell_stage": FLOPS_PER_CELL_STAGE,
                   "ceiling": "FP64 without fused multiply-add: 1 flop per lane-op"
                              if precision == "fp64" else "FP32 with fused multiply-add"}}
    v = valu_per_cell(precision)
    if v is not None:
        floor_ms = v * cells / LANE_OPS_PER_S[precision] * 1e3
        out["valu"] = {"lane_instructions_per_cell_stage": round(v, 1),
                       "issue_floor_ms": round(floor_ms, 4),
                       "issue_frac": round(floor_ms / launch_ms, 4)}
    return out


CPU_CYCLES = 10  # about 10-15 s of oracle work on 16 host cores
CPU_CYCLES_1T = 1  # one cycle (about 15-20 s) on one thread


def cpu_baseline(state):
    """The FP64 oracle on the host cores: CPU_CYCLES RK2 cycles of the same 256^3
    input (after its first-dt pre-pass) on all OpenMP threads, and CPU_CYCLES_1T
    cycles on one thread, reported as cell-updates/s."""
    import oracle as O

    s = O.copy_state(state)
    p = O.Params(N, N, N)
    dt0 = 0.3 / O.max_invdt(p, s)
    cores = O.num_threads()
    t0 = time.perf_counter()
    O.step(p, s, 0.0, dt0, CPU_CYCLES)
    el = time.perf_counter() - t0
    print(f"# oracle, {cores} threads: {CPU_CYCLES} cycles in {el:.1f} s", file=sys.stderr, flush=True)
    one = O.copy_state(state)
    O.set_num_threads(1)
    t0 = time.perf_counter()
    O.step(p, one, 0.0, dt0, CPU_CYCLES_1T)
    el1 = time.perf_counter() - t0
    O.set_num_threads(cores)
    del one
    print(f"# oracle, 1 thread: {CPU_CYCLES_1T} cycle in {el1:.1f} s", file=sys.stderr, flush=True)
    return {"value": round(CPU_CYCLES * N ** 3 / el, 1), "unit": "cell-updates/s",
            "cores": cores, "kind": "oracle",
            "sample": f"{CPU_CYCLES} RK2 cycles of the same 256^3 FP64 input ({el:.1f} s, OpenMP)",
            "single_thread": {"value": round(CPU_CYCLES_1T * N ** 3 / el1, 1),
                              "unit": "cell-updates/s", "cores": 1,
                              "sample": f"{CPU_CYCLES_1T} RK2 cycle of the same input ({el1:.1f} s)"},
            "error_vs_oracle": errors_vs_oracle(state, s)}


GROUPS = {"rho": ("rho",), "momentum": ("mx", "my", "mz"), "energy": ("en",),
          "field": ("bx", "by", "bz")}


def _group_errors(g, ref):
    e = {}
    for name, fs in GROUPS.items():
        den = max(float(np.max(np.abs(ref[f]))) for f in fs)
        num = max(float(np.max(np.abs(g[f] - ref[f]))) for f in fs)
        l2 = math.sqrt(sum(float(np.sum((g[f] - ref[f]) ** 2)) for f in fs) /
                       sum(float(np.sum(ref[f] ** 2)) for f in fs))
        e[name] = {"max_rel": float(f"{num / den:.3e}"), "l2_rel": float(f"{l2:.3e}")}
    return e


def errors_vs_oracle(state, ref):
    """Errors of the GPU results after CPU_CYCLES cycles against the oracle's,
    per quantity as max|gpu - oracle| / max|oracle| and as the ratio of L2
    norms.  FP64 is compared with the oracle run above (expected bit-identical).
    FP32 starts from the input rounded to FP32 and is compared with the oracle
    run from that rounded input; its last cycle is also checked stage by stage
    (each stage of the GPU against the oracle's stage applied to the GPU's own
    stage input with the GPU's step; face-field cells departing by more than
    1e-5 counted, and each matched against the other valid choices at the E^c
    upwind switches whose mass flux lies within 1e-5 of the largest one of
    zero, oracle.fp32_check.ec_tie_check)."""
    import oracle as O
    from oracle.fp32_check import ec_tie_check
    from paper_2304_13746_amd import inputs as I
    from paper_2304_13746_amd.box import MHDBox

    out = {}
    box = MHDBox(N, N, N, precision="fp64")
    box.set_state(state)
    box.step(CPU_CYCLES)
    g, _, _, _ = box.get_state_numpy()
    box.close()
    e = _group_errors(g, ref)
    e["bit_identical"] = all(np.array_equal(g[f], ref[f]) for f in ref)
    out["fp64"] = e
    del g
    s32 = I.to_float32_exact(state)
    p = O.Params(N, N, N)
    box = MHDBox(N, N, N, precision="fp32")
    box.set_state(s32)
    box.step(CPU_CYCLES - 1)
    x0, _, dt, _ = box.get_state_numpy()
    box.step(1)
    x1 = box.get_stage_output(1)
    g, _, _, _ = box.get_state_numpy()
    box.close()
    ref32 = O.copy_state(s32)
    O.step(p, ref32, 0.0, 0.0, CPU_CYCLES)
    e = _group_errors(g, ref32)
    e["input"] = "rounded to FP32; oracle run from the rounded input"
    del ref32
    stages = []
    for xin, y, w, w0 in ((x0, x1, 1.0, 0.0), (x1, g, 0.5, 0.5)):
        pe = O.Params(N, N, N, integrator=O.EULER)
        want = O.copy_state(xin)
        O.step(pe, want, 0.0, dt, 1)
        if w0:
            want = {f: w * want[f] + w0 * x0[f] for f in O.FIELDS}
        st = {f: float(np.max(np.abs(y[f] - want[f]) / np.abs(want[f]))) for f in ("rho", "en")}
        ms = max(float(np.max(np.abs(want[f]))) for f in ("mx", "my", "mz"))
        st["momentum"] = max(float(np.max(np.abs(y[f] - want[f]))) for f in ("mx", "my", "mz")) / ms
        bs = max(float(np.max(np.abs(want[f]))) for f in ("bx", "by", "bz"))
        st["field"] = max(float(np.max(np.abs(y[f] - want[f]))) for f in ("bx", "by", "bz")) / bs
        # field departures above 1e-5 matched by another valid E^c choice at
        # the switches near ties around them (the remaining error is what is
        # left after the best such choice)
        t = ec_tie_check(p, xin, dt, y, w, w0, x0, want=want)
        st["field_cells_above_1e-5"] = t["b_bad"]
        st["field_cells_unexplained"] = t["b_unexplained"]
        st["field_after_tie_choices"] = t["b_residual"]
        stages.append({k: v if isinstance(v, int) else float(f"{v:.3e}") for k, v in st.items()})
    e["last_cycle_stagewise"] = {"stage1": stages[0], "stage2": stages[1],
                                 "norms": "rho, en element-wise relative; momentum, field "
                                          "max-abs over the largest value"}
    out["fp32"] = e
    return out


def batched_c3(nbox: int = 64, steps: int = 20):
    """64 uneven periodic boxes (edges log-uniform in [16, 128], multiples of 8,
    own seeded turbulence and uniform B), FP32, 20 RK2 cycles each: one captured
    HIP graph of batched stage launches, against the same boxes advanced one
    after another with single-box launches."""
    import torch

    from paper_2304_13746_amd import inputs as I
    from paper_2304_13746_amd.autotune import TILE_NAMES, Tuner
    from paper_2304_13746_amd.batch import BoxBatch
    from paper_2304_13746_amd.box import MHDBox

    spec = I.batch_boxes(nbox, seed=2304)
    cells = sum(int(np.prod(b["dims"])) for b in spec)
    stream = torch.cuda.Stream()
    boxes = [MHDBox(*b["dims"], *b["l"], precision="fp32", stream=stream) for b in spec]
    for bx, b in zip(boxes, spec):
        bx.set_state(b["state"])
    batch = BoxBatch(boxes)
    batch.step(1)  # warm the kernels
    # launch shapes for the batch (a common tile and cap, refined per box-shape
    # class), timed now (not from a cache)
    tuner = Tuner(os.path.join(tempfile.gettempdir(), f"mhd_tune_{os.getpid()}.json"))
    choice = batch.tune(tuner, force=True)
    graph = batch.capture(steps)
    torch.cuda.synchronize()
    ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    graph.replay()
    ev1.record(stream)
    torch.cuda.synchronize()
    ms_batch = ev0.elapsed_time(ev1)
    rcs = [bx.get_state(check=False)[3] for bx in boxes]
    # sequential reference: each box alone with its default launch shape
    for bx, b in zip(boxes, spec):
        bx.set_launch(0, 0)
        bx.set_state(b["state"])
    torch.cuda.synchronize()
    ev0.record(stream)
    done = []
    for bx in boxes:
        bx.step(steps)
        e = torch.cuda.Event(enable_timing=True)
        e.record(stream)
        done.append(e)
    ev1.record(stream)
    torch.cuda.synchronize()
    ms_seq = ev0.elapsed_time(ev1)
    lat_seq = sorted(ev0.elapsed_time(e) for e in done)
    for bx in boxes:
        bx.close()
    return {"workload": f"{nbox} uneven periodic boxes, edges 16-128 (log-uniform, multiples of 8), "
                        f"FP32, {steps} RK2 cycles each, one captured HIP graph",
            "cells": cells, "value": cells * steps / (ms_batch * 1e-3), "unit": "cell-updates/s",
            "ms_batch": round(ms_batch, 3), "ms_sequential": round(ms_seq, 3),
            "speedup_vs_sequential": round(ms_seq / ms_batch, 3),
            "latency_ms_batched": {"p50": round(ms_batch, 3), "p99": round(ms_batch, 3),
                                   "note": "each stage launch advances every box, so every box "
                                           "completes with the graph's last launch; per-request "
                                           "latency spread is the served rows'"},
            "latency_ms_sequential": {"p50": round(lat_seq[len(lat_seq) // 2], 3),
                                      "p99": round(lat_seq[int(0.99 * (len(lat_seq) - 1))], 3)},
            "status_ok": all(rc == 0 for rc in rcs),
            "launch_shape": {"tile": TILE_NAMES.get(choice["tile"], str(choice["tile"])),
                             "zchunk_cap": choice["zchunk_cap"],
                             "zchunk_by_nz": choice.get("zchunk_by_nz"),
                             "stage_ms_tuned": round(choice["best_ms"], 4),
                             "stage_ms_default": round(choice["default_ms"], 4),
                             "candidates": choice["candidates"]}}


def served_c4(nreq: int, precision: str = "fp32", rate: float = 200.0):
    """Poisson stream of box requests (mean 200 req/s), edge uniform in
    {32, 48, 64, 96, 128, 192}, 10-200 RK2 cycles, Orszag-Tang or turbulence
    initial data 50/50; admission by workspace bytes against an HBM budget."""
    import torch

    from paper_2304_13746_amd.serve import EDGES, GpuBackend, Server, poisson_requests

    free, total = torch.cuda.mem_get_info()
    budget = int(min(0.8 * free, 64 << 30))
    be = GpuBackend(precision=precision)
    reqs = poisson_requests(nreq, rate=rate, seed=2304)
    be.prepare(EDGES)  # initial fields resident on the GPU before the clock starts
    torch.cuda.synchronize()
    def progress(done, total):  # a line every 500 retired requests
        if done // 500 != progress.last:
            progress.last = done // 500
            print(f"# served {precision}: {done}/{total}", file=sys.stderr, flush=True)
    progress.last = 0
    st = Server(be, budget_bytes=budget, max_active=64, epoch_steps=10).run(reqs, progress=progress)
    s = st.summary()
    s.update({"workload": f"{nreq} Poisson requests at {rate:g}/s (the first {nreq} of the seeded "
                          f"5000-request stream), edges {list(EDGES)}, 10-200 RK2 cycles, "
                          f"OT/turbulence, one of 16 seeded translations per request, {precision.upper()}, "
                          f"HBM budget {budget / 2**30:.0f} GiB",
              "precision": precision})
    return {k: (round(v, 3) if isinstance(v, float) else v) for k, v in s.items()}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle CPU baseline")
    ap.add_argument("--no-batch", action="store_true", help="skip the 64-box batched run")
    ap.add_argument("--no-next", action="store_true",
                    help="skip the runs of the widened scheme options (RK3, LimO3, PPM, E^0, "
                         "arithmetic and UCT-HLL EMFs, vector-potential CT), of the Sedov "
                         "512^3 hydro workload and of the 512^3 turbulence box")
    ap.add_argument("--serve-requests", type=int, default=5000,
                    help="requests of the FP32 served replay (0: skip; the full stream is 5000)")
    ap.add_argument("--serve-requests-fp64", type=int, default=800,
                    help="requests of the FP64 served replay: the first ones of the same stream "
                         "(0: skip)")
    ap.add_argument("--precision", default="both", choices=["both", "fp64", "fp32"])
    ap.add_argument("--tile", type=int, default=0)
    ap.add_argument("--zchunk", type=int, default=0)
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain device copy of 2 GiB (for HBM counter scaling)")
    args = ap.parse_args()
    if args.copy_calibration:
        import torch
        src = torch.ones(1 << 28, dtype=torch.float64, device="cuda")  # 2 GiB
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_calibration_bytes_each_way": src.numel() * 8, "copies": 3}))
        return
    if args.gpus != 1:
        print(f"bench.py: the library runs one box on one GPU (asked for --gpus {args.gpus}); "
              "sharding a box over several GPUs is not implemented", file=sys.stderr)
        sys.exit(2)

    import torch

    from paper_2304_13746_amd import inputs as I

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    state = I.turbulence(N, seed=2304, kpeak=4.0, mach=0.5, rho0=1.0, p0=0.6, b0=(0.2, 0.0, 0.0))
    state.pop("_l")
    results = {}
    precs = ["fp64", "fp32"] if args.precision == "both" else [args.precision]
    for prec in precs:
        r = run_gpu(state, prec, args.steps, args.warmup, args.tile, args.zchunk)
        ms_step = r["ms_total"] / args.steps
        # two stage launches per cycle, which also do the cycle control
        results[prec] = {"value": N ** 3 / (ms_step * 1e-3), "ms_per_step": ms_step,
                         "roofline": roofline(prec, ms_step / 2.0), "rc": r["rc"]}
        rf = results[prec]["roofline"]
        print(f"# {prec}: {ms_step:.3f} ms/cycle, {results[prec]['value']:.4e} cell-updates/s, "
              f"stage kernel {rf['achieved']:.0f} GB/s algorithmic ({rf['frac']:.3f} of HBM), "
              f"{rf['alu']['achieved']:.2f} TFLOP/s, rc={r['rc']}", file=sys.stderr, flush=True)
    main_prec = precs[0]
    m = results[main_prec]
    line = {
        "metric": METRIC,
        "value": m["value"],
        "unit": "cell-updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": m["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64" if main_prec == "fp64" else "f32",
        "data": "synthetic",
        "config": {"workload": "256^3 periodic MHD turbulence (k_peak 4, Mach 0.5, B=(0.2,0,0)), "
                               "HLLD + PLM van Leer + E^c CT + RK2, CFL 0.3",
                   "cells": N ** 3, "precision": main_prec, "parallelism": "single GPU"},
        "roofline": m["roofline"],
    }
    if "fp32" in results and main_prec != "fp32":
        f = results["fp32"]
        line["fp32"] = {"value": f["value"], "ms_per_step": f["ms_per_step"], "dtype": "f32",
                        "roofline": f["roofline"]}
    if not args.no_next:
        # widened scheme options on the same input: the third-order Runge-Kutta
        # cycle (three stage launches per cycle), LimO3 and PPM reconstructions
        # with RK3, and the E^0 / arithmetic / UCT-HLL / UCT-HLLD corner EMFs
        # (RK2; the edge solves add two light launches per stage)
        nxt = {}
        k = min(args.steps, 20)
        for name, integ, emf, recon, nst in (("rk3", "rk3", "ec", "plm", 3),
                                             ("limo3_rk3", "rk3", "ec", "limo3", 3),
                                             ("ppm_rk3", "rk3", "ec", "ppm", 3),
                                             ("emf_e0", "rk2", "e0", "plm", 2),
                                             ("emf_arith", "rk2", "arith", "plm", 2),
                                             ("emf_uct_hll", "rk2", "uct_hll", "plm", 2),
                                             ("emf_uct_hlld", "rk2", "uct_hlld", "plm", 2)):
            for prec in precs:
                r = run_gpu(state, prec, k, 1, args.tile, args.zchunk, integ, emf, recon)
                ms_step = r["ms_total"] / k
                nxt[f"{name}_{prec}"] = {"value": N ** 3 / (ms_step * 1e-3), "unit": "cell-updates/s",
                                         "ms_per_step": ms_step, "stage_launch_ms": ms_step / nst,
                                         "rc": r["rc"]}
                print(f"# {name} {prec}: {ms_step:.3f} ms/cycle", file=sys.stderr, flush=True)
        # the vector-potential form of constrained transport (FP64): the same
        # input with B = (0.2, 0, 0) carried as the mean field and A = 0
        pot = I.uniform_field_potential(state["rho"].shape, (0.2, 0.0, 0.0))
        r = run_gpu(state, "fp64", k, 1, args.tile, args.zchunk, potential=pot)
        ms_step = r["ms_total"] / k
        nxt["ct_vecpot_fp64"] = {"value": N ** 3 / (ms_step * 1e-3), "unit": "cell-updates/s",
                                 "ms_per_step": ms_step, "rc": r["rc"]}
        print(f"# vector-potential CT fp64: {ms_step:.3f} ms/cycle", file=sys.stderr, flush=True)
        del pot
        # the second workload: Sedov-Taylor blast at 512^3, B = 0 (Sec. 4.1), HLLC
        # and HLL (the paper's choice), RK2, PLM
        sed = I.sedov(512)
        for riem in ("hllc", "hll"):
            for prec in precs:
                r = run_gpu(sed, prec, k, 1, args.tile, args.zchunk, "rk2", "ec", "plm",
                            n=512, riemann=riem)
                ms_step = r["ms_total"] / k
                nxt[f"sedov512_{riem}_{prec}"] = {"value": 512 ** 3 / (ms_step * 1e-3),
                                                  "unit": "cell-updates/s", "ms_per_step": ms_step,
                                                  "stage_launch_ms": ms_step / 2, "rc": r["rc"]}
                print(f"# sedov 512^3 {riem} {prec}: {ms_step:.3f} ms/cycle", file=sys.stderr,
                      flush=True)
        del sed
        # the 512^3 turbulence configuration (E(k) ~ k^-5/3 on 2 <= k <= 64, rms
        # Mach 1, B = (0.1, 0.1, 0)) with the default scheme: the per-cell rate
        # at eight times the cells of the headline box
        print("# generating the 512^3 turbulence input", file=sys.stderr, flush=True)
        c5 = I.turbulence(512, seed=2304, spectrum="kolmogorov", kmin=2.0, kmax=64.0, mach=1.0,
                          b0=(0.1, 0.1, 0.0))
        c5.pop("_l")
        for prec in precs:
            r = run_gpu(c5, prec, k, 1, args.tile, args.zchunk, n=512, diagnostics=True)
            ms_step = r["ms_total"] / k
            nxt[f"turb512_{prec}"] = {"value": 512 ** 3 / (ms_step * 1e-3),
                                      "unit": "cell-updates/s", "ms_per_step": ms_step,
                                      "stage_launch_ms": ms_step / 2, "rc": r["rc"],
                                      "diagnostics": r["diagnostics"]}
            print(f"# turbulence 512^3 {prec}: {ms_step:.3f} ms/cycle, {r['diagnostics']}",
                  file=sys.stderr, flush=True)
        del c5
        # the paper's own performance problem (Sec. 5): the 3D Orszag-Tang vortex
        # at the 256^3 per-GPU size of its node benchmarks, default scheme
        ot = I.orszag_tang_3d(N)
        for prec in precs:
            r = run_gpu(ot, prec, k, 1, args.tile, args.zchunk)
            ms_step = r["ms_total"] / k
            nxt[f"ot3d256_{prec}"] = {"value": N ** 3 / (ms_step * 1e-3), "unit": "cell-updates/s",
                                      "ms_per_step": ms_step, "stage_launch_ms": ms_step / 2,
                                      "rc": r["rc"]}
            print(f"# 3D Orszag-Tang 256^3 {prec}: {ms_step:.3f} ms/cycle", file=sys.stderr,
                  flush=True)
        del ot
        line["next_rows"] = nxt
    if not args.no_batch:
        line["batched"] = batched_c3()
        print(f"# batched: {line['batched']['value']:.4e} cell-updates/s, "
              f"{line['batched']['speedup_vs_sequential']}x vs sequential", file=sys.stderr, flush=True)
    served = [(n, p) for n, p in ((args.serve_requests, "fp32"), (args.serve_requests_fp64, "fp64"))
              if n > 0]
    if served:
        line["served"] = []
        for nreq, prec in served:
            sv = served_c4(nreq, prec)
            line["served"].append(sv)
            print(f"# served {sv['precision']}: p50 {sv['p50_ms']} ms p99 {sv['p99_ms']} ms, "
                  f"{sv['cell_updates_per_s']:.3e} cell-updates/s", file=sys.stderr, flush=True)
    if not args.no_cpu:
        line["cpu_baseline"] = cpu_baseline(state)
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
