#!/usr/bin/env python3
"""Benchmark: MLUPS of the TO-LES hot path on one MI355X.

Default workload: the D3Q19 turbulent-channel TO-LES, 96x48x48 fluid nodes
(x streamwise periodic, y halfway bounce-back walls, z periodic), FP32 shifted
populations with FP64 reductions, Smagorinsky substrate Cs = 0.1, 12 QoIs
({E, Z} x {B^2, B - B^2, I - B} + 6 mean-profile bands), h = 0 LRS closure
switched on at step 2500, 10000 steps.  Inputs are synthetic and seeded.
The timed steps replay captured graphs (captured before the timed region).

Prints one JSON line with the contract fields plus
  roofline:        the whole step against the HBM roofline on the fixed
                   algorithmic bytes per lattice update (232 B/LUP), with the
                   HBM bytes per step the counters measured (traffic) and
                   their ratio to the algorithmic bytes (traffic_ratio);
  dominant_kernel: the kernel phase with the largest share of the step, its
                   achieved algorithmic bandwidth per launch timed live with
                   HIP events on the stream it runs on;
  cpu_baseline:    the FP64 CPU oracle timed on a bounded sample of the same
                   workload on the host cores (and on one core);
  system_forms:    the HBM-resident 384x192x192 scale-up, the precision,
                   batched and served forms and the other comparisons.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0   # MI355X HBM3E


def workload(name):
    import synth
    if name == "channel":
        nx, ny, nz = 96, 48, 48
        cfg, u0 = synth.channel_workload(nx, ny, nz, substrate=1, cmodel=0.1, seed=6)
        nb, dmin, dmax = synth.channel_bands(ny)
        C, mu, S = synth.lrs_model_channel(12, 7, 9)
        cargs = dict(mode="lrs", spinup=2500, C=C, mu=mu, Sigma=S, seed=8, nbands=nb, dmin=dmin, dmax=dmax)
        desc = ("D3Q19 channel TO-LES 96x48x48, FP32 shifted populations, Smagorinsky Cs=0.1, "
                "12 QoIs (E/Z x {B^2,B-B^2,I-B} + 6 mean-profile bands), LRS h=0 from step 2500")
        return dict(cfg=cfg, u0=u0, qois=synth.QOIS_3D, cargs=cargs, precision="fp32", desc=desc,
                    job_steps=10000, b_alg=232)
    if name == "channel_large":
        nx, ny, nz = 384, 192, 192
        cfg, u0 = synth.channel_workload(nx, ny, nz, substrate=1, cmodel=0.1, seed=6)
        nb, dmin, dmax = synth.channel_bands(ny)
        C, mu, S = synth.lrs_model_channel(12, 7, 9)
        cargs = dict(mode="lrs", spinup=250, C=C, mu=mu, Sigma=S, seed=8, nbands=nb, dmin=dmin, dmax=dmax)
        desc = ("D3Q19 channel TO-LES 384x192x192 (HBM-resident scale-up, same physics per cell), FP32 "
                "shifted populations, Smagorinsky Cs=0.1, 12 QoIs, LRS h=0 from step 250")
        return dict(cfg=cfg, u0=u0, qois=synth.QOIS_3D, cargs=cargs, precision="fp32", desc=desc,
                    job_steps=1000, b_alg=232)
    if name == "kolmogorov":
        n = 256
        cfg, _ = synth.kolmogorov_workload(n, tau=0.51, seed=2)
        u0 = synth.turbulent_velocity_2d(n, 0.03, seed=2)
        C, mu, S = synth.lrs_model(2, 3, 4, 5)
        cargs = dict(mode="lrs", spinup=5000, C=C, mu=mu, Sigma=S, seed=12)
        desc = ("D2Q9 Kolmogorov TO-LES 256x256, FP32 shifted, tau=0.51, E_B/Z_B QoIs, LRS h=0 from step 5000, "
                "turbulent synthetic initial field")
        return dict(cfg=cfg, u0=u0, qois=synth.QOIS_2D, cargs=cargs, precision="fp32", desc=desc,
                    job_steps=20000, b_alg=128)
    if name == "fine":
        nx, ny, nz = 480, 240, 240
        cfg, u0 = synth.channel_workload(nx, ny, nz, substrate=0, cmodel=0.0, seed=13)
        desc = "D3Q19 channel plain BGK 480x240x240, FP32 shifted populations"
        return dict(cfg=cfg, u0=u0, qois=None, cargs=None, precision="fp32", desc=desc,
                    job_steps=200, b_alg=152)
    raise SystemExit(f"unknown workload {name}")


def phase_bytes(w, ms, launches):
    """Algorithmic bytes per launch of each kernel phase: one read of every
    field element a launch needs and one write of every element it produces,
    per cell."""
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    d = 2 if cfg["lattice"] == 0 else 3
    nc = 1 if d == 2 else 3
    Q = 9 if d == 2 else 19
    e = 8 if w["precision"] == "fp64" else 4
    to = w["qois"] is not None
    ne = nz = mp = 0
    if to:
        ne = sum(k == "E" for k, _, _ in w["qois"])
        nz = sum(k == "Z" for k, _, _ in w["qois"])
        mp = any(k == "MP" for k, _, _ in w["qois"])
    per_cell = {
        # populations in and out, rho and v* out, and the SGS record (2d) in
        "stream_collide": e * (2 * Q + ((1 + d) + 2 * d if to else 0)),
        "curl": 0,
        # v* in; the E sensitivities and R R w of the Z QoIs out
        "binomial": e * (d + ne * d + nz * nc),
        # E sensitivities, R R w and v*_x in; the Z sensitivities out
        "reduce": e * (ne * d + nz * nc + (1 if mp else 0) + nz * d),
        # v*, rho and every sensitivity in; the record (rho dv, 2 v* + dv) out
        "apply": e * (d + 1 + (ne + nz) * d + 2 * d),
        "solve": 0,
    }
    return {k: per_cell[k] * N for k in per_cell}


# The kernel sources a counter summary is valid for (the kernels and the
# headers they share with the launch code).
KERNEL_SOURCES = ("lbm_kernels.hip", "lbm_dev.h", "lbm_launch.h")


def _profile_kv(workload_name):
    """Key-value lines of the committed rocprofv3 counter summary of a
    workload, or None when there is none or the kernel sources have changed
    since the counters were taken."""
    import hashlib
    path = os.path.join(ROOT, "profiles", f"{workload_name}_hbm_traffic.txt")
    srcs = [os.path.join(ROOT, "paper_2609_32892_amd", "csrc", f) for f in KERNEL_SOURCES]
    if not os.path.exists(path):
        return None
    kv = {}
    for line in open(path):
        if ":" in line and not line.startswith("#"):
            k, v = line.split(":", 1)
            kv[k.strip()] = v.strip()
    sha = hashlib.sha256(b"".join(open(f, "rb").read() for f in srcs)).hexdigest()
    return kv if kv.get("kernel_source_sha256") == sha else None


def measured_traffic(workload_name, phase=None):
    """HBM bytes from the committed rocprofv3 FETCH_SIZE/WRITE_SIZE summary,
    scaled by the copy-kernel calibration: per step of the whole TO step
    (phase None) or per launch of one phase's kernel; None if not measured
    for the current sources."""
    kv = _profile_kv(workload_name)
    if kv is None:
        return None
    key = "bytes_per_step" if phase is None else f"phase_{phase}_bytes_per_launch"
    return float(kv[key]) if key in kv else None


def step_roofline(w, mlups, workload_name):
    """The whole TO step against the HBM roofline on the fixed algorithmic
    bytes per lattice update (232 B/LUP for the D3Q19 FP32 TO-LES: 152 B of
    populations, 16 B of rho and v* written, 28 B of rho, v*, dv read at the
    next pull, 12 B of v* read twice and 12 B of dv written), with the HBM
    bytes per step the counters measured and their ratio to those bytes."""
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    achieved = mlups * 1e6 * w["b_alg"] / 1e9
    traffic = measured_traffic(workload_name)
    return {"bound": "hbm", "kernel": "whole step (every kernel of one step)", "achieved": round(achieved, 1),
            "peak": HBM_PEAK_GBS, "unit": "GB/s", "frac": round(achieved / HBM_PEAK_GBS, 4),
            "b_alg_bytes_per_lup": w["b_alg"],
            "traffic": None if traffic is None else round(traffic),
            "traffic_ratio": None if traffic is None else round(traffic / (w["b_alg"] * N), 3)}


def dominant_kernel(w, ms, nl, workload_name):
    """The kernel phase with the largest share of the step: its achieved
    algorithmic bandwidth per launch from the live per-phase event timing,
    and the HBM bytes per launch the counters measured."""
    bytes_per_launch = phase_bytes(w, ms, nl)
    dom = max((k for k in ms if nl[k] > 0), key=lambda k: ms[k])
    dur_ms = ms[dom] / nl[dom]
    achieved = bytes_per_launch[dom] / (dur_ms * 1e-3) / 1e9
    traffic = measured_traffic(workload_name, dom)
    return {"kernel": dom, "achieved": round(achieved, 1), "peak": HBM_PEAK_GBS, "unit": "GB/s",
            "frac": round(achieved / HBM_PEAK_GBS, 4), "avg_launch_us": round(dur_ms * 1e3, 2),
            "bytes_per_launch": bytes_per_launch[dom], "traffic": None if traffic is None else round(traffic)}


def timed_steps(run, K):
    """K steps of a run after its graphs are captured (already, when the
    caller prepared them before its warm-up steps): host clock and HIP events
    on the run's own stream around the same region."""
    import torch
    run.prepare(K)
    run.sync()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    e0.record(run.stream)
    run.step(K)
    e1.record(run.stream)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    status = run.sync()   # the run's instability flag, read once the timed work is complete
    return dt, e0.elapsed_time(e1) * 1e-3, status


def kolmogorov_member(lbm, n, ic_seed, noise_seed, spinup, precision="fp32"):
    import synth
    cfg, _ = synth.kolmogorov_workload(n, tau=0.51, seed=ic_seed)
    u0 = synth.turbulent_velocity_2d(n, 0.03, seed=ic_seed)
    C, mu, S = synth.lrs_model(2, 3, 4, 5)
    spec = lbm.ClosureSpec(synth.QOIS_2D, mode="lrs", spinup=spinup, C=C, mu=mu, Sigma=S, seed=noise_seed)
    return lbm.make_config(precision=precision, **cfg), spec, u0


def channel_request(lbm, m, seed, spinup):
    import synth
    ny = 24 * m
    cfg, u0 = synth.channel_workload(48 * m, ny, 24 * m, substrate=1, cmodel=0.1, seed=seed)
    nb, dmin, dmax = synth.channel_bands(ny)
    C, mu, S = synth.lrs_model_channel(12, 7, 9)
    spec = lbm.ClosureSpec(synth.QOIS_3D, mode="lrs", spinup=spinup, C=C, mu=mu, Sigma=S, seed=seed,
                           nbands=nb, dmin=dmin, dmax=dmax)
    return lbm.make_config(precision="fp32", **cfg), spec, u0


def form_precision(lbm, w, steps):
    """System form (1): FP32 shifted populations vs the plain FP32 kernel vs
    FP64, same workload; error of the FP32 runs against the FP64 run."""
    import numpy as np
    import torch
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    out, vel = {}, {}
    for prec in ("fp64", "fp32", "fp32_plain"):
        spec = lbm.ClosureSpec(w["qois"], **w["cargs"])
        r = lbm.Run(lbm.make_config(precision=prec, **cfg), spec)
        r.init_velocity(w["u0"])
        r.step(20)
        r.sync()
        t = time.perf_counter()
        r.step(steps)
        r.sync()
        dt = time.perf_counter() - t
        vel[prec] = r.fields()[1]
        out[prec] = {"mlups": round(N * (steps + 20) / 1e6 / dt * steps / (steps + 20), 1)}
        r.close()
    for prec in ("fp32", "fp32_plain"):
        out[prec]["max_rel_velocity_err_vs_fp64"] = float(
            np.max(np.abs(vel[prec] - vel["fp64"])) / np.max(np.abs(vel["fp64"])))
    out["steps"] = steps + 20
    return out


def form_history(lbm, w, steps, h=500):
    """The paper's history-h LRS (h = 500: 12000 history entries for 12
    QoIs) on the headline workload, against the same stretch with an h = 0
    model: MLUPS over corrected steps only."""
    import numpy as np
    import synth
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    nq = len(w["qois"])
    # scale: |q*| of the uncorrected flow after a short spin-up
    r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg),
                lbm.ClosureSpec(w["qois"], **dict(w["cargs"], mode="off")))
    r.init_velocity(w["u0"])
    r.step(h)
    r.sync()
    s = np.abs(r.record_arrays()["q"][-1])
    s[s == 0] = 1.0
    r.close()
    out = {"h": h, "history_entries": 2 * h * nq}
    for hh in (h, 0):
        C, mu, S = synth.lrs_history_model(hh, nq, 7, 9, 10)
        spec = lbm.ClosureSpec(w["qois"], **dict(w["cargs"], C=C, mu=mu, Sigma=S, h=hh, scale=s, spinup=h + 5))
        r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg), spec)
        r.init_velocity(w["u0"])
        r.step(h + 20)
        r.sync()
        t = time.perf_counter()
        r.step(steps)
        try:
            r.sync()
        except lbm.LbmError as e:
            out["error" if hh else "error_h0"] = str(e)
        dt = time.perf_counter() - t
        out["mlups" if hh else "mlups_h0"] = round(N * steps / dt / 1e6, 1)
        r.close()
    out["steps"] = steps
    out["ratio_to_h0"] = round(out["mlups"] / out["mlups_h0"], 3)
    return out


def form_kernel_filters(lbm, w, steps):
    """The paper's own 3-D QoI set (Sec. 7: {E, Z} x {G_3, L_3, L_1} plus the
    six mean-profile bands), FP32, LRS h = 0, on the headline channel (MLUPS
    and the per-phase split; the filter phase is the kernel-filter pass
    program) and on the paper's LF grid 295 x 47 x 98 (its 295 x 49 x 98 with
    the two solid rows not stored), where the paper measures its LF TO-LRS."""
    import synth
    out = {"qois": "E,Z x G3,L3,L1 + 6 mean-profile bands", "steps": steps}
    for name, (nx, ny, nz) in (("headline", (96, 48, 48)), ("paper_lf_grid", (295, 47, 98))):
        cfg, u0 = synth.channel_workload(nx, ny, nz, substrate=1, cmodel=0.1, seed=6)
        nb, dmin, dmax = synth.channel_bands(ny)
        qois = [(k, f, 0) for f in ("G3", "L3", "L1") for k in ("E", "Z")] + [("MP", "I", j) for j in range(nb)]
        spec = lbm.ClosureSpec(qois, **dict(w["cargs"], nbands=nb, dmin=dmin, dmax=dmax))
        r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg), spec)
        r.init_velocity(u0)
        r.step(20)
        r.sync()
        t = time.perf_counter()
        r.step(steps)
        r.sync()
        dt = time.perf_counter() - t
        ms, nl = r.profile_phases(20)
        r.close()
        out[name] = {"grid": [nx, ny, nz], "mlups": round(nx * ny * nz * steps / dt / 1e6, 1),
                     "ms_per_step": {k: round(v, 4) for k, v in ms.items()},
                     "launches_per_step": {k: int(v) for k, v in nl.items()}}
    return out


def form_fourier(lbm, steps):
    """The sharp Fourier band QoIs of the paper's earlier formulation (App. E
    variant; eq. scale-aware-energy-fourier) on the 256 x 256 Kolmogorov
    TO-LES: {E, Z} x {R_[0,12], R_[13,32], R_[33,128]} through hipFFT (eager
    launches), against the same run with the binomial pair {E_B, Z_B}."""
    import synth
    w = workload("kolmogorov")
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    out = {"grid": [cfg["nx"], cfg["ny"]], "steps": steps}
    for name, qois in (("fourier_bands", [(k, f, 0) for f in ("F0-12", "F13-32", "F33-128") for k in ("E", "Z")]),
                       ("binomial_pair", synth.QOIS_2D)):
        C, mu, S = synth.lrs_history_model(0, len(qois), 3, 4, 5, noise=1e-4)
        spec = lbm.ClosureSpec(qois, mode="lrs", spinup=steps // 2, C=C, mu=mu, Sigma=S, seed=12)
        r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg), spec)
        r.init_velocity(w["u0"])
        r.step(20)
        r.sync()
        t = time.perf_counter()
        r.step(steps)
        try:
            r.sync()
        except lbm.LbmError as e:
            out[name + "_error"] = str(e)
        dt = time.perf_counter() - t
        out[name + "_mlups"] = round(N * steps / dt / 1e6, 1)
        r.close()
    return out


def form_wale(lbm, steps):
    """The headline channel TO-LES (96 x 48 x 48, FP32, 12 QoIs, LRS) on the
    WALE substrate at C_w = 2.20, the paper's stable WALE setting (Sec. 7),
    next to the Smagorinsky headline."""
    import synth
    w = workload("channel")
    cfg = dict(w["cfg"], substrate=2, cmodel=2.2)
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    spec = lbm.ClosureSpec(w["qois"], **dict(w["cargs"], spinup=steps // 4))
    r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg), spec)
    r.init_velocity(w["u0"])
    r.step(20)
    r.sync()
    t = time.perf_counter()
    r.step(steps)
    status = 0
    try:
        r.sync()
    except lbm.LbmError as e:
        status = e.code
    dt = time.perf_counter() - t
    out = {"grid": [cfg["nx"], cfg["ny"], cfg["nz"]], "c_w": 2.2, "steps": steps, "status": status,
           "mlups": round(N * steps / dt / 1e6, 1)}
    r.close()
    return out


def form_paper_table(lbm, steps):
    """The rows of the paper's 3-D timing table (tab:timing-3d, H100, FP32)
    that run on the LF channel grid, here on 295 x 47 x 98 fluid rows (the
    paper's 295 x 49 x 98 with its two solid rows not stored): no model,
    Smagorinsky, WALE, TO tracking and TO-LRS with the paper's 12 QoIs
    ({E, Z} x {G3, L3, L1} + 6 bands).  ms per step, MLUPS over fluid nodes,
    and the paper's ms per step beside them."""
    import numpy as np
    import synth
    nx, ny, nz = 295, 47, 98
    N = nx * ny * nz
    nb, dmin, dmax = synth.channel_bands(ny)
    qois = [(k, f, 0) for f in ("G3", "L3", "L1") for k in ("E", "Z")] + [("MP", "I", j) for j in range(nb)]
    C, mu, S = synth.lrs_model_channel(12, 7, 9)
    paper_ms = {"no_model": 0.81, "smagorinsky": 1.07, "wale": 1.04, "to_tracking": 11.45, "to_lrs": 11.38}
    out = {"grid": [nx, ny, nz], "steps": steps}
    for name in ("no_model", "smagorinsky", "wale", "to_tracking", "to_lrs"):
        sub, cm = {"smagorinsky": (1, 0.1), "wale": (2, 2.2)}.get(name, (0, 0.0))
        if name.startswith("to_"):
            sub, cm = 1, 0.1
        cfg, u0 = synth.channel_workload(nx, ny, nz, substrate=sub, cmodel=cm, seed=6)
        spec = None
        if name == "to_lrs":
            spec = lbm.ClosureSpec(qois, mode="lrs", spinup=10, C=C, mu=mu, Sigma=S, seed=8, nbands=nb,
                                   dmin=dmin, dmax=dmax)
        elif name == "to_tracking":
            # the reference: the uncorrected run's own QoIs, scaled by 1.01
            ref = lbm.Run(lbm.make_config(precision="fp32", **cfg),
                          lbm.ClosureSpec(qois, mode="off", nbands=nb, dmin=dmin, dmax=dmax))
            ref.init_velocity(u0)
            ref.step(20 + steps)
            ref.sync()
            qref = 1.01 * ref.record_arrays()["q"]
            ref.close()
            spec = lbm.ClosureSpec(qois, mode="track", spinup=10, qref=qref, nbands=nb, dmin=dmin, dmax=dmax)
        r = lbm.Run(lbm.make_config(precision="fp32", **cfg), spec)
        r.init_velocity(u0)
        r.step(20)
        r.sync()
        t = time.perf_counter()
        r.step(steps)
        try:
            r.sync()
        except lbm.LbmError as e:
            out[name + "_error"] = str(e)
        dt = time.perf_counter() - t
        r.close()
        out[name] = {"ms_per_step": round(dt / steps * 1e3, 4), "mlups": round(N * steps / dt / 1e6, 1),
                     "paper_ms_per_step": paper_ms[name]}
    return out


def form_batched(lbm, nmem, steps):
    """System form (2): an ensemble of Kolmogorov TO-LES members on uneven
    grids advanced as one batch (one launch per kernel phase for all members,
    replayed from a hipGraph) vs the same members stepped one after another.
    Each distinct member shape is autotuned once (lbm_autotune, with a tuning
    cache in a temporary file); both sides use the tuned launch shapes."""
    import os
    import tempfile
    import numpy as np
    import synth
    mem = synth.ensemble_members(nmem)
    cells = sum(m["n"] ** 2 for m in mem)
    cache = os.path.join(tempfile.mkdtemp(prefix="lbm_tune_"), "tune.txt")
    tunings = {}
    t = time.perf_counter()
    for n in sorted({m["n"] for m in mem}):
        m = next(x for x in mem if x["n"] == n)
        cfg, spec, _ = kolmogorov_member(lbm, n, m["ic_seed"], m["noise_seed"], spinup=steps // 4)
        tunings[n] = lbm.autotune(cfg, spec, steps=100, cache=cache)
    tune_s = time.perf_counter() - t
    runs_b, runs_s = [], []
    for m in mem:
        for lst in (runs_b, runs_s):
            cfg, spec, u0 = kolmogorov_member(lbm, m["n"], m["ic_seed"], m["noise_seed"], spinup=steps // 4)
            for k in ("tune_zc", "tune_cpt", "tune_btx"):
                setattr(cfg, k, tunings[m["n"]][k])
            r = lbm.Run(cfg, spec)
            r.init_velocity(u0)
            lst.append(r)
    batch = lbm.Batch(runs_b)
    batch.step(16)
    batch.sync()
    t = time.perf_counter()
    batch.step(steps)
    batch.sync()
    tb = time.perf_counter() - t
    for r in runs_s:
        r.step(16)
        r.sync()
    t = time.perf_counter()
    for r in runs_s:
        r.step(steps)
        r.sync()
    ts = time.perf_counter() - t
    same = all(np.array_equal(runs_b[k].get_populations(), runs_s[k].get_populations()) for k in (0, nmem - 1))
    res = {"members": nmem, "cells": cells, "steps": steps,
           "batched_mlups": round(cells * steps / tb / 1e6, 1),
           "sequential_mlups": round(cells * steps / ts / 1e6, 1),
           "speedup": round(ts / tb, 3), "bitwise_equal_to_solo": bool(same),
           "autotune": {"shapes": len(tunings), "seconds": round(tune_s, 2),
                        "timed_candidates": sum(v["candidates"] for v in tunings.values()),
                        "cpt": {str(n): v["tune_cpt"] for n, v in sorted(tunings.items())}}}
    batch.close()
    for r in runs_b + runs_s:
        r.close()
    return res


def form_served(lbm, nreq, rate, steps, budget=0, sequential=True, sample_every=25):
    """System form (5): continuous-batching server on a Poisson trace of mixed
    2-D/3-D TO-LES requests (latency = completion - arrival), and the same
    requests run one after another, each alone, as the sequential baseline;
    every sample_every-th request's final state is compared bitwise between
    the two."""
    import hashlib
    import numpy as np
    import synth
    trace = synth.serve_trace(nreq, rate, steps=steps)
    reqs = []
    for q in trace:
        if q["kind"] == "2d":
            cfg, spec, u0 = kolmogorov_member(lbm, q["n"], q["seed"], q["seed"], spinup=steps // 4)
        else:
            cfg, spec, u0 = channel_request(lbm, q["m"], q["seed"], spinup=steps // 4)
        reqs.append((cfg, spec, u0, q["t"]))
    sample = set(range(0, len(reqs), sample_every)) if sequential else set()
    srv = lbm.Server(hbm_budget=budget)
    t0 = srv.clock() + 0.05
    # submit as arrivals happen; advance the server in between
    results, k, ids = [], 0, {}
    while k < len(reqs) or srv.pending() > 0:
        now = srv.clock()
        while k < len(reqs) and t0 + reqs[k][3] <= now:
            cfg, spec, u0, ta = reqs[k]
            ids[k] = srv.submit(cfg, spec, u0, steps, t0 + ta, keep_state=k in sample)
            k += 1
        if srv.pending() > 0:
            srv.advance(srv.clock(), 64)
            results += srv.poll()
        else:
            time.sleep(0.0005)
    lat = np.array([r.t_done - r.t_arrival for r in results])
    span = max(r.t_done for r in results) - t0
    st = srv.stats()
    ok = sum(1 for r in results if r.status == 0)
    images = {j: srv.take_state(ids[j]) for j in sample}
    srv.close()
    out = {"requests": len(results), "completed_ok": ok, "rate_per_s": rate, "steps": steps,
           "p50_latency_s": round(float(np.percentile(lat, 50)), 3),
           "p99_latency_s": round(float(np.percentile(lat, 99)), 3),
           "aggregate_mlups": round(st["lups"] / span / 1e6, 1),
           "busy_mlups": round(st["lups"] / st["busy_s"] / 1e6, 1),
           "span_s": round(span, 2), "budget_gb": round(st["budget"] / 1e9, 2)}
    if sequential:
        lups, same = 0.0, True
        t = time.perf_counter()
        for j, (cfg, spec, u0, _) in enumerate(reqs):
            r = lbm.Run(cfg, spec)
            r.init_velocity(u0)
            r.step(steps)
            r.sync()
            lups += r.N * steps
            if j in sample:
                same = same and hashlib.sha256(r.get_state()).digest() == hashlib.sha256(images[j]).digest()
            r.close()
        ts = time.perf_counter() - t
        out["sequential_mlups"] = round(lups / ts / 1e6, 1)
        out["sequential_s"] = round(ts, 2)
        out["served_over_sequential"] = round(out["aggregate_mlups"] / out["sequential_mlups"], 3)
        out["bitwise_equal_to_solo"] = {"sampled": len(sample), "equal": bool(same)}
    return out


def form_fine(lbm, steps):
    w = workload("fine")
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    r = lbm.Run(lbm.make_config(precision="fp32", **cfg))
    r.init_velocity(w["u0"])
    r.step(10)
    r.sync()
    t = time.perf_counter()
    r.step(steps)
    r.sync()
    dt = time.perf_counter() - t
    ms, _ = r.profile_phases(20)
    r.close()
    mlups = N * steps / dt / 1e6
    return {"grid": [cfg["nx"], cfg["ny"], cfg["nz"]], "steps": steps, "mlups": round(mlups, 1),
            "hbm_frac_152B": round(mlups * 1e6 * 152 / (HBM_PEAK_GBS * 1e9), 4),
            "stream_collide_gbs": round(152 * N / (ms["stream_collide"] * 1e-3) / 1e9, 1)}


def form_hf_lf(lbm, hf_steps, m=5):
    """The paper's HF -> LF channel pipeline at its grid sizes (Sec. 7.1):
    plain BGK on the 1475 x 235 x 490 HF grid (the paper's 1475 x 237 x 490
    with its two solid rows not stored), and after every m = 5 HF steps the
    12 QoIs of the wall-anchored stride-5 projection onto the 295 x 47 x 98 LF
    grid (lbm_project_qoi), the reference of LF tracking.  Reports the HF
    throughput and the added cost per reference evaluation (the paper: under
    1%, 0.8 ms on a 91 ms HF step)."""
    import numpy as np
    import synth
    nx, ny, nz = 1475, 235, 490
    cfg, _ = synth.channel_workload(8, ny, 8, substrate=0, cmodel=0.0, seed=13)
    cfg.update(nx=nx, nz=nz)
    N = nx * ny * nz
    hf = lbm.Run(lbm.make_config(precision="fp32", **cfg))
    hf.init_velocity(synth.channel_velocity(nx, ny, nz, seed=13))
    lcfg, _ = synth.channel_workload(nx // m, ny // m, nz // m, substrate=1, cmodel=0.1, seed=13)
    nb, dmin, dmax = synth.channel_bands(ny // m)
    bands = [("MP", "I", j) for j in range(nb)]
    hf.step(10)
    hf.sync()
    t = time.perf_counter()
    hf.step(hf_steps)
    hf.sync()
    t_plain = time.perf_counter() - t
    out = {"hf_grid": [nx, ny, nz], "lf_grid": [nx // m, ny // m, nz // m], "hf_steps": hf_steps,
           "hf_mlups": round(N * hf_steps / t_plain / 1e6, 1),
           "hf_ms_per_step": round(t_plain / hf_steps * 1e3, 3)}
    # the reference QoIs: the binomial set of the headline, and the paper's
    # own kernel-filter set {E, Z} x {G3, L3, L1} with the same six bands
    for name, qois in (("binomial_qois", synth.QOIS_3D),
                       ("paper_kernel_qois", [(k, f, 0) for f in ("G3", "L3", "L1") for k in ("E", "Z")] + bands)):
        probe = lbm.Run(lbm.make_config(precision="fp32", **lcfg),
                        lbm.ClosureSpec(qois, mode="off", nbands=nb, dmin=dmin, dmax=dmax))
        probe.init_velocity(np.zeros((3, probe.N)))
        probe.project_qoi_from(hf, m)
        hf.sync()
        t = time.perf_counter()
        for _ in range(hf_steps // m):
            hf.step(m)
            probe.project_qoi_from(hf, m)
        hf.sync()
        t_ref = time.perf_counter() - t
        q = probe.record_arrays()["q"]
        out[name] = {"reference_ms_per_lf_step": round((t_ref - t_plain) / (hf_steps // m) * 1e3, 3),
                     "reference_overhead_frac": round((t_ref - t_plain) / t_plain, 4),
                     "qoi_records": int(q.shape[0]), "qoi_finite": bool(np.all(np.isfinite(q)))}
        probe.close()
    hf.close()
    return out


def form_hf_lf_kolmogorov(lbm, hf_steps, m=5):
    """The HF -> LF pipeline of the periodic Kolmogorov case (Sec. 3, 6):
    plain BGK on a 1280^2 HF grid and, after every m = 5 HF steps, the
    {E_B, Z_B} QoIs of the bicubic projection onto the 256^2 LF grid
    (lbm_project_qoi_kind, LBM_PROJ_BICUBIC).  Reports the HF throughput and
    the added cost per reference evaluation."""
    import numpy as np
    import synth
    n = 1280
    cfg, _ = synth.kolmogorov_workload(n, tau=0.55, amp=2e-5, seed=14)
    N = n * n
    hf = lbm.Run(lbm.make_config(precision="fp32", **cfg))
    hf.init_velocity(synth.turbulent_velocity_2d(n, 0.02, seed=14))
    lcfg, _ = synth.kolmogorov_workload(n // m, tau=0.5 + 0.05 / m, amp=2e-5 * m, seed=14)
    hf.step(10)
    hf.sync()
    t = time.perf_counter()
    hf.step(hf_steps)
    hf.sync()
    t_plain = time.perf_counter() - t
    probe = lbm.Run(lbm.make_config(precision="fp32", **lcfg), lbm.ClosureSpec(synth.QOIS_2D, mode="off"))
    probe.init_velocity(np.zeros((2, probe.N)))
    probe.project_qoi_from(hf, m, "bicubic")
    hf.sync()
    t = time.perf_counter()
    for _ in range(hf_steps // m):
        hf.step(m)
        probe.project_qoi_from(hf, m, "bicubic")
    hf.sync()
    t_ref = time.perf_counter() - t
    q = probe.record_arrays()["q"]
    out = {"hf_grid": [n, n], "lf_grid": [n // m, n // m], "hf_steps": hf_steps,
           "hf_mlups": round(N * hf_steps / t_plain / 1e6, 1),
           "reference_ms_per_lf_step": round((t_ref - t_plain) / (hf_steps // m) * 1e3, 3),
           "reference_overhead_frac": round((t_ref - t_plain) / t_plain, 4),
           "qoi_records": int(q.shape[0]), "qoi_finite": bool(np.all(np.isfinite(q)))}
    probe.close()
    hf.close()
    return out


def form_large(lbm, steps):
    """The HBM-resident scale-up of the headline (384 x 192 x 192, the same
    physics per cell; about 2.5 GB of state): MLUPS over a timed stretch
    after warm-up, the whole step against the HBM roofline on 232 B/LUP with
    the counters' HBM bytes per step, and the dominant kernel."""
    w = workload("channel_large")
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    spec = lbm.ClosureSpec(w["qois"], **dict(w["cargs"], spinup=10))
    r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg), spec)
    r.init_velocity(w["u0"])
    r.prepare(steps)
    r.step(20)
    r.sync()
    dt, dt_ev, status = timed_steps(r, steps)
    ms, nl = r.profile_phases(20)
    r.close()
    mlups = N * steps / dt / 1e6
    return {"grid": [cfg["nx"], cfg["ny"], cfg["nz"]], "cells": N, "steps": steps, "status": status,
            "mlups": round(mlups, 1), "ms_per_step": round(dt / steps * 1e3, 4),
            "ms_per_step_events": round(dt_ev / steps * 1e3, 4),
            "roofline": step_roofline(w, mlups, "channel_large"),
            "dominant_kernel": dominant_kernel(w, ms, nl, "channel_large"),
            "phases": {k: {"ms_per_step": round(ms[k], 4), "launches": nl[k]} for k in ms}}


def cpu_baseline(w, seconds):
    """The FP64 oracle on the host's cores on a bounded sample of the same
    workload (its first steps: same grid, closure and inputs), once on every
    core OpenMP uses and once on one core, scaled to MLUPS."""
    import oracle
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]
    model = "unknown"
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                model = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    out = {}
    for label, nthreads in (("all", oracle.threads()), ("one", 1)):
        cores = oracle.set_threads(nthreads)
        o = oracle.Oracle(**cfg)
        o.init(w["u0"])
        if w["qois"] is not None:
            o.set_closure(oracle.make_closure(w["qois"], **w["cargs"]))
        t = time.perf_counter()
        o.step(1)
        one = time.perf_counter() - t
        n = max(1, min(2000, int(seconds / max(one, 1e-6))))
        t = time.perf_counter()
        o.step(n)
        tc = time.perf_counter() - t
        out[label] = dict(value=round(N * n / tc / 1e6, 4), cores=cores, steps=n, seconds=round(tc, 1))
        del o
    oracle.set_threads(out["all"]["cores"])
    return {"value": out["all"]["value"], "unit": "MLUPS", "cores": out["all"]["cores"], "kind": "oracle",
            "sample": f"steps 2..{out['all']['steps'] + 1} of the same workload (same grid, closure, inputs), "
                      f"{out['all']['seconds']} s on {out['all']['cores']} threads",
            "one_core": {"value": out["one"]["value"], "unit": "MLUPS", "cores": 1,
                         "sample": f"steps 2..{out['one']['steps'] + 1}, {out['one']['seconds']} s"},
            "cpu_model": model}


def main():
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=None, help="timed steps (default: the workload's job length)")
    ap.add_argument("--warmup", type=int, default=50)
    ap.add_argument("--workload", default="channel", choices=["channel", "channel_large", "kolmogorov", "fine"])
    ap.add_argument("--profile-steps", type=int, default=200)
    ap.add_argument("--cpu-seconds", type=float, default=12.0,
                    help="target length of each oracle sample (all cores, then one core)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-system-forms", action="store_true",
                    help="skip the precision / batched / served / fine-grid comparisons")
    ap.add_argument("--serve-requests", type=int, default=200)
    ap.add_argument("--ensemble-steps", type=int, default=200)
    ap.add_argument("--copy-probe", type=int, default=0, metavar="MIB",
                    help="first run a plain device copy of this many MiB (calibrates HBM byte counters)")
    args = ap.parse_args()

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py runs on one GPU only: the hot path of this build is a single-GPU kernel set "
              "(an ensemble shards by member across GPUs without communication); use --gpus 1",
              file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    from paper_2609_32892_amd import lbm

    if not torch.cuda.is_available():
        raise SystemExit("bench.py needs a GPU")
    torch.cuda.set_device(0)
    if args.copy_probe:
        a = torch.empty(args.copy_probe * (1 << 20) // 4, dtype=torch.float32, device="cuda")
        b = torch.empty_like(a)
        a.fill_(1.0)
        for _ in range(5):
            torch.mul(a, 1.0, out=b)   # plain elementwise kernel: reads and writes copy_probe MiB
        torch.cuda.synchronize()
        print(f"[bench] copy probe: 5 x {args.copy_probe} MiB elementwise copies", file=sys.stderr, flush=True)
        del a, b
    w = workload(args.workload)
    K = args.steps if args.steps is not None else w["job_steps"]
    W = args.warmup
    cfg = w["cfg"]
    N = cfg["nx"] * cfg["ny"] * cfg["nz"]

    def make_run():
        spec = lbm.ClosureSpec(w["qois"], **w["cargs"]) if w["qois"] is not None else None
        r = lbm.Run(lbm.make_config(precision=w["precision"], **cfg), spec)
        r.init_velocity(w["u0"])
        return r

    # The system forms run first: the headline's 20-odd timed steps are then
    # measured with the GPU at its working clocks (first in a fresh process
    # they read about 4% slower while the clocks ramp up).
    forms = None
    if args.workload == "channel" and not args.no_system_forms:
        forms = {}
        forms["channel_large"] = form_large(lbm, 200)
        print(f"[bench] HBM-resident TO-LES: {forms['channel_large']}", file=sys.stderr, flush=True)
        forms["precision"] = form_precision(lbm, w, 1000)
        print(f"[bench] precision forms: {forms['precision']}", file=sys.stderr, flush=True)
        forms["kernel_filters"] = form_kernel_filters(lbm, w, 1000)
        print(f"[bench] kernel filters: {forms['kernel_filters']}", file=sys.stderr, flush=True)
        forms["paper_timing_table"] = form_paper_table(lbm, 500)
        print(f"[bench] paper timing table: {forms['paper_timing_table']}", file=sys.stderr, flush=True)
        forms["fourier_bands"] = form_fourier(lbm, 1000)
        print(f"[bench] Fourier bands: {forms['fourier_bands']}", file=sys.stderr, flush=True)
        forms["history_lrs"] = form_history(lbm, w, 2000)
        print(f"[bench] history LRS: {forms['history_lrs']}", file=sys.stderr, flush=True)
        forms["batched"] = form_batched(lbm, 64, args.ensemble_steps)
        print(f"[bench] batched: {forms['batched']}", file=sys.stderr, flush=True)
        forms["served"] = form_served(lbm, args.serve_requests, 20.0, 2000)
        print(f"[bench] served: {forms['served']}", file=sys.stderr, flush=True)
        # the same trace under a 2 GB HBM budget: admission queues requests
        forms["served_2gb"] = form_served(lbm, args.serve_requests, 20.0, 2000, budget=2 << 30, sequential=False)
        print(f"[bench] served (2 GB budget): {forms['served_2gb']}", file=sys.stderr, flush=True)
        forms["wale_to_les"] = form_wale(lbm, 2000)
        print(f"[bench] WALE TO-LES: {forms['wale_to_les']}", file=sys.stderr, flush=True)
        forms["fine_grid_plain"] = form_fine(lbm, 200)
        print(f"[bench] fine grid: {forms['fine_grid_plain']}", file=sys.stderr, flush=True)
        forms["hf_to_lf"] = form_hf_lf(lbm, 200)
        print(f"[bench] HF to LF: {forms['hf_to_lf']}", file=sys.stderr, flush=True)
        forms["hf_to_lf_kolmogorov"] = form_hf_lf_kolmogorov(lbm, 500)
        print(f"[bench] HF to LF (Kolmogorov, bicubic): {forms['hf_to_lf_kolmogorov']}", file=sys.stderr, flush=True)
    run = make_run()
    run.prepare(K)      # graphs of the timed chunk first: the warm-up runs right before the timed steps
    run.step(W)
    run.sync()
    dt, dt_ev, status = timed_steps(run, K)
    mlups = N * K / dt / 1e6
    print(f"[bench] {args.workload}: {K} steps in {dt:.4f} s (events {dt_ev:.4f} s) -> {mlups:.1f} MLUPS "
          f"(status {status})", file=sys.stderr, flush=True)
    run.close()

    # live per-kernel timing (HIP events on the run's stream)
    prof = make_run()
    prof.step(W)
    ms, nl = prof.profile_phases(args.profile_steps)
    prof.close()
    phases = {k: {"ms_per_step": round(ms[k], 5), "launches": nl[k]} for k in ms}

    out = {
        "metric": "MLUPS (D3Q19 TO-LES)" if args.workload == "channel" else f"MLUPS ({args.workload})",
        "value": round(mlups, 2),
        "unit": "MLUPS",
        "n_gpus": 1,
        "steps": K,
        "warmup": W,
        "ms_per_step": round(dt / K * 1e3, 5),
        "ms_per_step_events": round(dt_ev / K * 1e3, 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "fp32" if w["precision"] != "fp64" else "f64",
        "data": "synthetic",
        "config": {"workload": w["desc"], "grid": [cfg["nx"], cfg["ny"], cfg["nz"]], "cells": N,
                   "job_steps": w["job_steps"], "parallelism": "single-gpu"},
        "roofline": step_roofline(w, mlups, args.workload),
        "dominant_kernel": dominant_kernel(w, ms, nl, args.workload),
        "phases": phases,
    }

    if forms is not None:
        out["system_forms"] = forms

    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, args.cpu_seconds)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
