"""Which TO runs carry the SGS change to the next step's pull as records: grids
on either side of the lines of that choice, against the FP64 oracle, and where
the choice is to apply it in place, the same bytes as with records (tune_mem
bit 2)."""
import numpy as np
import pytest

import synth
from gpu_util import fp64_bars, gpu_run, need_gpu, oracle_floor, oracle_run, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (nx, ny, nz, precision): rows of whole half tiles and not; 2-D below and
    # above 24 MB of populations; rows that are not whole lines on launches
    # that do not write through; above 64 MB in FP64
    (15, 9, 6, "fp64"), (16, 9, 6, "fp64"), (17, 8, 5, "fp64"), (48, 10, 9, "fp64"), (16, 9, 6, "fp32"),
    (592, 590, 1, "fp64"), (591, 592, 1, "fp64"), (992, 940, 1, "fp32"), (993, 940, 1, "fp32"),
    (836, 836, 1, "fp32"), (837, 836, 1, "fp32"), (97, 47, 49, "fp64"), (161, 41, 71, "fp32"), (129, 60, 58, "fp64"),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}x{c[2]}-{c[3]}")
def test_lines(case):
    """FP64: the stated bars or ten times the workload's own FP64 resolution;
    FP32: 1e-5 of the velocity and of each q* (6e-8 per power of v, amplified
    by the high-pass filters by about one on white noise)."""
    nx, ny, nz, prec = case
    lbm = need_gpu()
    qois = [("E", "B", 0), ("Z", "IMB", 0)]
    cfg = dict(lattice=int(nz > 1), nx=nx, ny=ny, nz=nz, walls_y=int(nz > 1), tau=0.55, substrate=int(nz > 1),
               cmodel=0.1 if nz > 1 else 0.0, force_kind=2 if nz > 1 else 1, force_amp=1e-6, force_k=1, drag=0.0)
    u0 = synth.noise_velocity(3 if nz > 1 else 2, (nz, ny, nx), 0.02, nx + ny)
    C, mu, S = synth.lrs_model_channel(len(qois), 7, 9)
    cargs = dict(mode="lrs", spinup=1, C=C, mu=mu, Sigma=S, seed=5)
    print(f"records {case}", flush=True)
    a, b = (gpu_run(lbm, cfg, u0, prec, qois, cargs, tune_mem=t) for t in (0, 4))
    for r in (a, b):
        r.step(4)
        assert r.sync() == 0
    assert np.array_equal(a.get_populations(), b.get_populations())
    ra, rb = a.record_arrays(), b.record_arrays()
    assert all(np.array_equal(ra[k], rb[k]) for k in ("q", "dq", "gamma", "flags"))
    o = oracle_run(cfg, u0, qois, cargs)
    o.step(4)
    ro = o.record_arrays()
    q = float(np.max(np.abs(ra["q"] - ro["q"]) / (np.max(np.abs(ro["q"]), axis=0) + 1e-300)))
    got = [rel_err(a.fields()[1], o.velocity()[1]), q]
    print("  velocity %.2e  q %.2e" % tuple(got), flush=True)
    bars = fp64_bars(oracle_floor(cfg, u0, qois, cargs, 4, ref=o))[:2] if prec == "fp64" else [1e-5, 1e-5]
    assert all(g <= v for g, v in zip(got, bars))
