"""The filter chains and the reduce of binomial closures against the FP64
oracle at the sizes where their tiles change: a tile of the chains holds
64 - 2 j cells in x (j = 2 or 4 powers) and, between walls, up to all its rows
in y (3-D: 32 in FP32, 24 in FP64; 2-D: 16), two tiles up to 2 (rows - j), else
rows - 2 j each; and closures of one kind, of either, and with more QoIs of one
kind than of the other."""
import numpy as np
import pytest

import synth
from gpu_util import fp64_bars, gpu_run, need_gpu, oracle_floor, oracle_run, rel_err

pytestmark = pytest.mark.gpu

SETS = {
    "four": [(k, f, 0) for f in ("B2", "BMID", "IMB") for k in ("E", "Z")],
    "two": [(k, f, 0) for f in ("B", "IMB") for k in ("E", "Z")],
    "energy": [("E", "B2", 0), ("E", "IMB", 0)],
    "enstrophy": [("Z", "I", 0), ("Z", "BMID", 0)],
    "uneven": [("Z", "B", 0)] + [("E", f, 0) for f in ("I", "B", "B2", "BMID", "IMB")],
    "pair": [("E", "B", 0), ("Z", "B", 0)],
    "pair4": [("Z", "BMID", 0), ("E", "B2", 0)],
    "one": [("Z", "IMB", 0)],
    "one4": [("E", "BMID", 0)],
}

CASES = [
    # (nx, ny, nz, walls, set): one cell within and past a tile's limits
    (56, 5, 3, 1, "four"), (57, 4, 5, 1, "four"), (113, 3, 4, 0, "two"), (60, 7, 3, 0, "two"), (61, 6, 3, 1, "two"),
    (5, 24, 3, 1, "four"), (6, 25, 4, 1, "four"), (4, 32, 3, 1, "two"), (5, 33, 7, 1, "four"), (4, 40, 3, 1, "four"),
    (5, 41, 3, 1, "four"), (4, 56, 3, 1, "four"), (3, 57, 4, 1, "four"), (5, 16, 9, 0, "four"), (4, 17, 3, 0, "four"),
    (5, 24, 3, 0, "two"), (6, 25, 3, 0, "four"), (9, 8, 23, 1, "four"),
    (9, 10, 6, 1, "energy"), (9, 10, 6, 1, "enstrophy"), (9, 10, 6, 1, "uneven"),
    (60, 12, 1, 0, "two"), (61, 13, 1, 0, "two"), (7, 16, 1, 1, "two"), (8, 17, 1, 1, "two"), (7, 28, 1, 1, "two"),
    (6, 29, 1, 1, "two"), (57, 8, 1, 0, "four"), (9, 9, 1, 0, "four"), (12, 11, 1, 0, "uneven"),
    # one QoI of each kind at most, in 2-D: 64 - 2 (j + 2) cells in x, 16 rows with a halo of j + 1
    (56, 10, 1, 0, "pair"), (57, 11, 1, 0, "pair"), (112, 3, 1, 0, "pair"), (7, 16, 1, 1, "pair"), (8, 17, 1, 1, "pair"),
    (7, 26, 1, 1, "pair"), (3, 27, 1, 1, "pair"), (52, 6, 1, 0, "pair4"), (53, 7, 1, 0, "pair4"), (9, 22, 1, 1, "pair4"),
    (9, 23, 1, 1, "pair4"), (20, 21, 1, 0, "one"), (20, 21, 1, 1, "one4"),
]


def _workload(nx, ny, nz, walls, name):
    qois = SETS[name]
    if nz == 1:
        cfg = dict(lattice=0, nx=nx, ny=ny, nz=1, walls_y=walls, tau=0.55, substrate=0, cmodel=0.0,
                   force_kind=2 if walls else 1, force_amp=1e-6, force_k=1, drag=0.0)
    else:
        cfg = dict(lattice=1, nx=nx, ny=ny, nz=nz, walls_y=walls, tau=0.55, substrate=1, cmodel=0.1,
                   force_kind=2 if walls else 1, force_amp=1e-6, force_k=1, drag=0.0)
    u0 = synth.noise_velocity(2 if nz == 1 else 3, (nz, ny, nx), 0.02, 100 + nx + ny)
    C, mu, S = synth.lrs_model_channel(len(qois), 7, 9)
    return cfg, u0, qois, dict(mode="lrs", spinup=2, C=C, mu=mu, Sigma=S, seed=5)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}x{c[2]}-{'walls' if c[3] else 'periodic'}-{c[4]}")
def test_tile_limits(case, prec):
    """Velocity, q*, dQ and gamma after 6 steps, corrected from the third.
    FP64: the stated bars or ten times the workload's own FP64 resolution.
    FP32: a power is wrong by 6e-8 of v, which the highest pass filter
    amplifies by |v| / |(I - B) v| (about one on white noise), and the QoIs
    average it: 1e-5 of the velocity and of each q*; the corrections of the
    uneven set, whose sensitivities are nearly dependent, amplify it further
    and are compared in FP64 alone."""
    lbm = need_gpu()
    cfg, u0, qois, cargs = _workload(*case)
    steps = 6 if prec == "fp64" or case[4] != "uneven" else 2
    print(f"chain tiles {case} {prec}", flush=True)
    run = gpu_run(lbm, cfg, u0, prec, qois, cargs)
    run.step(steps)
    assert run.sync() == 0
    o = oracle_run(cfg, u0, qois, cargs)
    o.step(steps)
    rg, ro = run.record_arrays(), o.record_arrays()

    def per_qoi(key):
        return float(np.max(np.abs(rg[key] - ro[key]) / (np.max(np.abs(ro[key]), axis=0) + 1e-300)))

    got = [rel_err(run.fields()[1], o.velocity()[1]), per_qoi("q"), per_qoi("dq"), per_qoi("gamma")]
    print("  velocity %.2e  q %.2e  dq %.2e  gamma %.2e" % tuple(got), flush=True)
    assert np.array_equal(rg["flags"], ro["flags"])
    bars = fp64_bars(oracle_floor(cfg, u0, qois, cargs, steps, ref=o)) if prec == "fp64" else [1e-5, 1e-5, np.inf, np.inf]
    assert all(g <= b for g, b in zip(got, bars))
