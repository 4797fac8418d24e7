"""The kernel filters' separable passes against the FP64 oracle, which applies
each kernel as one direct convolution: every radius the library takes (G_s, s
= 1..6 in 3-D and 1..3 in 2-D; L_1, L_3, L_5; the identity), on grids one
cell within and past a tile (64 x 16) and a z chunk (8), smaller than the
radius, with walls and periodic; and closures of one kind and with more QoIs of
one kind than of the other."""
import numpy as np
import pytest

import synth
from gpu_util import fp64_bars, gpu_run, need_gpu, oracle_floor, oracle_run, rel_err

pytestmark = pytest.mark.gpu

CASES = [
    # (nx, ny, nz, walls, filters of E, filters of Z)
    (65, 15, 8, 1, ("G1", "L1"), ("G1", "L1")), (64, 17, 9, 1, ("G2", "L3"), ("G2", "L3")),
    (13, 16, 17, 0, ("G3", "L5"), ("G3", "L5")), (9, 12, 7, 1, ("G4", "I"), ("G4",)), (10, 9, 8, 0, ("G5",), ("G5", "I")),
    (7, 5, 6, 1, ("G6", "L5"), ("L3",)), (63, 33, 1, 0, ("G1", "L1"), ("G1", "L3")), (66, 16, 1, 1, ("G2", "L5"), ("G2", "L5")),
    (30, 31, 1, 0, ("G3", "L3"), ("G3",)), (24, 18, 6, 1, ("G1", "G3"), ()), (24, 18, 6, 1, (), ("G1", "L3")),
    (24, 18, 6, 1, ("G1", "G2", "G3", "L1", "L3"), ("L1",)),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}x{c[1]}x{c[2]}-{'walls' if c[3] else 'periodic'}-E{'.'.join(c[4])}-Z{'.'.join(c[5])}")
def test_radii_and_tile_limits_fp64(case):
    """Velocity, q*, dQ and gamma after 6 steps, corrected from the third: the
    stated FP64 bars or ten times the workload's own FP64 resolution."""
    lbm = need_gpu()
    nx, ny, nz, walls, fe, fz = case
    cfg = dict(lattice=0 if nz == 1 else 1, nx=nx, ny=ny, nz=nz, walls_y=walls, tau=0.55, substrate=0 if nz == 1 else 1,
               cmodel=0.1, force_kind=2 if walls else 1, force_amp=1e-6, force_k=1, drag=0.0)
    u0 = synth.noise_velocity(2 if nz == 1 else 3, (nz, ny, nx), 0.02, 100 + nx + ny)
    qois = [("Z", f, 0) for f in fz] + [("E", f, 0) for f in fe]
    C, mu, S = synth.lrs_model_channel(len(qois), 7, 9)
    cargs = dict(mode="lrs", spinup=2, C=C, mu=mu, Sigma=S, seed=5)
    steps = 6
    print(f"kernel filters {case}", flush=True)
    run = gpu_run(lbm, cfg, u0, "fp64", qois, cargs)
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
    assert all(g <= b for g, b in zip(got, fp64_bars(oracle_floor(cfg, u0, qois, cargs, steps, ref=o))))
