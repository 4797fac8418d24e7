"""Fourier band closures whose QoIs need different packed fields (E alone, Z
alone, both of the same bands, of different ones, a band twice of one kind, a
band beside kernel filters) against the FP64 oracle, and the solve formed by the
apply for kernel-filter and Fourier closures against its own launch."""
import numpy as np
import pytest

import synth
from gpu_util import fp64_bars, gpu_run, need_gpu, oracle_floor, oracle_run, rel_err

pytestmark = pytest.mark.gpu

SETS = {
    "E": [("E", "F0-2", 0), ("E", "F3-4", 0)],
    "Z": [("Z", "F3-4", 0), ("Z", "F0-2", 0)],
    "same": [("Z", "F0-2", 0), ("E", "F0-2", 0), ("E", "F3-4", 0), ("Z", "F3-4", 0)],
    "different": [("E", "F0-2", 0), ("Z", "F1-3", 0)],
    "one_band_shared": [("E", "F0-1", 0), ("E", "F2-3", 0), ("Z", "F2-3", 0)],
    "mixed": [("E", "G1", 0), ("Z", "F0-2", 0), ("Z", "L1", 0)],
}


def _grid(d, seed=5):
    nx, ny, nz = (24, 17, 1) if d == 2 else (12, 9, 10)
    cfg = dict(lattice=d - 2, nx=nx, ny=ny, nz=nz, walls_y=0, tau=0.55, substrate=d - 2, cmodel=0.1, force_kind=1,
               force_amp=1e-6, force_k=1, drag=0.0)
    return cfg, synth.noise_velocity(d, (nz, ny, nx), 0.02, seed)


def _lrs(n):
    C, mu, S = synth.lrs_model_channel(n, 7, 9)
    return dict(mode="lrs", spinup=2, C=C, mu=mu, Sigma=S, seed=5)


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("name", sorted(SETS))
def test_packed_fields_fp64(name, d):
    """Velocity, q*, dQ and gamma after 6 steps, corrected from the third: the
    stated FP64 bars or ten times the workload's own FP64 resolution."""
    lbm = need_gpu()
    cfg, u0 = _grid(d)
    qois, cargs = SETS[name], _lrs(len(SETS[name]))
    print(f"fourier fields {name} {d}-D", flush=True)
    run = gpu_run(lbm, cfg, u0, "fp64", qois, cargs)
    run.step(6)
    assert run.sync() == 0
    o = oracle_run(cfg, u0, qois, cargs)
    o.step(6)
    rg, ro = run.record_arrays(), o.record_arrays()

    def per_qoi(key):
        return float(np.max(np.abs(rg[key] - ro[key]) / (np.max(np.abs(ro[key]), axis=0) + 1e-300)))

    got = [rel_err(run.fields()[1], o.velocity()[1]), per_qoi("q"), per_qoi("dq"), per_qoi("gamma")]
    print("  velocity %.2e  q %.2e  dq %.2e  gamma %.2e" % tuple(got), flush=True)
    assert np.array_equal(rg["flags"], ro["flags"])
    assert all(g <= b for g, b in zip(got, fp64_bars(oracle_floor(cfg, u0, qois, cargs, 6, ref=o))))


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("name", ["same", "mixed"])
def test_solve_in_apply_bitwise_equal(name, d):
    """Kernel-filter and Fourier closures: the solve formed by every apply
    workgroup (small launches) and k_solve (tune_mem bit 3) give the same
    bytes."""
    lbm = need_gpu()
    cfg, u0 = _grid(d)
    qois, cargs = SETS[name], _lrs(len(SETS[name]))
    out = []
    for tm in (0, 8):
        r = gpu_run(lbm, cfg, u0, "fp32", qois, cargs, tune_mem=tm)
        r.step(7)
        r.sync()
        out.append((r.get_state(), r.record_arrays()))
    assert out[0][0] == out[1][0]
    for key in ("q", "dq", "gamma"):
        assert np.array_equal(out[0][1][key], out[1][1][key])
