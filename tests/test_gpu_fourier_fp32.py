"""FP32 Fourier band closures against the FP64 oracle on flows whose components
differ by orders of magnitude: the error of a band-filtered component may scale
with that component, not with the others."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_run, need_gpu, oracle_run

pytestmark = pytest.mark.gpu


def test_small_vorticity_component_beside_a_large_velocity():
    """v_z = 0.1 cos x on 512 cells beside v_x, v_y of 5e-5 that vary over 8
    cells: w_z is 5e-4 of v_z and 0.03 of w_y.  One tracking step lowers the
    enstrophy by 5% at fixed energy, which takes dv_x, dv_y up to 7e-4.  What
    FP32 leaves in them: the stored state 2.1e-9 (the oracle with its state
    rounded to FP32), the rounding of Z in dQ 1e-7 / 0.05 of dv, 1.4e-9, and the
    transforms 3.3e-9 (emulated with complex64 transforms of one component each;
    1.7e-7 with w_z as the imaginary part of v_z).  The bar is four times
    their sum."""
    lbm = need_gpu()
    nx, ny, nz = 512, 8, 8
    z, y, x = np.meshgrid(*[2 * np.pi * np.arange(n) / n for n in (nz, ny, nx)], indexing="ij")
    u0 = np.stack([5e-5 * np.sin(y + z), 5e-5 * np.cos(x + z), 0.1 * np.cos(x)]).reshape(3, -1)
    cfg = dict(lattice=1, nx=nx, ny=ny, nz=nz, walls_y=0, tau=0.55, substrate=0, cmodel=0.0, force_kind=0, force_amp=0.0,
               force_k=1, drag=0.0)
    qois = [("E", "F0-2", 0), ("Z", "F0-2", 0)]
    free = oracle_run(cfg, u0, qois, dict(mode="off"))
    free.step(1)
    qref = free.record_arrays()["q"][:1] * np.array([[1.0, 0.95]])
    cargs = dict(mode="track", spinup=0)
    o = oracle_run(cfg, u0, qois, cargs, qref=qref)
    o.step(1)
    print("fourier fp32: small vorticity component", flush=True)
    run = gpu_run(lbm, cfg, u0, "fp32", qois, cargs, qref=qref)
    run.step(1)
    assert run.sync() == 0
    err = np.max(np.abs(run.fields()[1] - o.velocity()[1]), axis=1)
    print("  velocity error per component", err, flush=True)
    assert not np.any(o.record_arrays()["flags"])
    assert np.all(err[:2] <= 4 * (2.1e-9 + 1.4e-9 + 3.3e-9))


@pytest.mark.parametrize("d", [2, 3])
def test_a_band_twice_of_one_kind(d):
    """Two energy (enstrophy) QoIs of one band have the same q*, the oracle's to 8
    roundings of the field's energy, and a singular Gram matrix."""
    lbm = need_gpu()
    nx, ny, nz = (24, 17, 1) if d == 2 else (12, 9, 10)
    cfg = dict(lattice=d - 2, nx=nx, ny=ny, nz=nz, walls_y=0, tau=0.55, substrate=0, cmodel=0.0, force_kind=1,
               force_amp=1e-6, force_k=1, drag=0.0)
    u0 = synth.noise_velocity(d, (nz, ny, nx), 0.02, 5)
    qois = [("E", "F0-2", 0), ("Z", "F1-3", 0), ("E", "F0-2", 0), ("Z", "F1-3", 0)]
    print(f"fourier fp32: band twice {d}-D", flush=True)
    run = gpu_run(lbm, cfg, u0, "fp32", qois, dict(mode="off"))
    run.step(2)
    assert run.sync() == 0
    o = oracle_run(cfg, u0, qois, dict(mode="off"))
    o.step(2)
    q, ref = run.record_arrays()["q"], o.record_arrays()["q"]
    e = 0.5 * np.sum(u0 * u0)
    assert np.array_equal(q[:, :2], q[:, 2:])
    assert np.all(np.abs(q - ref) <= 8 * 1.2e-7 * e)
    assert np.all(run.record_arrays()["flags"] == 2) and np.all(o.record_arrays()["flags"] == 2)
