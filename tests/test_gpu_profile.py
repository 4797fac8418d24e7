"""Launches per phase that lbm_profile_phases reports."""
import pytest

import synth
from gpu_util import gpu_run, need_gpu

pytestmark = pytest.mark.gpu

E = lambda *f: [("E", x, 0) for x in f]
Z = lambda *f: [("Z", x, 0) for x in f]
CASES = [
    # closure, curl launches, filter launches in 2-D and 3-D, reduce launches in 2-D and 3-D
    (E("B") + Z("B"), 0, (1, 1), (0, 1)), (E("B", "IMB") + Z("B"), 0, (1, 1), (1, 1)),
    (E("G1") + Z("L1"), 1, (2, 4), (1, 1)), (E("G1", "L1"), 0, (2, 4), (1, 1)),
    (E("F0-2") + Z("F0-2"), 0, (5, 5), (1, 1)), (E("F0-2", "G1") + Z("L1"), 1, (7, 9), (1, 1)),
]


@pytest.mark.parametrize("d", [2, 3])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "_".join(k + f for k, f, _ in c[0]))
def test_launches_per_phase(case, d):
    """Binomial chains and 2-D pairs: one launch; kernel filters: x and y parts,
    in 3-D z parts, twice; Fourier bands: pack, mask, unpack and two transforms."""
    lbm = need_gpu()
    qois, curl, filters, reduce = case
    nx, ny, nz = (24, 20, 1) if d == 2 else (12, 10, 8)
    cfg = dict(lattice=d - 2, nx=nx, ny=ny, nz=nz, walls_y=0, tau=0.55, substrate=0, cmodel=0.0, force_kind=1,
               force_amp=1e-6, force_k=1, drag=0.0)
    run = gpu_run(lbm, cfg, synth.noise_velocity(d, (nz, ny, nx), 0.02, 7), "fp32", qois, dict(mode="off"))
    print("profile", case[0], d, flush=True)
    _, n = run.profile_phases(2)
    got = list(n.values())
    assert got[1:4] == [curl, filters[d - 2], reduce[d - 2]]
    assert run.sync() == 0
