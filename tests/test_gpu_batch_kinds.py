"""A member is bitwise the same alone and in a batch also where its batch mates
have other numbers of E and Z QoIs, so that the group's launches take other
variants of the chains and the reduce than the member's own would."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_run, need_gpu

pytestmark = pytest.mark.gpu

E = lambda *f: [("E", x, 0) for x in f]
Z = lambda *f: [("Z", x, 0) for x in f]
GROUPS = {
    "channel": (3, [E("B2", "BMID", "IMB") + Z("B2", "BMID", "IMB"), E("I", "B", "B2", "BMID", "IMB") + Z("B2"),
                    E("B", "B2") + Z("I", "B2", "BMID", "IMB"), E("B2", "BMID", "IMB", "B")]),
    "channel_8": (3, [E("I", "B", "B2", "IMB") + Z("I", "B", "B2", "IMB"), E("I", "B") + Z("I", "B", "B2", "BMID", "IMB")]),
    "pairs": (2, [E("B") + Z("B"), E("B"), Z("IMB")]),
    "periodic": (2, [E("B", "IMB") + Z("I", "B"), Z("I", "B", "IMB"), E("I", "B", "IMB")]),
}


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("name", sorted(GROUPS))
def test_batch_mates_of_other_kinds(name, prec):
    lbm = need_gpu()
    d, sets = GROUPS[name]
    print(f"batch kinds {name} {prec}", flush=True)
    runs = {"solo": [], "batch": []}
    for side in runs:
        for k, qois in enumerate(sets):
            nx, ny, nz = (33 + 8 * k, 29, 1) if d == 2 else (20 + 9 * k, 18, 11)
            cfg = dict(lattice=d - 2, nx=nx, ny=ny, nz=nz, walls_y=d - 2, tau=0.55, substrate=d - 2, cmodel=0.1,
                       force_kind=d - 1, force_amp=1e-6, force_k=1, drag=0.0)
            C, mu, S = synth.lrs_model_channel(len(qois), 7, 9)
            cargs = dict(mode="lrs", spinup=2, C=C, mu=mu, Sigma=S, seed=5 + k)
            runs[side].append(gpu_run(lbm, cfg, synth.noise_velocity(d, (nz, ny, nx), 0.02, 40 + k), prec, qois, cargs))
    for r in runs["solo"]:
        r.step(8)
        r.sync()
    b = lbm.Batch(runs["batch"])
    b.step(8)
    b.sync()
    for s, r in zip(runs["solo"], runs["batch"]):
        x, y = s.record_arrays(), r.record_arrays()
        for key in ("q", "dq", "gamma"):
            assert np.array_equal(x[key], y[key])
        assert np.any(x["dq"] != 0)
        assert np.array_equal(s.get_populations(), r.get_populations())
