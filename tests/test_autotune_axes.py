"""The autotuner times the launch shapes of the launches that a run makes, and
returns no line that was written when they shaped other launches."""
import ctypes as ct

import pytest

import synth
from paper_2609_32892_amd import lbm

from gpu_util import need_gpu


def _channel(prec, nx=64, ny=24, nz=16):
    cfg, _ = synth.channel_workload(nx, ny, nz, substrate=1, cmodel=0.1)
    nb, dmin, dmax = synth.channel_bands(ny)
    return (lbm.make_config(precision=prec, **cfg),
            lbm.ClosureSpec(synth.QOIS_3D, mode="off", nbands=nb, dmin=dmin, dmax=dmax))


def test_a_line_of_the_first_format_is_not_returned(tmp_path):
    cfg, spec = _channel("fp32")
    key = lbm.autotune_key(cfg, spec)
    assert key.startswith("lbm-tune-v")
    old = "lbm-tune-v1" + key[len("lbm-tune-v1"):]
    path = tmp_path / "tune.txt"
    path.write_text(f"{old}\t2 1 32 90.5\n")
    out = lbm.Tuning()
    rc = lbm.lib().lbm_autotune(ct.byref(cfg), ct.byref(spec.c), None, 0, None, 1, str(path).encode(), ct.byref(out))
    assert rc == lbm.ENOMEM and out.from_cache == 0   # a miss goes on to the (missing) arena


@pytest.mark.gpu
@pytest.mark.parametrize("case", ["pair", "two_each", "in_place", "records"])
def test_axes_of_the_launches_that_run(case, tmp_path):
    """A 2-D pair closure launches neither (one candidate); other closures the
    reduce (five); FP64 channels the tiled stream-collide as well."""
    need_gpu()
    if case in ("pair", "two_each"):
        cfg = lbm.make_config(precision="fp32", nx=48, ny=40, tau=0.55)
        q = [("E", "B", 0), ("Z", "B", 0)]
        spec = lbm.ClosureSpec(q if case == "pair" else q + [("E", "IMB", 0)])
    else:
        cfg, spec = _channel("fp32" if case == "in_place" else "fp64")
    print(f"autotune axes {case}", flush=True)
    t = lbm.autotune(cfg, spec, steps=20, cache=str(tmp_path / "tune.txt"))
    print(" ", t, flush=True)
    if case == "pair":
        assert t["candidates"] == 1 and t["tune_cpt"] == 0
    elif case != "records":
        assert t["candidates"] == 5
    else:
        assert t["candidates"] > 8
    if case != "records":
        assert t["tune_btx"] == 0 and t["tune_zc"] == 0
