"""A closure that set_closure refuses leaves the run as it was."""
import numpy as np
import pytest

import synth
from gpu_util import gpu_run, need_gpu

pytestmark = pytest.mark.gpu


def test_a_residual_covariance_that_is_not_positive_definite():
    """The refused closure has other filters, radii and bands; the run goes on
    bitwise as one that was never offered it."""
    lbm = need_gpu()
    cfg, u0 = synth.channel_workload(24, 20, 10)
    nb, dmin, dmax = synth.channel_bands(20, 2)
    mp = [("MP", "I", 0), ("MP", "I", 1)]
    qois, other = [("E", "G1", 0), ("Z", "L1", 0)] + mp, [("E", "G3", 0), ("Z", "G2", 0)] + mp
    C, mu, S = synth.lrs_model_channel(4, 7, 9)
    cargs = dict(mode="lrs", spinup=2, C=C, mu=mu, Sigma=S, seed=5, nbands=nb, dmin=dmin, dmax=dmax)
    print("refused closure", flush=True)
    a, b = (gpu_run(lbm, cfg, u0, "fp32", qois, cargs) for _ in range(2))
    for r in (a, b):
        r.step(34)
    with pytest.raises(lbm.LbmError) as e:
        a.set_closure(lbm.ClosureSpec(other, **dict(cargs, Sigma=-S, dmin=2 * dmin)))
    assert e.value.code == lbm.EINVAL
    a.closure = b.closure
    for r in (a, b):
        r.step(33)
        assert r.sync() == 0
    assert np.array_equal(a.get_populations(), b.get_populations())
    x, y = a.record_arrays(), b.record_arrays()
    assert all(np.array_equal(x[k], y[k]) for k in ("q", "dq", "gamma"))
