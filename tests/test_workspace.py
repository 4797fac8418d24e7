"""Arena sizes (no GPU): what a closure's workspace is made of."""
import ctypes as ct

import pytest

import synth  # noqa: F401  (the test folder's path set-up)
from paper_2609_32892_amd import lbm

SLACK = 4 << 20   # records, tables, partial sums


def _bytes(cfg, qois):
    spec = lbm.ClosureSpec(qois)
    return lbm.lib().lbm_required_bytes(ct.byref(cfg), ct.byref(spec.c))


@pytest.mark.parametrize("d", [2, 3])
def test_fourier_closures_have_no_kernel_filter_fields(d):
    """Populations twice, rho, v*, v, the records, V_s and (with Z QoIs) U_s and w
    of every QoI, and complex fields: the spectra of v* and w, and every component
    of a band QoI.  Nothing for kernel filters, three more fields per such QoI."""
    n = 128 if d == 3 else 2048
    cfg = lbm.make_config(lattice=d - 2, nx=n, ny=n, nz=n if d == 3 else 1, tau=0.6)
    N, Q, NC = n ** d, (9, 19)[d - 2], (1, 3)[d - 2]
    base = 2 * Q + 1 + d + d + 2 * d
    e, z = [("E", "F0-3", 0), ("E", "F4-8", 0)], [("Z", "F0-3", 0), ("Z", "F4-8", 0)]
    for qois in (e, z, e + z):
        ne, nz = (sum(k == x for k, _, _ in qois) for x in "EZ")
        fields = base + (ne + nz) * d + ((ne + nz + 1) * NC if nz else 0)
        fields += 2 * ((d if ne else 0) + (NC if nz else 0) + ne * d + nz * NC)
        need = _bytes(cfg, qois)
        assert 4 * N * fields <= need <= 4 * N * fields + 8 * N // 16 + SLACK
        both = _bytes(cfg, qois + [("E", "G1", 0)])
        assert both >= need + 4 * N * 4 * d
