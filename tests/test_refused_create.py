"""A context that nmfa_create refuses is released: the copy of the explicit temperatures (8 MB here) does not stay
behind. No GPU is needed to refuse one."""
import os

import numpy as np
import pytest


def _resident_mb():
    with open("/proc/self/statm") as f:
        return int(f.read().split()[1]) * os.sysconf("SC_PAGE_SIZE") / 2**20


@pytest.mark.parametrize("kw", [dict(precision="fp32", force_xcd=True), dict(precision="fp8j_fp8s", force_step=True)])
def test_nothing_is_kept(kw):
    # imported here: the module is collected for GPU runs too, and the library loaded before torch brings a second HIP
    # runtime into the process, in which no device is found
    from paper_1806_08422_amd import nmfa

    J = np.ones((8, 8)) - np.eye(8)
    T = np.ones(1 << 20)
    before = None
    for k in range(60):
        with pytest.raises(nmfa.NmfaError) as e:
            nmfa.Solver(J, None, temperatures=T, **kw)
        assert e.value.code == nmfa.NMFA_EINVAL
        if k == 9:
            before = _resident_mb()
    assert _resident_mb() - before < 100
