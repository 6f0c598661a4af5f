"""Couplings that FP4 does not hold, N <= 2048: the small register-J tiles serve them up to some replica
count, and beyond it the LDS-J group kernel (FP8) or the per-iteration kernel, whichever is estimated to be
the fastest. Which of them runs shows in the path and in the number of launches; a replica's run does not
depend on it, bit for bit, recorded iterations and a run resumed half-way included."""
import numpy as np
import pytest

import instances
from contraction_cases import signed_fields

pytestmark = pytest.mark.gpu


def _couplings(fmt, n):
    if fmt == "fp8":
        return 5.0 * instances.sk(n, 71).J
    u = np.triu(np.random.default_rng(n).normal(size=(n, n)), 1)
    return u + u.T


# (replicas, kernel): tiles: several launches of the small tiles, lds: one or two of the LDS-J kernel
@pytest.mark.parametrize("fmt,n,runs", [
    ("bf16", 1500, [(40, "tiles"), (300, "tiles"), (4096, "step"), (130, "tiles")]),
    ("bf16", 2000, [(33, "tiles"), (4000, "step")]),
    ("bf16", 1025, [(17, "tiles"), (9000, "step")]),
    ("fp8", 1300, [(40, "tiles"), (1024, "lds"), (2048, "lds"), (4096, "step")]),
    ("fp8", 1537, [(21, "tiles"), (1000, "lds")]),
    ("fp8", 2000, [(40, "tiles"), (1024, "lds")])])
def test_route_and_bits(fmt, n, runs):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    J, h = _couplings(fmt, n), signed_fields(n, 0.5, 72)
    keep, t_f, first = runs[0][0], 40, None
    with nmfa.Solver(J, h, precision="bf16", record_iters=2) as s:
        for R, kernel in runs:
            s.anneal(R, t_f, 73)
            out = [s.state()[:min(keep, R)], s.spins()[:min(keep, R)], s.trajectory()[:, :min(keep, R)]]
            info, launches = s.info(), s.last_timing()["launches"]
            if kernel == "step":
                assert info["path"] == "step" and launches == t_f, (R, info, launches)
            else:
                assert info["path"] in ("xcd", "xcd_fenced"), (R, info)
                # the 64 x 16 tile serves at most 256 replicas per launch, the LDS-J kernel 1024 or more
                assert kernel == "tiles" or launches <= (R + 1023) // 1024, (R, info, launches)
            if first is None:
                first = out
            assert all(np.array_equal(a, b) for a, b in zip(out, first)), (R, info)
            s.anneal_range(R, t_f, 1, 15, 73)
            s.anneal_range(R, t_f, 16, t_f, 73)
            assert np.array_equal(s.state()[:keep], first[0]), R
        s.anneal(runs[0][0], t_f, 73)
        E = s.energies()[0]
    bar = (2 * n + n / 64 + 8) * 2.0**-53 * (np.abs(J).sum() + np.abs(h).sum())
    sp = first[1].astype(np.float64)
    want = 0.5 * ((sp @ J) * sp).sum(axis=1) + sp @ h
    assert np.max(np.abs(E - want)) <= 2 * bar  # numpy's own sums are as far off


def test_forced_group_kernel_stays():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    with nmfa.Solver(_couplings("fp8", 1300), None, precision="bf16", force_xcd=True) as s:
        s.anneal(4096, 20, 74)
        assert s.info()["path"] in ("xcd", "xcd_fenced")
