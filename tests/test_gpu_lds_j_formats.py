"""The LDS-J group kernel with FP8 and BF16 couplings, which only force_lds_j pins for every replica count, and the
bits that it shares with the register-J tiles and the per-iteration kernel.

* One noise-free step from a 1/64-grid state against the oracle (bar and exactness: tests/test_gpu_contraction.py).
* The first replicas of runs at counts that take all three register-J tiles (n <= 1024: 64 x 16, 128 x 16 and
  128 x 32), of the LDS-J kernel and of the per-iteration kernel agree bit for bit, noise and fields included.
"""
import numpy as np
import pytest

import instances
import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL,
                               bf16_grid_couplings, grid_states, signed_fields)

pytestmark = pytest.mark.gpu

LDS_J = {"force_xcd": True, "force_lds_j": True}


@pytest.fixture(scope="module")
def nmfa():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa as m

    return m


def _couplings(fmt, n):
    return 5.0 * instances.sk(n, 11).J if fmt == "fp8_e4m3" else bf16_grid_couplings(n, 12)


@pytest.mark.parametrize("fmt,n,R", [
    ("fp8_e4m3", 400, 300), ("fp8_e4m3", 1290, 130), ("bf16", 400, 300), ("bf16", 321, 1)])
def test_one_step(nmfa, fmt, n, R):
    J, h, s0 = _couplings(fmt, n), signed_fields(n, 0.5, 13), grid_states(R, n, 14)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(J, h, precision="bf16", alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T, **LDS_J) as s:
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 15)
        got, info = s.state(), s.info()
    assert info["j_format"] == fmt and info["path"] in ("xcd", "xcd_fenced"), info
    sub = sorted({0, R // 2, R - 1})
    _, want, _ = oracle.anneal(J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=15, alpha=ONE_STEP_ALPHA, sigma=0.0,
                               t_first=ONE_STEP_T_AT, s_init=s0[sub])
    assert np.max(np.abs(got[sub] - want)) <= ONE_STEP_TOL


@pytest.mark.parametrize("fmt,n", [("fp8_e4m3", 900), ("fp8_e4m3", 1024), ("bf16", 700)])
def test_same_bits(nmfa, fmt, n):
    J, h, first = _couplings(fmt, n), signed_fields(n, 0.5, 16), None
    for R, flags in [(40, {}), (400, {}), (1000, {}), (40, LDS_J), (1000, LDS_J), (40, {"force_step": True})]:
        with nmfa.Solver(J, h, precision="bf16", **flags) as s:
            s.anneal(R, 150, 17)
            got, info = s.state()[:40], s.info()
        assert info["j_format"] == fmt
        if first is None:
            first = got
        assert np.array_equal(got, first), (R, flags, info)
