"""Couplings that are multiples of 1/2 up to 6 are classified and coded by a lookup, others by search: the
storage format that each kind of matrix takes, odd sizes included (FP4 packs two columns to a byte), one
noise-free step of it against the oracle (bars of tests/test_gpu_contraction.py; every partial sum is a
multiple of 2^-13 and below 2^10, so exact in FP32) and the cut, whose total weight is summed by rows."""
import numpy as np
import pytest

import oracle
from contraction_cases import ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, grid_states

pytestmark = pytest.mark.gpu

FP4 = [0.0, 0.5, 1.0, 1.5, 2.0, 3.0, 4.0, 6.0]


@pytest.mark.parametrize("n", [300, 301, 1025])
@pytest.mark.parametrize("extra,fmt", [((), "fp4_e2m1"), ((2.5, 5.0), "fp8_e4m3"), ((7.0,), "fp8_e4m3"),
                                       ((0.25, 5.5), "fp8_e4m3"), ((1.0 + 2.0**-7,), "bf16")])
def test_formats(n, extra, fmt):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    g = np.random.default_rng(n)
    mags = np.array(FP4 + list(extra))
    u = np.triu(g.choice(mags, size=(n, n)) * np.where(g.random((n, n)) < 0.5, -1.0, 1.0), 1)  # -0.0 too
    J = u + u.T
    R = 21
    s0 = grid_states(R, n, 5)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(J, None, precision="bf16", alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T) as s:
        assert s.info()["j_format"] == fmt
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 6)
        got = s.state()
        cut, E, spins = s.cuts(), s.energies()[0], s.spins().astype(np.float64)
    sub = [0, R // 2, R - 1]
    _, want, _ = oracle.anneal(J, None, T[:ONE_STEP_T_AT], replicas=sub, seed=6, alpha=ONE_STEP_ALPHA, sigma=0.0,
                               t_first=ONE_STEP_T_AT, s_init=s0[sub])
    assert np.max(np.abs(got[sub] - want)) <= ONE_STEP_TOL
    assert np.array_equal(E, 0.5 * ((spins @ J) * spins).sum(axis=1))  # multiples of 2^-8: exact
    assert np.array_equal(cut, (np.triu(J, 1).sum() - E) / 2.0)
