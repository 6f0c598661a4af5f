"""Tiles of the FP64 / FP32 per-iteration kernel (the mean field and update of Alg. 1, Sec. II).

The launcher picks the tile by the instance and replica count. At n = 1990 (a last row tile that is
nearly all padding) R = 1000, 500 and 100 run the 128 x 64, 64 x 64 and 32 x 32 tiles on a GPU with
256 CUs, each with a ragged last replica tile. One step at constant T = 1 from a 1/64-grid state is
compared with the oracle: every partial sum of J . s is exact in FP32 for +-1 couplings and such
states (19 significant bits), so the bar is that of tests/test_gpu_contraction.py, 1e-5 (1e-9 in
FP64, whose rounding errors stay below 1e-13). The tiles add the terms of a sum in one order, so
replicas 0..99 of three noisy steps agree bit for bit whatever the tile.
"""
import numpy as np
import pytest

import instances
import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, grid_states,
                               signed_fields)

pytestmark = pytest.mark.gpu

N, SIZES = 1990, (1000, 500, 100)


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-9), ("fp32", ONE_STEP_TOL)])
def test_step_tiles(precision, tol):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    inst = instances.sk(N, 61)
    h = signed_fields(N, 0.5, 62)
    s0 = grid_states(SIZES[0], N, 63)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    first = {}
    for R in SIZES:
        sub = [0, 17, 63, 64, R - 1]
        with nmfa.Solver(inst.J, h, precision=precision, alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T) as s:
            s.set_state(s0[:R])
            s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 64)
            got = s.state()
            assert s.info()["path"] == "step"
        _, want, _ = oracle.anneal(inst.J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=64, alpha=ONE_STEP_ALPHA,
                                   sigma=0.0, t_first=ONE_STEP_T_AT, s_init=s0[sub])
        assert np.max(np.abs(got[sub] - want)) <= tol, R
        with nmfa.Solver(inst.J, h, precision=precision) as s:
            s.set_state(s0[:R])
            s.anneal_range(R, 2000, 1001, 1003, 65)
            first[R] = s.state()[:100]
    assert np.array_equal(first[1000], first[500]) and np.array_equal(first[1000], first[100])
