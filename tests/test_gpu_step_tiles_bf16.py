"""Tile sizes of the per-iteration BF16 kernel (FP4, FP8 and BF16 couplings): the replica count picks
64 x 32, 128 x 32 or 128 x 64, 256 x 64, or 256 x 128. A replica's run depends on neither the replica count
nor the tile (every tile sums in the same order), so the first replicas of runs of all sizes agree bit for
bit, and one noise-free step of each agrees with the oracle (bars of tests/test_gpu_contraction.py)."""
import numpy as np
import pytest

import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, grid_states,
                               signed_fields)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt,scale", [("fp4_e2m1", 1.0), ("fp8_e4m3", 2.5), ("bf16", 1.0 + 2.0**-7)])
@pytest.mark.parametrize("n,counts", [(270, (1, 33, 16000)), (2100, (70, 300, 700, 1400, 3200))])
def test_tiles(fmt, scale, n, counts):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    g = np.random.default_rng(n)
    u = np.triu(np.where(g.random((n, n)) < 0.5, -scale, scale), 1)
    J, h = u + u.T, signed_fields(n, 0.5, 81)
    R = max(counts)
    s0 = grid_states(R, n, 82)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(J, h, precision="bf16", alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T, force_step=True) as s, \
            nmfa.Solver(J, h, precision="bf16", force_step=True) as noisy:
        assert s.info()["path"] == "step" and s.info()["j_format"] == fmt
        first = None
        for R in counts:
            s.set_state(s0[:R])
            s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 83)
            got = s.state()
            sub = sorted({0, R // 2, R - 1})
            _, want, _ = oracle.anneal(J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=83, alpha=ONE_STEP_ALPHA, sigma=0.0,
                                       t_first=ONE_STEP_T_AT, s_init=s0[sub])
            assert np.max(np.abs(got[sub] - want)) <= ONE_STEP_TOL, R
            noisy.set_state(s0[:R])
            noisy.anneal_range(R, 2000, 1001, 1003, 84)
            st = noisy.state()
            if first is None:
                first = st
            assert np.array_equal(st[:len(first)], first), R
