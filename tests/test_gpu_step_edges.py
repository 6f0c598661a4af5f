"""The tiled per-iteration kernels run over the N rows and the blocks of k that hold some k below N, not over
the padded matrix: sizes on both sides of a tile and of a block. One noise-free step against the oracle (bars of
tests/test_gpu_contraction.py; FP64 1e-9), and three noisy iterations on buffers that a longer run with more
replicas has used before against fresh ones, bit for bit."""
import numpy as np
import pytest

import instances
import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, grid_states,
                               signed_fields)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16", "fp8j_bf16s"])
@pytest.mark.parametrize("n,R", [(257, 1), (288, 65), (320, 129), (321, 64), (384, 33), (385, 200), (513, 257)])
def test_edges(precision, n, R):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    inst, h, s0 = instances.sk(n, 91), signed_fields(n, 0.5, 92), grid_states(R, n, 93)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(inst.J, h, precision=precision, alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T,
                     force_step=True) as s:
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 94)
        got = s.state()
        assert s.info()["path"] == "step"
    sub = sorted({0, R // 2, R - 1})
    _, want, _ = oracle.anneal(inst.J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=94, alpha=ONE_STEP_ALPHA, sigma=0.0,
                               t_first=ONE_STEP_T_AT, s_init=s0[sub])
    assert np.max(np.abs(got[sub] - want)) <= (1e-9 if precision == "fp64" else ONE_STEP_TOL)
    out = []
    for used in (False, True):
        with nmfa.Solver(inst.J, h, precision=precision, force_step=True) as s:
            if used:
                s.anneal(R + 300, 7, 95)
            s.set_state(s0)
            s.anneal_range(R, 2000, 1001, 1003, 96)
            out.append((s.state(), s.spins()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])
