"""Couplings that are no FP8 E4M3 values but round to FP4 E2M1 ones (a +-1 matrix with float noise): the
FP8-J precisions round them to FP8 first and keep the result in FP4, two columns to a byte. One noise-free
step from a state that the spin operands hold exactly, on every kernel that reads FP4 J, against the same
step in FP64 numpy on the rounded couplings (the normaliser is that of the given ones). The bar and its
derivation are those of tests/test_gpu_contraction.py: every partial sum is exact in FP32."""
import numpy as np
import pytest

from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, fp8_states,
                               grid_states)

pytestmark = pytest.mark.gpu

# given value -> FP8 E4M3 (steps of 2^-4 below 1, 2^-3 from 1, 2^-2 from 2, 2^-1 from 4; 2^-9 around 0)
ROUNDED = {1.01: 1.0, -0.99: -1.0, 0.999999999: 1.0, -1.0: -1.0, 1e-5: 0.0, 0.0: 0.0, 2.04: 2.0, -5.9: -6.0,
           3.1: 3.0, -0.52: -0.5, 1.0: 1.0}


@pytest.mark.parametrize("precision,n,flags", [
    ("fp8j_bf16s", 300, {}), ("fp8j_bf16s", 301, {}), ("fp8j_bf16s", 1025, {}), ("fp8j_bf16s", 2101, {}),
    ("fp8j_bf16s", 300, {"force_step": True}), ("fp8j_bf16s", 301, {"force_step": True}),
    ("fp8j_bf16s", 301, {"force_xcd": True, "force_lds_j": True}), ("fp8j_bf16s", 100, {}),
    ("fp8j_fp8s", 300, {}), ("fp8j_fp8s", 301, {})])
def test_rounded_before_packing(precision, n, flags):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    g = np.random.default_rng(n)
    given, held = np.array(list(ROUNDED)), np.array(list(ROUNDED.values()))
    k = np.triu(g.integers(0, len(given), (n, n)), 1)
    up = np.triu(np.ones((n, n)), 1)
    J, Jr = given[k] * up, held[k] * up
    J, Jr = J + J.T, Jr + Jr.T
    R = 21
    s0 = fp8_states(R, n, 5) if precision == "fp8j_fp8s" else grid_states(R, n, 5)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(J, None, precision=precision, alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T, **flags) as s:
        if n > 256:
            assert s.info()["j_format"] == "fp4_e2m1"
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 6)
        got = s.state()
    phi = (s0 @ Jr) / np.sqrt((J * J).sum(axis=1))
    want = ONE_STEP_ALPHA * -np.tanh(phi / ONE_STEP_T) + (1.0 - ONE_STEP_ALPHA) * s0
    assert np.max(np.abs(got - want)) <= ONE_STEP_TOL
