"""Sizes at which the persistent small-N kernel and the register-ELL sparse kernel take another
variant: operand reads per lane (the padded row length), FP64 waves per row tile, slots per row.

* Small N: one noise-free step at constant T = 1 from a 1/64-grid state against the oracle (bars of
  tests/test_gpu_contraction.py; FP64 1e-9), then noisy runs of 1, 2 and 3 iterations from the same
  state: the iterations are unrolled by two, so an odd and an even count end in different buffers;
  continuing a run of 1 or 2 must give the run of 3 bit for bit.
* Sparse: every slot count against the generic ELL kernel, bit for bit, over 1, 2 and 5 iterations.
"""
import numpy as np
import pytest

import instances
import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, grid_states,
                               signed_fields)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nmfa():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa as m

    return m


@pytest.mark.parametrize("precision,n", [
    ("bf16", 32), ("bf16", 33), ("bf16", 96), ("bf16", 128), ("bf16", 129), ("bf16", 192), ("bf16", 224),
    ("bf16", 256), ("fp8j_bf16s", 31), ("fp8j_bf16s", 160), ("fp8j_bf16s", 256), ("fp32", 16), ("fp32", 49),
    ("fp32", 112), ("fp32", 160), ("fp32", 176), ("fp64", 16), ("fp64", 17), ("fp64", 32), ("fp64", 33),
    ("fp64", 64), ("fp64", 80), ("fp64", 112)])
@pytest.mark.parametrize("R", [1, 37])
def test_small_kernel(nmfa, precision, n, R):
    inst = instances.sk(n, 71)
    h = signed_fields(n, 0.5, 72)
    s0 = grid_states(R, n, 73)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(inst.J, h, precision=precision, alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T) as s:
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 74)
        got = s.state()
        assert s.info()["path"] == "persistent"
    sub = sorted({0, R // 2, R - 1})
    _, want, _ = oracle.anneal(inst.J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=74, alpha=ONE_STEP_ALPHA, sigma=0.0,
                               t_first=ONE_STEP_T_AT, s_init=s0[sub])
    assert np.max(np.abs(got[sub] - want)) <= (1e-9 if precision == "fp64" else ONE_STEP_TOL)
    with nmfa.Solver(inst.J, h, precision=precision) as s:
        ends = {}
        for first in (3, 1, 2):
            s.set_state(s0)
            s.anneal_range(R, 2000, 1001, 1000 + first, 75)
            if first < 3:
                s.anneal_range(R, 2000, 1001 + first, 1003, 75)
            ends[first] = (s.state(), s.spins())
    for first in (1, 2):
        assert np.array_equal(ends[first][0], ends[3][0]) and np.array_equal(ends[first][1], ends[3][1])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,d", [(301, 3), (300, 4), (302, 5), (513, 6), (400, 8), (400, 9), (402, 10), (400, 12),
                                 (400, 13), (500, 16), (2050, 3), (2051, 4), (2052, 6), (2100, 8)])
def test_sparse_slots(nmfa, precision, n, d):
    g = np.random.default_rng(n + d)
    J = np.zeros((n, n))
    for _ in range(d):  # up to d neighbours per spin, weights on a 1/8 grid
        p = g.permutation(n)
        a, b = p[: n // 2], p[n // 2: 2 * (n // 2)]
        J[a, b] = J[b, a] = g.integers(1, 16, n // 2) / 8.0
    h = g.normal(0.0, 0.5, n)
    R = 19
    s0 = grid_states(R, n, 76)
    for count in (1, 2, 5):
        out = []
        for generic in (False, True):
            with nmfa.Solver(J, h, precision=precision, force_sparse=True, sparse_generic=generic) as s:
                s.set_state(s0)
                s.anneal_range(R, 2000, 1001, 1000 + count, 77)
                out.append((s.state(), s.spins()))
        assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]), count


@pytest.mark.parametrize("precision,n,w,T", [("bf16", 33, 1.0, 1e-40), ("fp32", 17, 1.0, 1e-40),
                                             ("fp64", 17, 1.0, 1e-310), ("bf16", 300, 0.7, 1e-40),
                                             ("bf16", 1100, 0.7, 1e-40)])
def test_padding_rows_at_vanishing_temperature(nmfa, precision, n, w, T):
    """1 / T overflows: every spin goes to the sign of its field, and the rows that pad n to the tile, which
    have no field, must not turn into NaNs that the zero couplings to them would spread. Two iterations of
    s <- 0.15 (-1) + 0.85 s from 0.5, a few roundings each. (The group kernels with real couplings: w = 0.7.
    With couplings exact in FP4 they multiply the noise by 1 / T first, which an infinite one makes NaN.)"""
    J = w * (np.ones((n, n)) - np.eye(n))
    with nmfa.Solver(J, np.full(n, 0.5), precision=precision, alpha=0.15, sigma=0.0,
                     temperatures=np.full(4, T)) as s:
        s.set_state(np.full((5, n), 0.5))
        s.anneal_range(5, 4, 2, 3, 78)
        got = s.state()
    want = 0.15 * -1.0 + 0.85 * (0.15 * -1.0 + 0.85 * 0.5)
    assert np.max(np.abs(got - want)) <= (1e-15 if precision == "fp64" else 1e-6)
