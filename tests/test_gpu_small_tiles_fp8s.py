"""Small tiles of the register-J group kernel with FP8 spins, taken by instance size and replica count: one
noise-free step from states exact in FP8 against the oracle (bars and exactness of
tests/test_gpu_contraction.py), every replica count's first replicas bit for bit (the largest counts take
the 256 x 32 tiles), and device-scope fences against the exchange inside an XCD."""
import numpy as np
import pytest

import instances
import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, fp8_states,
                               signed_fields)

pytestmark = pytest.mark.gpu

P = "fp8j_fp8s"


@pytest.fixture(scope="module")
def nmfa():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa as m

    return m


@pytest.mark.parametrize("n,R", [(257, 1), (300, 300), (600, 700), (1024, 300), (1290, 130), (1700, 33), (2000, 100),
                                 (2000, 500), (2048, 16)])
def test_one_step(nmfa, n, R):
    J, h, s0 = instances.sk(n, 20).J, signed_fields(n, 0.5, 22), fp8_states(R, n, 23)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(J, h, precision=P, alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T) as s:
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 24)
        got = s.state()
        assert s.info()["path"].startswith("xcd_rj")
    sub = sorted({0, R // 2, R - 1})
    _, want, _ = oracle.anneal(J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=24, alpha=ONE_STEP_ALPHA, sigma=0.0,
                               t_first=ONE_STEP_T_AT, s_init=s0[sub])
    assert np.max(np.abs(got[sub] - want)) <= ONE_STEP_TOL


@pytest.mark.parametrize("n,counts,negate", [(300, (40, 600, 5000), True), (1000, (40, 500, 1000, 4000), False),
                                             (1290, (40, 400), True), (2000, (40, 200, 500, 1024), False)])
def test_replica_prefix_across_tiles(nmfa, n, counts, negate):
    inst, h = instances.sk(n, 31), np.random.default_rng(31).normal(0.0, 0.5, n)
    first = None
    for R, fenced in [(counts[0], True)] + [(R, False) for R in counts]:
        with nmfa.Solver(inst.J, h, precision=P, negate_noise=negate, force_fenced=fenced) as s:
            s.anneal(R, 600, 32)
            got = s.state()[:counts[0]]
        if first is None:
            first = got
        assert np.array_equal(got, first), (R, fenced)
