"""Small tiles of the register-J group kernel (N <= 2048, BF16 spins): 64 x 16, 128 x 16 and 128 x 32
rows x replicas per workgroup, taken by instance size and replica count.

* One noise-free step at constant T = 1 from a 1/64-grid state against the oracle, in the three J
  formats, at sizes on both sides of a padding step and replica counts that leave a ragged last
  group and take different tiles. All partial sums are exact in FP32 (the bar and its derivation are
  those of tests/test_gpu_contraction.py; the +-5 couplings scale the sums by 5, three bits more).
* Replica-prefix invariance across tiles and launches: a replica's trajectory depends on neither,
  bit for bit, with fields and negated noise. 600 iterations at n = 300, where the spins of two
  iterations fit a CU's L1, also show a workgroup that reads the spins of two iterations ago.
* Device-scope fences give the same bits as the exchange inside an XCD.
"""
import numpy as np
import pytest

import instances
import oracle
from contraction_cases import (ONE_STEP_ALPHA, ONE_STEP_T, ONE_STEP_T_AT, ONE_STEP_TF, ONE_STEP_TOL, bf16_grid_couplings,
                               grid_states, signed_fields)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nmfa():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa as m

    return m


def _couplings(fmt, n):
    if fmt == "bf16":
        return bf16_grid_couplings(n, 21)
    return instances.sk(n, 20).J * (5.0 if fmt == "fp8_e4m3" else 1.0)


# n = 300: Kp = 512; 1024 / 1025: the largest Kp whose BF16 J fits 128 rows x 32 replicas, and one
# step more; 2000: Kp = 2048. The BF16-grid sums need few terms to stay exact (n <= 400).
@pytest.mark.parametrize("fmt,n,R", [
    ("fp4_e2m1", 300, 17), ("fp4_e2m1", 1024, 300), ("fp4_e2m1", 1025, 30), ("fp4_e2m1", 2000, 100),
    ("fp4_e2m1", 2000, 250), ("fp4_e2m1", 2000, 500), ("fp8_e4m3", 300, 1), ("fp8_e4m3", 1024, 700),
    ("fp8_e4m3", 1290, 130), ("fp8_e4m3", 2000, 40), ("bf16", 257, 33), ("bf16", 400, 1000)])
def test_one_step(nmfa, fmt, n, R):
    J = _couplings(fmt, n)
    h = signed_fields(n, 0.5, 22)
    s0 = grid_states(R, n, 23)
    T = np.full(ONE_STEP_TF, ONE_STEP_T)
    with nmfa.Solver(J, h, precision="bf16", alpha=ONE_STEP_ALPHA, sigma=0.0, temperatures=T) as s:
        s.set_state(s0)
        s.anneal_range(R, ONE_STEP_TF, ONE_STEP_T_AT, ONE_STEP_T_AT, 24)
        got, info = s.state(), s.info()
    assert info["j_format"] == fmt and info["path"].startswith("xcd"), info
    sub = sorted({0, R // 2, R - 1})
    _, want, _ = oracle.anneal(J, h, T[:ONE_STEP_T_AT], replicas=sub, seed=24, alpha=ONE_STEP_ALPHA, sigma=0.0,
                               t_first=ONE_STEP_T_AT, s_init=s0[sub])
    assert np.max(np.abs(got[sub] - want)) <= ONE_STEP_TOL


@pytest.mark.parametrize("fmt,n,counts,negate", [
    ("fp4_e2m1", 300, (40, 600, 5000), False), ("fp4_e2m1", 1000, (40, 500, 1000, 3000), True),
    ("fp4_e2m1", 2000, (40, 200, 500, 1024), False), ("fp8_e4m3", 1300, (40, 400), True),
    ("bf16", 900, (40, 400, 1000), False), ("bf16", 1500, (40, 700), True)])
def test_replica_prefix_across_tiles(nmfa, fmt, n, counts, negate):
    g = np.random.default_rng(31)
    if fmt == "bf16":
        u = np.triu(g.normal(size=(n, n)), 1)
        J = u + u.T
    else:
        J = _couplings(fmt, n)
    h = g.normal(0.0, 0.5, n)
    first = None
    for R in counts:
        with nmfa.Solver(J, h, precision="bf16", negate_noise=negate) as s:
            s.anneal(R, 600, 32)
            got, info = s.state()[:40], s.info()
        assert info["j_format"] == fmt
        if first is None:
            first = got
        assert np.array_equal(got, first), (R, info)


@pytest.mark.parametrize("n,R", [(300, 40), (1000, 300), (2000, 100), (2000, 500)])
def test_fenced_exchange_agrees(nmfa, n, R):
    inst = instances.sk(n, 41)
    out = []
    for fenced in (False, True):
        with nmfa.Solver(inst.J, None, precision="bf16", force_fenced=fenced) as s:
            s.anneal(R, 300, 42)
            out.append(s.state())
            assert s.info()["path"] == ("xcd_rj_fenced" if fenced else "xcd_rj")
    assert np.array_equal(out[0], out[1])
