"""Register-ELL kernel: 7 and 8 couplings per row (8 slots) and 9 and 10 (10 slots), whose loop is rolled or
unrolled by the replicas per thread and, for one replica, by the replica count. Same trajectory as the
generic ELL kernel, bit for bit, on both sides of the counts, recorded iterations and odd lengths included."""
import numpy as np
import pytest

import instances
from contraction_cases import signed_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n,d,counts", [
    ("fp32", 300, 7, (64, 256, 257, 600, 1100)), ("bf16", 1998, 8, (256, 300, 520)), ("fp32", 1500, 9, (100, 520)),
    ("fp32", 1000, 10, (300, 1030)), ("fp64", 1000, 8, (70, 300))])
def test_slots(precision, n, d, counts):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    J = instances.random_regular(n, d, 81).J
    h = signed_fields(n, 0.25, 82)
    for R in counts:
        for t_f in (30, 31):
            out = []
            for generic in (False, True):
                with nmfa.Solver(J, h, precision=precision, sparse_generic=generic, record_iters=3) as s:
                    s.anneal(R, t_f, 83)
                    out.append((s.state(), s.spins(), s.trajectory()))
                    assert s.info()["path"] == ("sparse" if generic else "sparse_rq")
            assert all(np.array_equal(a, b) for a, b in zip(*out)), (R, t_f)
