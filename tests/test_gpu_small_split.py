"""With few replicas the small-N kernel gives a workgroup 8 or 4 replicas instead of 16 and shares a replica's
rows among the lanes of its copies. A replica's run does not depend on it: the first replicas of runs on both
sides of the counts where the split changes agree bit for bit, noise of either sign, and with a recorded
run (whose noise is always drawn in the kernel)."""
import numpy as np
import pytest

import instances
from contraction_cases import signed_fields

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n,counts", [
    ("fp64", 16, (1, 1024, 2048, 4100)), ("fp64", 31, (5, 1024, 1025, 2049, 4100)), ("fp64", 62, (9, 1023, 1030, 2050)),
    ("fp64", 112, (3, 1024, 2000, 2100)), ("fp32", 33, (1, 2048, 2049)), ("fp32", 170, (13, 2047, 2100)),
    ("bf16", 17, (7, 2048, 2049)), ("bf16", 256, (8, 100, 2100)), ("fp8j_bf16s", 130, (21, 2060))])
@pytest.mark.parametrize("negate", [False, True])
def test_prefix(precision, n, counts, negate):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    inst, h = instances.sk(n, 61), signed_fields(n, 0.5, 62)
    first = None
    for R in counts:
        for record in (0, 3):
            with nmfa.Solver(inst.J, h, precision=precision, negate_noise=negate, record_iters=record) as s:
                s.anneal(R, 101, 63)
                st, sp = s.state()[:counts[0]], s.spins()[:counts[0]]
                tr = s.trajectory()[:, :counts[0]] if record else None
            if first is None:
                first = st, sp
            assert np.array_equal(st, first[0]) and np.array_equal(sp, first[1]), (R, record)
            if record:
                if len(first) == 2:
                    first = first + (tr,)
                assert np.array_equal(tr, first[2]), R
