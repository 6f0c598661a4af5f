"""A group run whose spins cross XCDs (device-scope fences) beside one that keeps its spins in the XCDs' L2, which
leaves these full of lines to be written back: the fenced run's arrival at the group barrier must not pass the
write-back of its spins. Both together have fewer workgroups than the chip has CUs. Same bits as alone."""
import numpy as np
import pytest

import instances

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R,precision", [(500, 64, "bf16"), (512, 64, "fp8j_fp8s"), (1000, 20, "bf16")])
def test_fenced_run_beside_local(n, R, precision):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    t_f, st = 500, [torch.cuda.Stream(), torch.cuda.Stream()]
    with nmfa.Solver(instances.sk(n, 96).J, None, precision=precision, force_fenced=True) as a, \
            nmfa.Solver(instances.sk(1000, 97).J, None, precision="bf16") as b:
        a.anneal(R, t_f, 1)
        want = a.spins(), a.state()
        b.anneal(128, 4 * t_f, 2)
        want_b = b.spins()
        for k in range(40):
            b.anneal(128, 4 * t_f, 2, st[0].cuda_stream)
            for _ in range(3):
                a.anneal(R, t_f, 1, st[1].cuda_stream)
            assert np.array_equal(a.state(), want[1]) and np.array_equal(a.spins(), want[0]), k
            assert a.info()["path"].endswith("_fenced")
            assert np.array_equal(b.spins(), want_b), k
