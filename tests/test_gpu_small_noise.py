"""Small FP64 instances with few replicas have their noise drawn ahead of the annealing launches, a bounded
number of iterations at a time. A recorded run draws it in the annealing kernel, as does a run of few iterations:
the same bits from both, over iteration counts that end inside, at and one past a launch, with noise of
either sign, for a continued run, and from a captured graph."""
import numpy as np
import pytest

import instances
from contraction_cases import signed_fields

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nmfa():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa as m

    return m


# n, R: iterations per launch 2 MB / (16 ceil(R / 16) * 16 ceil(n / 16) * 8 bytes)
@pytest.mark.parametrize("precision,n,R,counts", [
    ("fp64", 16, 1, (23, 24, 25, 1026)), ("fp64", 20, 256, (24, 32, 33, 67)), ("fp64", 33, 40, (27, 130)),
    ("fp64", 49, 131, (28, 30)), ("fp64", 112, 90, (24, 41)), ("fp64", 112, 17, (73, 150)), ("bf16", 78, 73, (83,))])
@pytest.mark.parametrize("negate", [False, True])
def test_same_bits(nmfa, precision, n, R, counts, negate):
    inst, h = instances.sk(n, 51), signed_fields(n, 0.5, 52)
    for count in counts:
        out = []
        for kw in ({}, {"record_iters": 1}):
            with nmfa.Solver(inst.J, h, precision=precision, negate_noise=negate, **kw) as s:
                s.anneal_range(R, 5000, 1, count, 53)
                first = s.state()
                s.anneal_range(R, 5000, count + 1, 2 * count, 53)
                out.append((first, s.state(), s.spins()))
        assert all(np.array_equal(x, y) for x, y in zip(*out)), count


def test_captured(nmfa):
    import torch

    inst = instances.sk(60, 54)
    with nmfa.Solver(inst.J, None, precision="fp64") as fresh:
        fresh.anneal(48, 200, 55)
        want = fresh.state()
    st = torch.cuda.Stream()
    with nmfa.Solver(inst.J, None, precision="fp64") as s:
        s.anneal(48, 200, 56, stream=st.cuda_stream)
        st.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=st):
            s.anneal(48, 200, 55, stream=st.cuda_stream)
        for _ in range(3):
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(s.state(), want)
            torch.zeros(1 << 20, device="cuda").add_(1.0)  # the program's own work between the replays
