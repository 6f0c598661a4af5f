"""An eager run on one stream while another stream is being captured (in the default mode, which forbids calls that
could disturb the capture): it must neither fail nor end the capture, also where the run is the first to need the
buffer for noise drawn ahead or shares the CUs with unfinished group launches."""
import numpy as np
import pytest

import instances

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,n,R", [("fp64", 20, 64), ("bf16", 600, 40)])
def test_eager_run_during_a_capture(precision, n, R):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    t_f, J = 200, instances.sk(n, 99).J
    with nmfa.Solver(J, None, precision=precision) as s, nmfa.Solver(J, None, precision=precision) as ref:
        ref.anneal(R, t_f, 3)
        want = ref.spins()
        s.anneal_range(R, t_f, 1, 10, 3)  # allocates for R and t_f; too short for noise drawn ahead
        s.spins()
        st, side = torch.cuda.Stream(), torch.cuda.Stream()
        x = torch.zeros(64, device="cuda")
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            x.add_(1.0)
            s.anneal(R, t_f, 3, st.cuda_stream)
            s.anneal(R, t_f, 3, st.cuda_stream)
            x.add_(1.0)
        assert np.array_equal(s.spins(), want)
        for k in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert x.tolist() == [2.0 * (k + 1)] * 64
