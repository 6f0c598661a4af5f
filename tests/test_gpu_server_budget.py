"""What a request with real couplings is charged to the server's budget covers the device memory that its context
holds, the partial sums of its energies included."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,R", [(1300, 1024), (2000, 2048)])
def test_charge_covers_the_context(n, R):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    u = np.triu(np.random.default_rng(n).normal(size=(n, n)), 1)
    t_f, kp = 20, (n + 255) // 256 * 256
    held = (2 * kp * kp + 8 * n * n            # BF16 couplings of the kernel, FP64 ones of the energies
            + R * n * (4 + 1 + 2 * 2 * kp / n)  # state, spins, two operand copies of the state
            + 16 * R + (n + 63) // 64 * R * 8)  # energies, their partial sums by 64 rows
    with nmfa.Server(precision="bf16", hbm_budget_bytes=1 << 30) as srv:
        t = srv.submit(u + u.T, None, R, t_f, 1)
        assert srv.wait(t, 60000) and srv.poll(t) == nmfa.JOB_DONE
        assert held <= srv.stats()["peak_bytes"] <= 1.05 * held
