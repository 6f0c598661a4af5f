"""Energies at the ends of their range (limits of the sums, not of the tiles).

* nmfa_energies_of_noalloc takes other values than +-1 as the integers they are: all spins 40 and all
  couplings 127, where the sum of s_i y_i over 64 rows is beyond 32 bits (16 rows: 9.7e8 at n = 300).
* One row of couplings of 1e307, whose field at n = 70 is beyond the largest double: the energy is an
  infinity, not a NaN, whatever rows a tile holds beyond n.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    return nmfa, torch


@pytest.mark.parametrize("n", [64, 256, 257, 300, 640])
def test_wide_integer_spins(env, n):
    nmfa, torch = env
    J = 127.0 * (np.ones((n, n)) - np.eye(n))
    spins = np.full((3, n), 40, dtype=np.int8)
    spins[1] = -40
    spins[2, ::2] = -40
    with nmfa.Solver(J, None, precision="fp32") as s:
        d_s = torch.from_numpy(spins).cuda()
        d_E = torch.zeros(3, dtype=torch.float64, device="cuda")
        d_Ei = torch.zeros(3, dtype=torch.int64, device="cuda")
        s.energies_of_noalloc(3, d_s.data_ptr(), d_E.data_ptr(), d_Ei.data_ptr())
        torch.cuda.synchronize()
    w = spins.astype(np.int64)
    want = 127 * (w.sum(axis=1) ** 2 - (w * w).sum(axis=1)) // 2
    assert np.array_equal(d_Ei.cpu().numpy(), want) and np.array_equal(d_E.cpu().numpy(), want.astype(np.float64))


@pytest.mark.parametrize("sign", [1, -1])
def test_infinite_energy(env, sign):
    nmfa, torch = env
    n = 70
    J = np.zeros((n, n))
    J[:, n - 1] = J[n - 1, :] = 1e307 * sign
    J[n - 1, n - 1] = 0.0
    spins = np.ones((17, n), dtype=np.int8)
    with nmfa.Solver(J, None, precision="fp64") as s:
        E, _ = s.energies_of(spins)
        d_s = torch.from_numpy(spins).cuda()
        d_E = torch.zeros(17, dtype=torch.float64, device="cuda")
        s.energies_of_noalloc(17, d_s.data_ptr(), d_E.data_ptr())
        torch.cuda.synchronize()
    assert np.array_equal(E, np.full(17, sign * np.inf)) and np.array_equal(d_E.cpu().numpy(), E)
