"""Energies of Eq. 1 at the edges of the energy kernels' tiles (nmfa_energies_of and the allocation-
free form, which must agree bit for bit).

* Integral couplings: exact integers, or (real fields) the ascending FP64 sum of the oracle bit for
  bit. n on both sides of the one-launch limit (256 padded columns), with a last k block of 64 or 128
  (n = 320, 384) and row tiles that end inside a 128-row tile; R around 16, 64 and 128.
* Other couplings: the FP64 matrix product. |E - E_ref| <= (2 n + n / 64 + 8) 2^-53 (sum |J_ij| +
  sum |h_i|): n terms per row, as many products and partial sums over the rows, and the fields' terms.
"""
import numpy as np
import pytest

import instances
import oracle

pytestmark = pytest.mark.gpu


def _fields(kind, n):
    if kind == "none":
        return None
    g = np.random.default_rng(n)
    return g.integers(-5, 6, n).astype(float) if kind == "int" else g.normal(0.0, 0.5, n)


def _evaluate(J, h, spins):
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_08422_amd import nmfa

    R = spins.shape[0]
    with nmfa.Solver(J, h, precision="fp32") as s:
        E, Ei = s.energies_of(spins)
        d_s = torch.from_numpy(spins).cuda()
        d_E = torch.zeros(R, dtype=torch.float64, device="cuda")
        d_Ei = torch.zeros(R, dtype=torch.int64, device="cuda")
        s.energies_of_noalloc(R, d_s.data_ptr(), d_E.data_ptr(), d_Ei.data_ptr())
        torch.cuda.synchronize()
    assert np.array_equal(d_E.cpu().numpy(), E) and np.array_equal(d_Ei.cpu().numpy(), Ei)
    return E, Ei


def _signs(R, n):
    return np.where(np.random.default_rng(R + n).random((R, n)) < 0.5, -1, 1).astype(np.int8)


@pytest.mark.parametrize("n,R,fields", [
    (1, 1, "real"), (64, 17, "none"), (65, 16, "int"), (255, 33, "real"), (256, 130, "none"), (257, 1, "real"),
    (320, 64, "int"), (321, 65, "real"), (384, 129, "none"), (700, 127, "real"), (1100, 300, "int")])
def test_integral_couplings(n, R, fields):
    J, h, spins = instances.sk(n, 5).J, _fields(fields, n), _signs(R, n)
    E, Ei = _evaluate(J, h, spins)
    assert np.array_equal(E, oracle.energies(J, h, spins))
    if fields != "real":
        assert np.array_equal(Ei, oracle.energies_int(J, h, spins))


@pytest.mark.parametrize("n,R,fields", [
    (3, 5, "real"), (64, 64, "none"), (65, 17, "real"), (129, 1, "int"), (257, 100, "real"), (1000, 1100, "none")])
def test_real_couplings(n, R, fields):
    g = np.random.default_rng(7)
    u = np.triu(g.normal(size=(n, n)), 1)
    J, h, spins = u + u.T, _fields(fields, n), _signs(R, n)
    E, Ei = _evaluate(J, h, spins)
    assert not Ei.any()
    bar = (2 * n + n / 64 + 8) * 2.0**-53 * (np.abs(J).sum() + (0.0 if h is None else np.abs(h).sum()))
    rows = np.arange(0, R, max(1, R // 50))
    assert np.max(np.abs(E[rows] - oracle.energies(J, h, spins[rows]))) <= bar
