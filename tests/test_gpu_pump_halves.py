"""The chain's pump factorised by its symmetric and antisymmetric blocks, odd
and even lengths from the first that is, against the oracle and against the
solve of the whole matrix (the dense builder).  Bounds: those of the dense
builder's own test (round-off of a symmetric eigensolver, F's through the
square root)."""
import numpy as np
import pytest

from oracle import pump as opump

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


@pytest.mark.parametrize("n", [15, 16, 17, 65, 130, 257])
@pytest.mark.parametrize("w,alpha", [(2.0, 0.7), (0.3, 3.0), (1.5, 0.0), (0.0, 1.0)])
def test_chain_pump_matches_oracle_and_dense_solve(twa, n, w, alpha):
    p, ref = twa.build_pump(n, w, alpha), opump.build_pump(n, w, alpha)
    W, F = p.matrix("W"), p.matrix("F")
    lmax = max(ref.lam_max, 1e-300)
    assert np.max(np.abs(W - ref.W)) <= 1e-14 * lmax
    assert np.array_equal(F, F.T)
    assert np.max(np.abs(F @ F - W)) <= 1e-10 * lmax
    assert abs(p.lam_max - ref.lam_max) <= 1e-12 * lmax and abs(p.lam_min - ref.lam_min) <= 1e-11 * lmax
    d = twa.Pump(n, dense=W)
    assert np.max(np.abs(F - d.matrix("F"))) <= 1e-11 * max(1.0, np.sqrt(lmax))
    lam, V = np.linalg.eigh(W)
    assert np.max(np.abs((V * np.sqrt(np.maximum(lam, 0) * (lam > 8 * n * 2.3e-16 * lmax))) @ V.T - F)) <= \
        1e-11 * max(1.0, np.sqrt(lmax))
