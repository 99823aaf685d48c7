"""Chains of short range: with a large exponent the whole spectrum of Eq. (2)
lies within round-off of w, so nothing but a real gap keeps the row that pads
an odd chain's antisymmetric block out of it.  A lost mode leaves F F off W by
its eigenvalue; the bound is round-off of the eigensolver and of the product,
as for the other chains.  The oracle's copy of the split, with the padding
eigenvalue at the bound of the row sums itself, shows what that loses."""
import numpy as np
import pytest


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


def _chain(n, w, alpha):
    d = np.abs(np.arange(n)[:, None] - np.arange(n)[None, :]).astype(float)
    return w * (1.0 + d) ** -alpha


def _split_root(n, w, alpha, factor):
    """Square root of an odd chain from its two halves, the padding row at factor x the bound of the row sums."""
    W, m = _chain(n, w, alpha), n // 2
    sym = W[:m + 1, :m + 1] + W[:m + 1, ::-1][:, :m + 1]
    anti = W[:m + 1, :m + 1] - W[:m + 1, ::-1][:, :m + 1]
    sym[m, :] *= np.sqrt(0.5)
    sym[:, m] *= np.sqrt(0.5)
    sym[m, m] = W[m, m]
    anti[m, :] = anti[:, m] = 0.0
    anti[m, m] = factor * w * (1.0 + 2.0 * sum((d + 1.0) ** -alpha for d in range(1, n)))
    l0, u0 = np.linalg.eigh(sym)
    l1, u1 = np.linalg.eigh(anti)
    V = np.zeros((n, n))
    for j in range(m + 1):
        V[:m, j], V[m, j], V[m + 1:, j] = u0[:m, j] / np.sqrt(2), u0[m, j], u0[:m, j][::-1] / np.sqrt(2)
    for j in range(m):   # the last of the second list is taken for the padding row
        V[:m, m + 1 + j], V[m + 1:, m + 1 + j] = u1[:m, j] / np.sqrt(2), -u1[:m, j][::-1] / np.sqrt(2)
    lam = np.concatenate([l0, l1[:m]])
    return W, (V * np.sqrt(np.maximum(lam, 0))) @ V.T


def test_the_gap_is_what_keeps_every_mode():
    lost = 0
    for n, alpha, w in ((51, 50.0, 0.3), (201, 50.0, 1.0), (1001, 40.0, 2.7), (51, 100.0, 1.0), (201, 20.0, 0.7)):
        for factor in (1.0, 2.0):
            W, F = _split_root(n, w, alpha, factor)
            off = np.max(np.abs(F @ F - W)) / w
            if factor == 2.0:
                assert off < 1e-10, (n, alpha, off)
            lost += off > 1e-3
    assert lost >= 1


@pytest.mark.gpu
@pytest.mark.parametrize("n", [17, 51, 52, 201, 1001])
@pytest.mark.parametrize("alpha", [20.0, 40.0, 50.0, 100.0, 700.0])
def test_short_range_chain_keeps_every_mode(twa, n, alpha):
    for w in (0.3, 1.0, 2.7):
        p = twa.build_pump(n, w, alpha)
        W, F = p.matrix("W"), p.matrix("F")
        assert np.max(np.abs(W - _chain(n, w, alpha))) <= 1e-14 * w
        assert np.max(np.abs(F @ F - W)) <= 1e-10 * w, (n, w, alpha)
        lam = np.linalg.eigvalsh(W)
        assert abs(p.lam_min - lam[0]) <= 1e-11 * w and abs(p.lam_max - lam[-1]) <= 1e-11 * w
