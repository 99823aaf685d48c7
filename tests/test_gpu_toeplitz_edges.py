"""The Toeplitz path at the edges of its half-length transforms through the C
ABI against the oracle: N = M / 2 (the largest chain whose padding fills half
of the embedding), M / 2 + 1 (the general form) and one less, at every radix
plan; FP64 1e-11 and FP32 1e-5 per trajectory."""
import numpy as np
import pytest

from oracle import twa as otwa

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


@pytest.mark.parametrize("half", [128, 256, 512, 1024, 2048, 4096, 8192])
def test_half_length_edges(twa, half):
    for N in (half - 1, half, half + 1):
        for prec, tol in (("fp64", 1e-11), ("fp32", 1e-5)):
            if prec == "fp64" and N > 8193:
                continue
            T, dt, B = 3, 0.02 / N, 3
            ref = otwa.run(otwa.RunConfig(n_spin=N, w=3.0, alpha=0.9, n_traj=B, dt=dt, n_steps=T, seed=4,
                                          toeplitz=True))
            print("toeplitz %s N=%d" % (prec, N), flush=True)
            r = twa.run(twa.build_pump_toeplitz(N, 3.0, 0.9), B, dt, T, seed=4, precision=prec, pump_path="toeplitz",
                        want_final_state=True, norm_tol=-1)
            rs = np.stack(ref.final_state)
            rel = np.sqrt(((r.final_state - rs) ** 2).sum(axis=(0, 2)) / (rs ** 2).sum(axis=(0, 2))).max()
            assert rel < tol, (N, prec, rel)


@pytest.mark.parametrize("alpha", [0.0, 0.3, 3.0])
def test_spectrum_on_the_device(twa, alpha):
    """The embedding's spectrum is formed on the device: a chain whose noise
    and drift depend on all of it (alpha = 0: one eigenvalue, the rest clamped)."""
    N, B, T = 300, 6, 20
    dt = 0.02 / N
    ref = otwa.run(otwa.RunConfig(n_spin=N, w=0.5, alpha=alpha, n_traj=B, dt=dt, n_steps=T, seed=8, toeplitz=True))
    r = twa.run(twa.build_pump_toeplitz(N, 0.5, alpha), B, dt, T, seed=8, precision="fp64", pump_path="toeplitz",
                want_final_state=True, norm_tol=-1)
    assert np.abs(r.final_state - np.stack(ref.final_state)).max() < 1e-11
