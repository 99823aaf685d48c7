"""The fused small-N kernel over its whole range through the C ABI against the
FP64 oracle: chain lengths at and around the edges of its 16-spin blocks (one
block; FP64 to 64, FP32 to 128), ensembles that leave the last workgroup
partly filled in both of its widths (8 and 16 trajectories), step counts
around its batches of 8, and the first lengths beyond it.  Bounds as the other
parity tests: FP64 1e-11, FP32 1e-5 per trajectory."""
import numpy as np
import pytest

from oracle import twa as otwa

pytestmark = pytest.mark.gpu
FUSED = 99


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


def _check(twa, prec, N, B, T, integ, fused=True, only=None):
    w, alpha, dt, s0z, burn = 2.0, 0.8, 0.02 / max(N, 8), -1.0 if N % 2 else 1.0, T // 3
    traj = None if only is None else np.array(only)
    ref = otwa.run(otwa.RunConfig(n_spin=N, w=w, alpha=alpha, n_traj=B if traj is None else len(traj), dt=dt,
                                  n_steps=T, seed=21, s0z=s0z, burnin=burn, integrator=integ, traj=traj))
    print("%s N=%d B=%d T=%d %s" % (prec, N, B, T, integ), flush=True)
    r = twa.run(twa.build_pump(N, w, alpha), B, dt, T, seed=21, s0z=s0z, burnin=burn, precision=prec, integrator=integ,
                want_final_state=True, want_traj=True, norm_tol=-1)
    assert (r.obs["tile_config"] == FUSED) == fused
    pick = slice(None) if traj is None else traj
    tol = 1e-11 if prec == "fp64" else 1e-5
    fs, rs = r.final_state[:, pick], np.stack(ref.final_state)
    rel = np.sqrt(((fs - rs) ** 2).sum(axis=(0, 2)) / (rs ** 2).sum(axis=(0, 2))).max()
    assert rel < tol, rel
    mrel = np.max(np.abs(r.traj_moments[pick] - ref.traj_moments) / np.abs(ref.traj_moments).max(axis=0))
    assert mrel < 10 * tol, mrel


@pytest.mark.parametrize("prec,N", [("fp64", n) for n in (1, 2, 15, 16, 17, 32, 33, 48, 49, 63, 64)] +
                         [("fp32", n) for n in (1, 16, 17, 33, 64, 65, 80, 81, 96, 97, 112, 113, 127, 128)])
def test_block_edges(twa, prec, N):
    for B, T, integ in ((1, 9, "heun"), (9, 17, "sib")):
        _check(twa, prec, N, B, T, integ)


@pytest.mark.parametrize("prec,N", [("fp64", 11), ("fp64", 40), ("fp32", 16), ("fp32", 100)])
def test_wide_workgroups(twa, prec, N):
    # more than 8 x 256 trajectories: 16 per workgroup, the last one with 3
    _check(twa, prec, N, 2051, 10, "heun", only=[0, 7, 8, 15, 16, 1024, 2047, 2048, 2050])


@pytest.mark.parametrize("T", [1, 2, 7, 8, 9, 16])
def test_batches_of_steps(twa, T):
    _check(twa, "fp64", 12, 20, T, "heun")
    _check(twa, "fp32", 30, 20, T, "sib")


def test_first_lengths_beyond(twa):
    _check(twa, "fp64", 65, 9, 10, "heun", fused=False)
    _check(twa, "fp32", 129, 9, 10, "heun", fused=False)


def test_timed_run_keeps_its_launches(twa):
    r = twa.run(twa.build_pump(100, 1.0, 1.0), 16, 2e-4, 10, precision="fp32", timing=True, norm_tol=-1)
    assert r.obs["tile_config"] != FUSED and r.obs["stage1_launches"] == 10
