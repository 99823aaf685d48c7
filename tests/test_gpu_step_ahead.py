"""The noise of a step made beside the corrector of the step before, and the
window sums taken beside the predictor of the step after: every window edge
(no sample, one, all), odd and even step counts, chain lengths at the edges of
four spins and of a K stage, ensembles at the edges of a noise block, replayed
from graphs and launched directly.  Bounds: the window moments are of the
fourth order in the state, so four times those of the state of the precision
(FP64 1e-11, FP32 1e-5, BF16 5e-3)."""
import numpy as np
import pytest

from oracle import pump as opump, twa as otwa

pytestmark = pytest.mark.gpu
TOL = {"fp64": 4e-11, "fp32": 4e-5, "bf16": 2e-2}


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


def _rel(got, ref):
    num = np.sqrt(((got - ref) ** 2).sum(axis=1))
    return float(np.max(num / np.sqrt((ref ** 2).sum(axis=1))))


@pytest.mark.parametrize("N,B,T,burnin", [(49, 17, 1, 0), (66, 33, 33, 0), (95, 64, 34, 33), (129, 65, 35, 17)])
@pytest.mark.parametrize("prec,cfgs", [("fp64", (0, 1, 2)), ("fp32", (0, 1, 4)), ("bf16", (0, 1))])
def test_window_moments_match_oracle(twa, prec, cfgs, N, B, T, burnin):
    w, alpha, dt = 2.0, 0.7, 0.02 / N
    p, op = twa.build_pump(N, w, alpha), opump.build_pump(N, w, alpha)
    for integ in ("heun", "sib"):
        ref = otwa.run(otwa.RunConfig(n_spin=N, w=w, alpha=alpha, n_traj=B, dt=dt, n_steps=T, burnin=burnin, seed=5,
                                      integrator=integ), op)
        for cfg in cfgs:
            got = [twa.run(p, B, dt, T, burnin=burnin, seed=5, precision=prec, integrator=integ, tile_config=cfg,
                           want_traj=True, norm_tol=-1, use_graph=ug) for ug in (True, False)]
            assert np.array_equal(got[0].traj_moments, got[1].traj_moments)
            rel = _rel(got[0].traj_moments, ref.traj_moments)
            assert rel < TOL[prec], (cfg, integ, rel)


def test_no_window_and_batch(twa):
    N, B, dt = 70, 40, 2e-4
    p = twa.build_pump(N, 2.0, 0.7)
    r = twa.run(p, B, dt, 20, burnin=20, seed=5, tile_config=1, norm_tol=-1)
    assert r.obs["n_samples"] == 0
    pts = [(N, 2.0, 0.7, dt, 5), (131, 1.0, 1.5, dt, 6)]
    for T, burnin in ((33, 0), (34, 33)):
        res = twa.run_batch(pts, B, T, burnin=burnin, tile_config=1, want_traj=True, norm_tol=-1)
        for i, (n, w, a, d, seed) in enumerate(pts):
            one = twa.run(twa.build_pump(n, w, a), B, d, T, burnin=burnin, seed=seed, point=i, precision="fp32",
                          tile_config=1, want_traj=True, norm_tol=-1)
            assert np.array_equal(res[i].traj_moments, one.traj_moments)
