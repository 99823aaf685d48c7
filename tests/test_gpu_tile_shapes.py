"""Every tile shape of every contraction precision through the C ABI against
the FP64 oracle, per trajectory: chain lengths and ensembles one short of, at
and one past a tile, so that padding rows, padding columns and the last round
of the operand ring are all met.  Bounds: those of the precision (FP64 1e-11;
FP32 1e-5, its operands hold all 24 bits of a value in three bf16 parts; split
BF16 1e-4; BF16 5e-3: 2^-8 per increment of 0.04 over 12 steps)."""
import numpy as np
import pytest

from oracle import pump as opump, twa as otwa

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-11, "fp32": 1e-5, "bf16x3": 1e-4, "bf16": 5e-3}


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


def _per_traj(got, ref):
    num = np.sqrt(((got - ref) ** 2).sum(axis=(0, 2)))
    return float(np.max(num / np.sqrt((ref ** 2).sum(axis=(0, 2)))))


@pytest.mark.parametrize("N,B", [(31, 17), (64, 32), (65, 33), (193, 97), (257, 64), (321, 129)])
@pytest.mark.parametrize("prec,cfgs", [("fp64", range(4)), ("fp32", range(9)), ("bf16x3", range(9)),
                                       ("bf16", range(9))])
def test_tile_shapes_match_oracle(twa, prec, cfgs, N, B):
    w, alpha, T, dt = 2.0, 0.7, 12, 0.02 / N
    p = twa.build_pump(N, w, alpha)
    op = opump.build_pump(N, w, alpha)
    for integ in ("heun", "sib"):
        ref = otwa.run(otwa.RunConfig(n_spin=N, w=w, alpha=alpha, n_traj=B, dt=dt, n_steps=T, seed=11,
                                      integrator=integ), op)
        for cfg in cfgs:
            print("%s N=%d B=%d %s tile %d" % (prec, N, B, integ, cfg), flush=True)
            r = twa.run(p, B, dt, T, seed=11, precision=prec, integrator=integ, tile_config=cfg, want_final_state=True,
                        want_traj=True, norm_tol=-1)
            assert r.obs["tile_config"] == cfg
            rel = _per_traj(r.final_state, np.stack(ref.final_state))
            assert rel < TOL[prec], (cfg, integ, rel)


def test_fp32_error_stays_at_binary32_rounding(twa):
    """A uniform rounding bias of the contraction is amplified by the
    collective decay: over 800 steps it must stay out of the trajectories
    (the binary32 matrix unit's own error here is below 8e-6)."""
    N, B, T, dt, w, alpha = 201, 64, 800, 2e-4, 3.0, 1.5
    p = twa.build_pump(N, w, alpha)
    ref = otwa.run(otwa.RunConfig(n_spin=N, w=w, alpha=alpha, n_traj=B, dt=dt, n_steps=T, seed=3))
    r = twa.run(p, B, dt, T, seed=3, precision="fp32", want_final_state=True, norm_tol=-1)
    assert _per_traj(r.final_state, np.stack(ref.final_state)) < 1e-5
