"""The order in which the binary32 and split-BF16 contractions add up.

Below threshold <S+S-> = T2 + Z/2 is the small difference of two numbers of
the size of the chain, and g2, its jackknife error and dg2 divide by its
square and cube: a change of rounding that the moments do not show moves them
by 1e-5 and more.  So the order of every sum is part of what a precision
promises.  The values below were recorded with the binary32 matrix instruction
over K in order (split BF16: A.hi X.hi, A.hi X.lo, A.lo X.hi, one sweep after
the other) and 64-row tiles.  Bound: with the same order only the last bit of
the binary64 square root of the pump can differ, which flips the rounding of a
few elements of the operand by one part in 2^24; 1e-6 leaves a factor of 16
for the amplification of that one flip.

The narrow tiles that the automatic choice takes for few trajectories have the
rows of the tiles that a caller can ask for, so they give their bits.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


RECORDED = [
    ("adjoint", "fp32", 105, 255, 0.351, 2.741, 800,
     dict(SpSm=0.3813675006522885, g2=-43.792451909285525, g2_se=2037.1534730503088, d_SpSm_dw=1.3746772779815473,
          d_SpSm_dalpha=-0.1450539049306654, d_g2_dw=488.12701565933094, d_g2_dalpha=-29.564404292739482)),
    ("tangent", "fp32", 105, 255, 0.351, 2.741, 800,
     dict(g2_se=2037.1534730503088, d_SpSm_dw=1.3746715029795986, d_g2_dw=488.1264380532998,
          d_Sz_dw=32.65197323640189)),
    ("tangent", "bf16x3", 301, 241, 0.748, 1.675, 762,
     dict(SpSm=3.9615269037298333, g2=74.19343497573212, g2_se=116.02942205456053, d_SpSm_dw=3.0037754337889773,
          d_g2_dw=-121.10469363612812)),
    ("run", "fp32", 161, 732, 0.41, 2.543, 800,
     dict(SpSm=-0.11493800258844544, g2=-12636.016510784062, g2_se=2167852.903985613)),
    ("run", "bf16x3", 186, 158, 0.986, 2.298, 800,
     dict(SpSm=2.998681679022752, g2=7.454423624094745, g2_se=47.88975505674949)),
    ("run", "bf16x3", 179, 92, 0.864, 2.767, 800,
     dict(SpSm=1.9155904279902387, g2=132.60176547105993, g2_se=5952.777693957416)),
]


@pytest.mark.parametrize("path,prec,N,B,w,alpha,T,want", RECORDED)
def test_ill_conditioned_outputs_keep_their_values(twa, path, prec, N, B, w, alpha, T, want):
    p, dt, kw = twa.build_pump(N, w, alpha), 0.04 / N, dict(precision=prec, norm_tol=-1.0)
    if path == "run":
        got = twa.run(p, B, dt, T, 11, **kw).obs
    else:
        obs, g = (twa.adjoint(p, B, dt, T, 11, ckpt_every=16, **kw) if path == "adjoint"
                  else twa.tangent_w(p, B, dt, T, 11, **kw))
        got = {**obs, **g}
    for k, v in want.items():
        assert abs(got[k] - v) <= 1e-6 * abs(v), (k, got[k], v)


def _outputs(twa, path, p, N, B, prec, cfg):
    dt, T = 0.02 / N, 36
    kw = dict(precision=prec, norm_tol=-1.0, tile_config=cfg)
    if path in ("heun", "sib", "decay"):
        r = twa.run(p, B, dt, T, 3, integrator="sib" if path == "sib" else "heun", want_traj=True,
                    want_final_state=True, **kw)
        more = [r.traj_gen] if path == "decay" else []
    elif path == "lags":
        r = twa.run(p, B, dt, T, 3, burnin=16, n_lags=5, lag_stride=3, want_traj=True, want_final_state=True,
                    want_lags=True, **kw)
        more = [r.corr_blocks, r.chi_blocks]
    else:
        obs, g = (twa.adjoint(p, B, dt, T, 3, ckpt_every=16, **kw) if path == "adjoint"
                  else twa.tangent_w(p, B, dt, T, 3, **kw))
        return obs["tile_config"], [np.array([obs["T4"], obs["g2"], obs["g2_se"]]), np.array(list(g.values()))]
    return r.obs["tile_config"], [r.traj_moments, r.final_state] + more


@pytest.mark.parametrize("N,B", [(129, 33), (257, 100), (769, 70), (897, 33)])
@pytest.mark.parametrize("prec", ["fp32", "bf16x3", "bf16", "fp64"])
def test_narrow_tiles_give_the_wide_tiles_bits(twa, prec, N, B):
    pump = twa.build_pump(N, 2.0, 1.0)
    paths = ["heun", "sib", "lags", "tangent"] + (["adjoint"] if prec != "bf16" else [])
    if prec != "bf16x3":
        paths.append("decay")
    for path in paths:
        p = pump
        if path == "decay":
            i = np.arange(N)
            d = np.abs(i[:, None] - i[None, :])
            p = twa.build_model(pump.matrix("W"), 0.5 ** d, 0.1 * (d == 1.0))
        print(prec, N, B, path, flush=True)
        tile, got = _outputs(twa, path, p, N, B, prec, -1)
        _, ref = _outputs(twa, path, p, N, B, prec, tile)
        for a, b in zip(got, ref):
            if prec == "fp64":   # its automatic tiles add up in an order of their own
                assert np.max(np.abs(a - b)) <= 1e-10 * np.max(np.abs(b)), path
            else:
                assert np.array_equal(a, b), path
