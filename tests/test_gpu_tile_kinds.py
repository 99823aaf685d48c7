"""The response copies, the reverse sweep and the forward-mode tangent on the
tiles that the automatic choice takes for them in FP32 and split BF16 (64x64
and 128x128, and 16x32 in split BF16; the narrower tiles give the bits of
these), one spin and one trajectory past a tile, against the FP64 oracle with
the bounds of the other tiles' tests; and FP64's own automatic tiles (32x32,
64x64 with two groups of waves) against its 64x64, rounding order apart."""
import numpy as np
import pytest

from . import test_gpu_tangent as tangent
from . import test_gpu_tiles as tiles
from .test_gpu_binary32_order import _outputs

pytestmark = pytest.mark.gpu

CASES = [("fp32", 1, 65, 33), ("fp32", 2, 257, 65), ("fp32", 3, 129, 65), ("bf16x3", 0, 65, 17),
         ("bf16x3", 1, 65, 33), ("bf16x3", 3, 129, 65)]


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


@pytest.mark.parametrize("prec,cfg,N,B", CASES)
def test_kinds_match_oracle(twa, prec, cfg, N, B):
    tiles.test_two_time_on_tile(twa, prec, cfg, N, B, {"fp32": 1e-5, "bf16x3": 1e-4}[prec])
    tiles.test_adjoint_on_tile(twa, prec, cfg, N, B, 2e-3)
    tangent.test_tangent_matches_oracle_gradient(twa, prec, N, B, cfg, 2e-3)


@pytest.mark.parametrize("N,B", [(700, 401), (1001, 497)])
@pytest.mark.parametrize("path", ["heun", "sib", "lags", "tangent", "adjoint"])
def test_fp64_automatic_tiles(twa, path, N, B):
    p = twa.build_pump(N, 2.0, 1.0)
    _, got = _outputs(twa, path, p, N, B, "fp64", -1)
    _, ref = _outputs(twa, path, p, N, B, "fp64", 1)
    for a, b in zip(got, ref):
        assert np.max(np.abs(a - b)) <= 1e-10 * np.max(np.abs(b))
