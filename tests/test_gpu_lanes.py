"""Chains of a few spins in many trajectories, a spin to a lane: chain lengths
at both ends of the powers of two that share a wave, the last length and the
first ensemble that take this kernel and their neighbours that do not, the last
workgroup partly filled; sampled trajectories through the C ABI against the
FP64 oracle with the bounds of the other fused tests."""
import pytest

from .test_gpu_fused_range import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


@pytest.mark.parametrize("N", [1, 2, 3, 4])
@pytest.mark.parametrize("B,T", [(1, 9), (31, 17), (33, 1)])
def test_few_spins_any_ensemble(twa, N, B, T):
    for integ in ("heun", "sib"):
        _check(twa, "fp32", N, B, T, integ)


@pytest.mark.parametrize("prec,N", [("fp32", n) for n in (5, 8, 9, 15, 16, 17, 20, 27, 28, 29)] +
                         [("fp64", n) for n in (1, 2, 7, 8, 9)])
@pytest.mark.parametrize("B", [4096, 4097])
def test_many_trajectories(twa, prec, N, B):
    only = [0, 1, 7, 8, 31, 32, 63, 64, 2047, 4094, 4095] + ([4096] if B > 4096 else [])
    for integ in ("heun", "sib"):
        _check(twa, prec, N, B, 11, integ, only=only)
