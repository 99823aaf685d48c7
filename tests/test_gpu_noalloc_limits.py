"""Which runs twa_run_noalloc accepts: the largest ensemble of a chain length
and precision runs, one trajectory more is refused, and both ends are where
the buffers, padded to the counted tile (16x32 to N = 48, 64x64 to 768, above
that 128x128 here), reach the size of the scratch array; the largest ensemble
gives twa_run's result."""
import pytest

pytestmark = pytest.mark.gpu
LIMIT = 64 << 20


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


def _up(a, b):
    return (a + b - 1) // b * b


def _need(prec, N, B):
    mt, nt = (16, 32) if N <= 48 else (64, 64) if N <= 768 else (128, 128)
    se = 8 if prec == "fp64" else 4
    elt = {"fp64": 8, "fp32": 4}.get(prec, 2)
    op = 6 if prec == "bf16x3" else elt
    P, Bp = _up(N, max(mt, 64 // elt)), _up(B, nt // 2)
    nmt = P // mt
    pieces = [2 * P * P * op, 4 * Bp * P * op, 2 * Bp * P * op, 3 * Bp * P * se, 3 * Bp * P * se, 2 * Bp * se,
              2 * Bp * P * se, 3 * nmt * Bp * se, 3 * nmt * Bp * se, 2 * Bp * se, Bp * P * se, 10 * Bp * se, 8,
              2 * 1024 * 4, (32 * 5 + 3) * 8]
    return sum(_up(max(16, b), 256) for b in pieces)


def _largest(prec, N):
    lo, hi = 1, 1 << 20
    while lo < hi:
        mid = (lo + hi + 1) // 2
        lo, hi = (mid, hi) if _need(prec, N, mid) <= LIMIT else (lo, mid - 1)
    return lo


def test_known_limits():
    known = {("fp64", 16): 32256, ("fp32", 16): 64512, ("fp64", 48): 11136, ("fp32", 48): 22288, ("fp32", 32): 33136}
    for (prec, N), B in known.items():
        assert _largest(prec, N) == B


@pytest.mark.parametrize("prec,N", [(p, n) for p in ("fp64", "fp32", "bf16x3", "bf16")
                                    for n in (10, 16, 17, 32, 40, 48, 49, 64, 65, 128, 129, 700, 768, 769, 1000)])
def test_largest_ensemble_runs_and_one_more_is_refused(twa, prec, N):
    B = _largest(prec, N)
    p = twa.build_pump(N, 1.0, 1.0)
    print(prec, N, B, flush=True)
    kw = dict(seed=3, precision=prec, burnin=0, norm_tol=-1)
    got = twa.run_noalloc(p, B, 1e-5, 3, **kw)
    ref = twa.run(p, B, 1e-5, 3, use_graph=False, **kw).obs
    for k in ("T2", "T3", "T4", "Z", "ZZ"):
        if prec == "fp64":   # at the limit its tile may be the counted one: rounding order only
            assert abs(got[k] - ref[k]) <= 1e-12 * abs(ref[k]), k
        else:
            assert got[k] == ref[k], k
    with pytest.raises(twa.TWAError) as e:
        twa.run_noalloc(p, B + 1, 1e-5, 3, **kw)
    assert e.value.code == twa.TWA_ENOMEM
    need = int(str(e.value).split("needs ")[1].split()[0])
    assert need == _need(prec, N, B + 1) > LIMIT
