"""A scan's tune file of an earlier version: an entry that names a tile which
is no candidate any more, but which scans have, is taken as it stands and
nothing is timed again; one that no scan has is replaced once."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def twa():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_10075_amd as m
    return m


@pytest.mark.parametrize("prec,old,taken", [("fp32", 3, True), ("fp32", 2, True), ("bf16", 2, True), ("fp64", 3, True),
                                            ("fp32", 5, False), ("fp64", 7, False), ("bf16x3", 99, False)])
def test_entries_of_earlier_versions(twa, tmp_path, prec, old, taken):
    pts, cache = [(200, 1.0, 1.0, 1e-4, 3), (230, 2.0, 0.5, 1e-4, 4)], tmp_path / "tune.txt"
    kw = dict(precision=prec, norm_tol=-1, tune_cache=str(cache))
    twa.run_batch(pts, 40, 12, **kw)
    key = cache.read_text().split()[0]
    cache.write_text("%s %d\n" % (key, old))
    outs = twa.run_batch(pts, 40, 12, **kw)
    lines = cache.read_text().splitlines()
    assert len(lines) == (1 if taken else 2)
    if taken:
        assert all(o["tile_config"] == old for o in outs)
    again = twa.run_batch(pts, 40, 12, **kw)
    assert cache.read_text().splitlines() == lines
    assert [o["tile_config"] for o in again] == [o["tile_config"] for o in outs]
    assert [o["SpSm"] for o in again] == [o["SpSm"] for o in outs]
