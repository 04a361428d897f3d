"""Sizes at which the kernels' tilings, remainders and fallbacks change,
against the oracle."""
import numpy as np
import pytest

import oracle as O
from tests.util import log, t

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mvf():
    import paper_1511_07106_amd as mvf
    return mvf


def _random_depth(rng, w, h, lo=0.3, hi=4.0):
    d = rng.uniform(lo, hi, (h, w)).astype(np.float32)
    d[rng.random((h, w)) < 0.05] = 0.0
    d[rng.random((h, w)) < 0.02] = np.nan
    d[rng.random((h, w)) < 0.02] = np.inf
    return d


POSE = np.array([[0.8, 0.0, 0.6, 0.1], [0.0, 1.0, 0.0, -0.2], [-0.6, 0.0, 0.8, 0.3]])


@pytest.mark.parametrize("w,h", [(1, 1), (63, 15), (64, 16), (65, 17), (131, 5), (200, 49)])
@pytest.mark.parametrize("d_v", [3, 12, 200])
def test_placement_counts_edges(mvf, w, h, d_v):
    """Block and wavefront remainders; cells of one voxel (every pixel its
    own cell, more than a block's LDS table holds) to one cell a frame.
    Counts are integers and must be equal."""
    log(f"placement counts {w}x{h} d_v {d_v}")
    rng = np.random.default_rng(w * 1000 + h)
    d = _random_depth(rng, w, h)
    K = np.array([60.0, 61.0, w / 2 - 0.3, h / 2 + 0.2], np.float32)
    og = O.OGrid((-1.0, -2.0, -0.5), 0.01, 4.0, 128)
    with mvf.Context() as ctx:
        gid = ctx.grid((-1.0, -2.0, -0.5), 0.01)
        want = O.placement_counts(d, K, POSE, og, d_v)
        if len(want) > 8192:   # the table's slots
            with pytest.raises(mvf._lib.MvfError):
                ctx.placement_count(t(d), POSE, K, gid, d_v, max_cells=16384)
        else:
            assert ctx.placement_count(t(d), POSE, K, gid, d_v, max_cells=16384) == want


def test_placement_counts_after_overflow(mvf):
    """More distinct cells than the table holds is refused; the next count on
    the context is exact again."""
    log("placement counts overflow")
    rng = np.random.default_rng(5)
    d = rng.uniform(0.5, 4.0, (110, 130)).astype(np.float32)
    K = np.array([60.0, 61.0, 64.7, 54.2], np.float32)
    og = O.OGrid((-1.0, -2.0, -0.5), 0.001, 4.0, 128)
    with mvf.Context() as ctx:
        gid = ctx.grid((-1.0, -2.0, -0.5), 0.001)
        for _ in range(2):
            with pytest.raises(mvf._lib.MvfError):
                ctx.placement_count(t(d), POSE, K, gid, 3, max_cells=16384)
            assert ctx.placement_count(t(d), POSE, K, gid, 500) == O.placement_counts(d, K, POSE, og, 500)
