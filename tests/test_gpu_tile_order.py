"""The raycast's launch order from given durations: every tile once, the slow
ones first and split over more blocks, within the launch's blocks, for every
level and both block sizes that compute it."""
import ctypes as C
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1511_07106_amd",
                   "libmvf_selftest.so")
PLAN, LEVELS, XCDS, SLACK, SLOTS = 16, 5, 8, 512, 256 * 20


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        raise ImportError(f"{LIB} not built; run paper_1511_07106_amd.build")
    import torch  # noqa: F401  (one HIP runtime per process: torch's, loaded first)
    lib = C.CDLL(LIB)
    lib.mvf_selftest_tile_order.argtypes = [C.c_void_p, C.c_void_p] + [C.c_int] * 6
    return lib


def launch(tiles, lanes=4):
    """(level of tiles without durations, blocks of the launch) as the library chooses them."""
    level = 0
    while level < 3 and tiles << (level + 1) <= 2 * lanes * SLOTS:
        level += 1
    blocks = max(tiles << level, min(8 * tiles, tiles + SLOTS)) + SLACK
    return level, (blocks + XCDS - 1) // XCDS * XCDS


def order(lib, cost, threads, fresh=0, lanes=4):
    tiles = len(cost)
    level, blocks = launch(tiles, lanes)
    cost = np.ascontiguousarray(cost, np.uint32).copy()
    out = np.full(PLAN + tiles, -1, np.int32)
    print(f"[gpu-case] tile order {tiles} tiles, {threads} threads", flush=True)
    assert lib.mvf_selftest_tile_order(cost.ctypes.data, out.ctypes.data, tiles, level, blocks, SLOTS, fresh, threads) == 0
    assert not cost.any()   # used up
    pos, block, perm = out[:LEVELS], out[8:8 + LEVELS + 1], out[PLAN:]
    np.testing.assert_array_equal(np.sort(perm), np.arange(tiles))
    # levels from the highest to 0, each on a whole window of tiles, its blocks behind the ones before
    ends = [tiles if l == 0 else pos[l - 1] for l in range(LEVELS)]
    assert pos[LEVELS - 1] == 0 and block[LEVELS - 1] == 0
    levels = np.zeros(tiles, int)
    for l in range(LEVELS - 1, -1, -1):
        n = ends[l] - pos[l]
        assert n >= 0 and (pos[l] % XCDS == 0 or n == 0)
        nxt = block[LEVELS] if l == 0 else block[l - 1]
        assert nxt - block[l] == (-(-n // XCDS) * XCDS << l)
        levels[pos[l]:ends[l]] = l
    assert block[LEVELS] <= blocks
    return perm, levels, level


@pytest.mark.parametrize("threads", [256, 1024])
@pytest.mark.parametrize("tiles", [1, 7, 8, 300, 2048, 2049, 4800, 8193, 14168, 25956, 70001])
def test_tile_order(lib, tiles, threads):
    rng = np.random.default_rng(tiles)
    # no durations, or one missing: one level for all tiles
    for cost, fresh in ((np.zeros(tiles), 0), (rng.integers(1, 5000, tiles), 1)):
        _, levels, level = order(lib, cost, threads, fresh)
        assert (levels == level).all()
    one = rng.integers(1, 5000, tiles)
    one[tiles // 2] = 0
    _, levels, level = order(lib, one, threads)
    assert (levels == level).all()
    # spread durations: longest first (by quarter octaves, from 16 ticks to 1.5 * 2^19, all beyond in the
    # first and the last), and no lower level in front of a higher one
    cost = np.exp(rng.uniform(np.log(1), np.log(3e6), tiles)).astype(np.uint32)
    perm, levels, level = order(lib, cost, threads)
    d = cost[perm].astype(np.float64).clip(16.0, 1.5 * 2 ** 19)
    assert (d[1:] < d[:-1] * 1.26).all()
    assert (np.diff(levels) <= 0).all() and levels.min() >= max(level - 1, 0)


@pytest.mark.parametrize("tiles,lowest", [(25956, 0), (14168, 0), (4800, 2), (300, 2)])
def test_tile_order_levels(lib, tiles, lowest):
    """A few slow tiles among quick ones: the slow ones at the highest level, the
    quick ones at the lowest that images of their size take."""
    rng = np.random.default_rng(tiles)
    cost = rng.integers(30, 60, tiles)
    slow = rng.choice(tiles, max(8, tiles // 300), replace=False)
    cost[slow] = 30000
    perm, levels, _ = order(lib, cost, 256)
    assert (levels[np.isin(perm, slow)] == LEVELS - 1).all()
    assert levels[-1] == lowest and (levels == lowest).sum() > tiles // 2
