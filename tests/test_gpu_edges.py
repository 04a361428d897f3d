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


@pytest.mark.parametrize("dims,share", [((2, 2, 2), 1.0), ((8, 8, 8), 1.0), ((9, 17, 8), 1.0), ((8, 8, 1100), 0.1),
                                        ((72, 80, 96), 1.0), ((40, 33, 130), 0.02), ((208, 200, 204), 0.15),
                                        ((200, 207, 211), 0.0003)])
def test_surface_points_edges(mvf, dims, share):
    """One brick, a brick and a voxel, a column of more than 128 bricks, more
    surface bricks than one group, one chunk and one sum of sums hold, volumes
    below and above the size at which surface bricks are listed first: points
    of random values in a share of the bricks, against the oracle on the same
    values (emitting voxels equal; positions within 1e-4 m and normals within
    2e-3, the bounds of the room tests)."""
    log(f"surface points {dims} share {share}")
    rng = np.random.default_rng(dims[0] + 7 * dims[2])
    nx, ny, nz = dims
    F = rng.uniform(0.05, 0.95, (nz, ny, nx)).astype(np.float32)
    bricks = rng.random([(n + 7) // 8 for n in (nz, ny, nx)]) < share
    neg = np.kron(bricks, np.ones((8, 8, 8), bool))[:nz, :ny, :nx] & (rng.random(F.shape) < 0.3)
    F[neg] *= -1.0
    W = np.where(rng.random(F.shape) < 0.002, 0, 7).astype(np.uint16)
    F[W == 0] = 0.0
    og = O.OGrid((-0.3, 0.1, 0.2), 0.02, 4.0, 128)
    with mvf.Context() as ctx:
        gid = ctx.grid((-0.3, 0.1, 0.2), 0.02)
        vid = ctx.volume(gid, (3, -5, 11), dims)
        ctx.write_volume(vid, F, W, np.zeros(F.shape + (4,), np.uint8))
        ov = O.OVolume(dims, (3, -5, 11), F.astype(np.float64), W, np.zeros(W.shape + (4,), np.uint8))
        ref = O.extract(ov, og, F32=F)
        got = {k: v.cpu().numpy() if hasattr(v, "cpu") else v for k, v in ctx.extract(vid).items()}
    assert got["n"] == ref["n"]

    def by_voxel(G, *arrs):
        order = np.lexsort((G[:, 0], G[:, 1], G[:, 2]))
        return [G[order]] + [a[order] for a in arrs]

    # the device writes bricks z fastest, then slices, then x fastest
    l = got["G"].astype(np.int64) - (3, -5, 11)
    bd = [(n + 7) // 8 for n in dims]
    key = (((l[:, 0] >> 3) * bd[1] + (l[:, 1] >> 3)) * bd[2] + (l[:, 2] >> 3)) * 512 + (l[:, 2] & 7) * 64 + \
        (l[:, 1] & 7) * 8 + (l[:, 0] & 7)
    assert np.all(np.diff(key) > 0)
    Gd, Vd, Nd = by_voxel(got["G"], got["V"].astype(np.float64), got["N"].astype(np.float64))
    Go, Vo, No = by_voxel(ref["G"], ref["V"], ref["N"])
    np.testing.assert_array_equal(Gd, Go)
    if got["n"]:
        assert np.abs(Vd - Vo).max() <= 1e-4
        ok = np.isfinite(No).all(axis=1)
        assert np.array_equal(ok, np.isfinite(Nd).all(axis=1))
        assert not ok.any() or np.abs(Nd[ok] - No[ok]).max() <= 2e-3


@pytest.mark.parametrize("w,h,iters", [(17, 13, (2,)), (64, 48, (2, 2)), (333, 251, (2, 1, 2)), (1100, 500, (2, 2, 1))])
def test_track_edges(mvf, w, h, iters):
    """Images of less than a block, of partial blocks and of more blocks than
    the last block sums in one go; one to three levels.  Every step pairs the
    oracle's pixels; squared errors within 1e-9 (sums in another order) and
    the pose within 1e-6, the bounds of the room tests."""
    log(f"track {w}x{h} {iters}")
    import torch
    f = 0.9 * w
    K = np.array([f, f, w / 2 - 0.4, h / 2 + 0.3], np.float32)
    u, v = np.meshgrid(np.arange(w), np.arange(h))
    x, y = (u - w / 2) / f, (v - h / 2) / f

    def surface(dz):
        z = 2.0 + dz + 0.25 * np.sin(5 * x + 0.3) * np.cos(4 * y) + 0.3 * x - 0.2 * y
        rng = np.random.default_rng(w)
        z[rng.random(z.shape) < 0.01] = 0.0
        return z.astype(np.float32)

    Tm = POSE
    Vc, Nc = O.vertex_normal(surface(0.0), K)
    Vm = (Vc.astype(np.float64) @ Tm[:, :3].T + Tm[:, 3]).astype(np.float32)
    Nm = (Nc.astype(np.float64) @ Tm[:, :3].T).astype(np.float32)
    d = surface(0.012)
    T32 = Tm.astype(np.float32).astype(np.float64)
    model = {"vertex": t(Vm), "normal": t(Nm)}
    with mvf.Context() as ctx:
        for _ in range(3):   # the state starts afresh with every call
            T, st = ctx.track(t(d), K, model, Tm, T32, iters=iters)
    T_ora, steps = O.icp_track(d, K, Vm, Nm, T32, T32, iters=iters)
    assert [s[1] for s in steps] == st["pairs"]
    for (_, _, e), e_dev in zip(steps, st["sq_err"]):
        assert abs(e - e_dev) <= 1e-9 * max(e, 1e-12)
    assert np.abs(T - T_ora).max() <= 1e-6
