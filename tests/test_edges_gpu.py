"""GPU parity at the edges of the kernels' tiles and of their dispatch rules.

- FP64 solves above 16 points: kept counts on both sides of every 16-point strip and bucket,
  grids whose queries do not fill a strip, rotated frames, FP32 buckets re-solved in FP64; the
  oracle's tolerances of the other fit tests.
- Frame kernel: voxel counts on both sides of the lines at 8,192 and 32,768 voxels. Sums are
  taken in the same order on either side, so a call's rows equal those of calls on parts of it.
- Map update: voxel counts on both sides of the 64 voxels a workgroup takes.
- Structure loss: point counts on both sides of a workgroup's and a list part's, points left
  open together, cells across the filter's 32-cell words and at the key range's ends. Values
  are compared with a float64 brute force (each is a handful of float32 roundings of numbers
  up to the distance: 1e-6 of it) and between cell sizes, where they have to be equal.
"""
import dataclasses

import numpy as np
import pytest

from oracle import vgpr_oracle as O
from paper_2410_17084_amd import configs
from tests import parity
from tests.test_parity_gpu import _ragged_voxels, dev, env, run_fit, say  # noqa: F401

pytestmark = pytest.mark.gpu

STRIP_EDGES = [16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96, 97, 111, 112, 113, 127, 128, 129,
               143, 144, 145, 255, 256, 257, 271, 272, 273, 495, 496, 497, 511, 512]


@pytest.mark.parametrize("nq,frame_mode,fp32_last", [(1, 0, 0), (3, 0, 0), (5, 1, 0), (11, 0, 0), (8, 0, 3), (15, 1, 0)])
def test_strip_solver_edges(env, nq, frame_mode, fp32_last):  # noqa: F811
    torch, vgpr, ctx = env
    xyz = _ragged_voxels(31 + nq, STRIP_EDGES)
    w = dict(configs.params_for("spin32"), max_pts=512, min_pts=3, grid_side=nq, frame_mode=frame_mode)
    say("strip edges", nq, frame_mode, fp32_last)
    old = ctx.tuning()
    t = ctx.tuning()
    t.fp32_last_bucket = fp32_last
    ctx.set_tuning(t)
    try:
        _, (out, axis, status) = run_fit(env, xyz, w, precision=vgpr.PREC_FP32 if fp32_last else vgpr.PREC_FP64)
    finally:
        ctx.set_tuning(old)
    ov = O.voxelize(xyz, w["voxel_size"])
    cmp = parity.compare_fit_rotated if frame_mode else parity.compare_fit
    assert cmp(xyz, ov, parity.oracle_params(w), out, axis, status)["solved"] == len(STRIP_EDGES)


@pytest.mark.parametrize("n_vox", [8191, 8192, 32767, 32768, 32801])
def test_fit_voxel_count_rules(env, n_vox):  # noqa: F811
    torch, vgpr, ctx = env
    r = np.random.default_rng(n_vox)
    counts = r.integers(1, 9, n_vox)
    counts[r.choice(n_vox, 40, replace=False)] = r.choice([17, 40, 64, 65, 66, 100, 128, 129, 140], 40)
    side = int(np.ceil(np.sqrt(n_vox)))
    cell = np.stack([np.arange(n_vox) // side, np.arange(n_vox) % side, np.zeros(n_vox)], 1)
    xyz = (np.repeat(cell, counts, 0) + r.uniform(0.05, 0.95, (counts.sum(), 3)) * [1, 1, 0.2]) * 0.5
    w = dict(configs.params_for("spin32"), max_pts=130, min_pts=3, grid_side=4)
    say("voxel count rule", n_vox)
    x = dev(torch, xyz)
    p = parity.gpu_params(vgpr, w, precision=vgpr.PREC_FP32)
    v = ctx.voxelize(x, p)
    assert v.n_vox == n_vox
    whole = [t.cpu().numpy() for t in ctx.fit_predict(x, v, p)]
    for a in range(0, n_vox, 7000):
        b = min(a + 7000, n_vox)
        part = dataclasses.replace(v, keys=v.keys[a:b].contiguous(), offsets=v.offsets[a:b].contiguous(),
                                   counts=v.counts[a:b].contiguous(), n_vox=b - a)
        got = [t.cpu().numpy() for t in ctx.fit_predict(x, part, p)]
        for e, g in zip(whole, got):
            assert np.array_equal(e[a:b], g, equal_nan=e.dtype.kind == "f")


@pytest.mark.parametrize("nv", [1, 15, 63, 64, 65, 127, 128, 129, 1023, 1024, 1025])
def test_map_voxel_count_edges(env, nv):  # noqa: F811
    torch, vgpr, ctx = env
    w = dict(configs.params_for("paper_stream"), max_pts=20, min_pts=4)
    p = parity.gpu_params(vgpr, w)
    s = w["voxel_size"]
    om = O.VoxelMap(parity.oracle_params(w))
    gm = vgpr.Map(ctx, p, max_voxels=2 * nv)
    r = np.random.default_rng(nv)
    for k in range(3):  # half of a frame's voxels are new, counts run past max_pts
        first = k * (nv // 2)
        counts = r.integers(1, 24, nv)
        cell = np.stack([np.arange(first, first + nv) % 37, np.arange(first, first + nv) // 37, np.zeros(nv)], 1)
        xyz = (np.repeat(cell, counts, 0) + r.uniform(0.05, 0.95, (counts.sum(), 3)) * [1, 1, 0.2]) * s
        xyz = xyz[r.permutation(len(xyz))].astype(np.float32)
        say("map voxels", nv, k)
        keys, _, _, status = gm.update(dev(torch, xyz))
        ref = om.update(xyz)
        assert np.array_equal(parity.as_u64(keys), ref["keys"])
        both = O.ST_SOLVED | O.ST_CAPPED
        assert np.array_equal(status.cpu().numpy() & both, ref["status"] & both)
        assert gm.stats()["voxels"] == len(om.points)
        assert gm.stats()["points"] == sum(len(q) for q in om.points.values())


@pytest.mark.parametrize("n", [1, 3, 4, 5, 1023, 1025, 4097, 20000])
def test_loss_ring_edges(env, n):  # noqa: F811
    torch, vgpr, ctx = env
    r = np.random.default_rng(n)
    h = 0.05
    far = (2 ** 20 - 2) * h
    g = np.zeros((700, 8), np.float32)
    g[:, :3] = r.uniform(-1, 1, (700, 3)) * [1, 1, 2]  # about 80 cells along z, both signs
    g[:3, :3] = [[0, 0, far], [0, far, 0], [-far, 0, 0]]
    g[:, 4:7] = r.uniform(0.001, 0.02, (700, 3))
    pts = (r.uniform(-1.2, 1.2, (n, 3)) * [1, 1, 2]).astype(np.float32)
    pts[: n // 3] += np.float32(3.0)  # a run of points that no ring settles
    pts[-1] = [0.01, 0, far]
    say("loss rings", n)
    d = np.sqrt(((pts[:, None].astype(np.float64) - g[None, :, :3]) ** 2).sum(2))
    ref = (d - g[None, :, 4:7].mean(2)).min(1)
    got = {}
    for cell in (h, 0.5):
        loss, nv, val, arg = ctx.structure_loss(dev(torch, pts), dev(torch, g), cell, 0)
        got[cell] = (val.cpu().numpy(), arg.cpu().numpy())
        assert nv == n
        tol = 1e-6 * (1 + np.abs(pts).max(1))
        assert (np.abs(got[cell][0] - ref) <= tol).all()
        assert abs(loss - ref.mean()) <= tol.max()
    assert np.array_equal(got[h][0], got[0.5][0]) and np.array_equal(got[h][1], got[0.5][1])


def test_map_block_taken_again(env):  # noqa: F811
    """A map in a block that another map left behaves, and is exported, as one in a new block."""
    torch, vgpr, ctx = env
    w = dict(configs.params_for("paper_stream"), max_pts=20, min_pts=4)
    p = parity.gpu_params(vgpr, w)
    r = np.random.default_rng(3)
    a, b = (dev(torch, r.uniform(-3, 3, (n, 3)) * [1, 1, 0.1]) for n in (6000, 4000))

    def session(c, x, size, feedback):
        m = vgpr.Map(c, p, max_voxels=size, feedback=feedback)
        got = [t.cpu().numpy().copy() for t in m.update(x)] + [np.frombuffer(m.export(), np.uint8)]
        m.close()
        return got

    for feedback in (False, True):
        say("map block", feedback)
        own = vgpr.Context(0)
        held = own.workspace_bytes()
        session(own, a, 9000, feedback)
        again = session(own, b, 8000, feedback)  # in the first map's block
        assert own.workspace_bytes() - held < (1 << 30)
        fresh = vgpr.Context(0)
        for e, g in zip(session(fresh, b, 8000, feedback)[:4], again[:4]):
            assert np.array_equal(np.sort(e.ravel()), np.sort(g.ravel()), equal_nan=e.dtype.kind == "f")
        assert len(session(fresh, b, 8000, feedback)[4]) == len(again[4])
        own.close()
        fresh.close()


@pytest.mark.parametrize("n_vox", [1, 767, 768, 769, 3071, 3072, 3073, 6145, 9300])
def test_strip_voxels_at_a_stride(env, n_vox):  # noqa: F811
    """FP64 voxels of 17 to 32 points, fewer and more than the launch's wavefronts: every voxel is
    solved, as in calls on parts of them (bit for bit)."""
    torch, vgpr, ctx = env
    r = np.random.default_rng(n_vox)
    counts = r.integers(17, 33, n_vox)
    side = int(np.ceil(np.sqrt(n_vox)))
    cell = np.stack([np.arange(n_vox) // side, np.arange(n_vox) % side, np.zeros(n_vox)], 1)
    xyz = (np.repeat(cell, counts, 0) + r.uniform(0.05, 0.95, (counts.sum(), 3)) * [1, 1, 0.2]) * 0.5
    w = dict(configs.params_for("spin32"), max_pts=32, min_pts=3, grid_side=5)
    say("strip stride", n_vox)
    x = dev(torch, xyz)
    p = parity.gpu_params(vgpr, w, precision=vgpr.PREC_FP64)
    v = ctx.voxelize(x, p)
    assert v.n_vox == n_vox
    whole = [t.cpu().numpy() for t in ctx.fit_predict(x, v, p)]
    assert (whole[2] & vgpr.ST_SOLVED).all() and np.isfinite(whole[0]).all()
    for a in range(0, n_vox, 500):
        b = min(a + 500, n_vox)
        part = dataclasses.replace(v, keys=v.keys[a:b].contiguous(), offsets=v.offsets[a:b].contiguous(),
                                   counts=v.counts[a:b].contiguous(), n_vox=b - a)
        for e, g in zip(whole, [t.cpu().numpy() for t in ctx.fit_predict(x, part, p)]):
            assert np.array_equal(e[a:b], g)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n_vox,merge", [(255, 0), (256, 0), (257, 0), (400, 0), (400, 1)])
def test_largest_voxels_in_order(env, n_vox, merge, prec):  # noqa: F811
    """Voxels of 250 to 512 points, fewer and more than the largest solver's workgroups (the launch
    then takes the longest first): bit for bit as in calls on few of them."""
    torch, vgpr, ctx = env
    r = np.random.default_rng(n_vox)
    counts = r.integers(250, 520, n_vox)
    cell = np.stack([np.arange(n_vox) // 20, np.arange(n_vox) % 20, np.zeros(n_vox)], 1)
    xyz = (np.repeat(cell, counts, 0) + r.uniform(0.05, 0.95, (counts.sum(), 3)) * [1, 1, 0.2]) * 0.5
    w = dict(configs.params_for("spin32"), max_pts=512, min_pts=3, grid_side=6)
    p = parity.gpu_params(vgpr, w, precision={"fp64": vgpr.PREC_FP64, "mixed": vgpr.PREC_MIXED}[prec])
    say("largest voxels", n_vox, merge, prec)
    x = dev(torch, xyz)
    old, t = ctx.tuning(), ctx.tuning()
    t.tiled_merge = merge
    ctx.set_tuning(t)
    try:
        v = ctx.voxelize(x, p)
        whole = [a.cpu().numpy() for a in ctx.fit_predict(x, v, p)]
        assert v.n_vox == n_vox and (whole[2] & vgpr.ST_SOLVED).all()
        for a in range(0, n_vox, 97):
            b = min(a + 97, n_vox)
            part = dataclasses.replace(v, keys=v.keys[a:b].contiguous(), offsets=v.offsets[a:b].contiguous(),
                                       counts=v.counts[a:b].contiguous(), n_vox=b - a)
            for e, g in zip(whole, [c.cpu().numpy() for c in ctx.fit_predict(x, part, p)]):
                assert np.array_equal(e[a:b], g)
    finally:
        ctx.set_tuning(old)
