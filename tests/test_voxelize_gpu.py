"""GPU parity of vgpr_voxelize against the oracle at the edges of its kernels: tiles of the
sort (1,024, 4,096 and 6,144 elements, the rule's line at 2^18 points) and of the segmentation
(2,048 and 8,192), sort keys of one to eight passes, frames that are empty, end inside a tile or need
passes of their own, voxels longer than a tile, and batches without a usable point. Every
output is a whole number and has to be equal.
"""
import numpy as np
import pytest

from oracle import vgpr_oracle as O

pytestmark = pytest.mark.gpu

SIZES = [1, 63, 1023, 1024, 1025, 2047, 2048, 2049, 40000, 131072, 135169, 262143, 262144, 262145, 270337, 300000]


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2410_17084_amd import vgpr
    ctx = vgpr.Context(0)
    yield torch, vgpr, ctx
    torch.cuda.synchronize()
    ctx.close()


def check(env, xyz, offsets=None):
    torch, vgpr, ctx = env
    print("[case]", len(xyz), None if offsets is None else len(offsets) - 1, flush=True)
    p = vgpr.default_params(voxel_size=0.5)
    got = ctx.voxelize(torch.from_numpy(np.ascontiguousarray(xyz, dtype=np.float32)).cuda(), p, offsets)
    ref = O.voxelize(xyz, 0.5, offsets)
    assert got.n_vox == len(ref["keys"]) and got.n_invalid == ref["n_invalid"]
    assert np.array_equal(got.keys.cpu().numpy().view(np.uint64), ref["keys"])
    assert np.array_equal(got.offsets.cpu().numpy(), ref["offsets"])
    assert np.array_equal(got.counts.cpu().numpy(), ref["counts"])
    assert np.array_equal(got.perm.cpu().numpy(), ref["perm"])
    assert np.array_equal(np.asarray(got.frame_vox), ref["frame_vox"])


def cloud(r, n, extent, invalid=0.0):
    x = r.uniform(-1, 1, (n, 3)) * np.asarray(extent)
    x[r.random(n) < invalid] = np.nan
    return x.astype(np.float32)


@pytest.mark.parametrize("n", SIZES)
def test_tile_edges(env, n):
    r = np.random.default_rng(n)
    check(env, cloud(r, n, (40, 30, 3), 0.02))                       # three passes
    cuts = np.sort(r.integers(0, n + 1, 6))
    frames = np.concatenate([[0], cuts, cuts[-1:], [n, n]])          # two of them empty, one at the end
    check(env, cloud(r, n, (40, 30, 3), 0.02), frames)


@pytest.mark.parametrize("extent", [(0.1, 0.1, 0.1), (9, 0.1, 0.1), (1e3, 1e3, 30), (1e4, 1e4, 1e4), (5e5, 5e5, 5e5)])
def test_key_widths(env, extent):
    r = np.random.default_rng(5)
    for n in (5000, 270000):
        x = cloud(r, n, extent)
        x[: n // 2] = x[0]                                            # one voxel over many tiles
        check(env, x[r.permutation(n)])
        check(env, x, np.array([0, n // 3, n // 2, n // 2, n]))
    many = np.arange(0, 3001, 10)                                     # 300 frames: two passes for them at the widest
    check(env, cloud(r, 3000, extent, 0.3), many)


def test_no_usable_point(env):
    x = np.full((3000, 3), np.inf, np.float32)
    check(env, x)
    check(env, x, np.array([0, 1000, 3000]))
    x[2999] = 1.0
    check(env, x)
