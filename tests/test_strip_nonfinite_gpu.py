"""FP64 solves above 16 points with a value that is not finite among a voxel's points or noise
variances: the factorisation is reported as failed, the rows hold no numbers, and the voxels
that the same workgroups solve before and after are not touched (bit for bit)."""
import numpy as np
import pytest

from paper_2410_17084_amd import configs
from tests import parity
from tests.test_parity_gpu import dev, env, say  # noqa: F401

pytestmark = pytest.mark.gpu


# on both sides of strips and buckets, and whole strips, where the last pivot is the last point's
@pytest.mark.parametrize("n", [17, 32, 40, 64, 65, 96, 128, 130, 256, 300, 512])
@pytest.mark.parametrize("frame_mode", [0, 1])
def test_strip_solver_nonfinite_input(env, n, frame_mode):  # noqa: F811
    torch, vgpr, ctx = env
    nv = 1600 if n <= 64 else 200  # several voxels a workgroup with the smallest grids
    r = np.random.default_rng(n)
    s = 0.5
    cell = np.stack([np.arange(nv) // 40, np.arange(nv) % 40, np.zeros(nv, int)], 1)
    q = r.uniform(0.03, 0.97, (nv, n, 3))
    q[:, :, 2] = 0.4 + 0.2 * q[:, :, 0] + r.normal(0, 0.02, (nv, n))
    xyz = ((cell[:, None] + q) * s).astype(np.float32).reshape(-1, 3)
    noise = np.full(nv * n, 1e-3, np.float32)
    key = (((cell[:, 0] + 2 ** 20) << 42) | ((cell[:, 1] + 2 ** 20) << 21) | (cell[:, 2] + 2 ** 20)).astype(np.int64)
    cuda = lambda a, t: torch.from_numpy(np.ascontiguousarray(a, t)).cuda()  # noqa: E731
    vox = vgpr.Voxels(cuda(key, np.int64), cuda(np.arange(nv) * n, np.int32), cuda(np.full(nv, n), np.int32), None,
                      nv, [0, nv], 0)
    w = dict(configs.params_for("spin32"), max_pts=512, min_pts=3, grid_side=5, frame_mode=frame_mode)
    p = parity.gpu_params(vgpr, w, precision=vgpr.PREC_FP64)
    old, t = ctx.tuning(), ctx.tuning()
    for b in range(7):
        t.grid_scale[b] = 1
    say("strip nonfinite", n, frame_mode)

    def fit():
        return [a.cpu().numpy() for a in ctx.fit_predict(dev(torch, xyz), vox, p, noise_var=dev(torch, noise))]

    ctx.set_tuning(t)
    try:
        good = fit()
        bad = r.choice(nv, nv // 3, replace=False)
        for k, v in enumerate(bad):
            at = v * n + [0, n - 1, int(r.integers(n))][k % 3]
            kind = k // 3 % 5
            if kind < 3:
                xyz[at, kind] = [np.nan, np.inf, -np.inf][k // 15 % 3]
            else:
                noise[at] = [np.inf, np.nan][kind - 3]
        got = fit()
    finally:
        ctx.set_tuning(old)
    assert (good[2] & vgpr.ST_SOLVED).all()
    ok = np.setdiff1d(np.arange(nv), bad)
    for e, g in zip(good, got):
        assert np.array_equal(e[ok], g[ok])
    assert (got[2][bad] == vgpr.ST_FACTOR_FAIL | (got[2][bad] & vgpr.ST_AXIS_TIE)).all()
    assert np.isnan(got[0][bad, :, 3]).all() and np.isnan(got[0][bad]).any(2).all()
    finite_points = bad[np.isfinite(xyz.reshape(nv, n, 3)[bad]).all((1, 2))]
    value = np.take_along_axis(got[0][finite_points], got[1][finite_points, None, None].astype(int), 2)
    if frame_mode == 0:
        assert np.isnan(value).all()
