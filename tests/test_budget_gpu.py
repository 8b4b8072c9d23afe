"""Calls that just fit an HBM budget: their scratch has not grown, and the results are those
without a budget."""
import numpy as np
import pytest

from paper_2410_17084_amd import configs
from tests import parity
from tests.test_parity_gpu import dev, env, say  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,frames", [(40000, 1), (100003, 1), (100003, 9), (262144, 1), (262145, 1), (500000, 3)])
def test_voxelize_in_21_bytes_a_point(env, n, frames):  # noqa: F811
    torch, vgpr, ctx = env
    r = np.random.default_rng(n + frames)
    x = dev(torch, r.uniform(-30, 30, (n, 3)) * [1, 1, 0.1])
    p = parity.gpu_params(vgpr, configs.params_for("spin32"))
    fo = [n * f // frames for f in range(frames + 1)]
    say("voxelize budget", n, frames)
    for scale in (1.0, 200.0):  # sort keys of 32 bits and of more
        tight = vgpr.Context(0, hbm_budget=int(21.1 * n))
        a, b = (c.voxelize(x * scale, p, frame_offsets=fo) for c in (tight, ctx))
        assert tight.workspace_bytes() <= int(21.1 * n)
        assert a.n_vox == b.n_vox and a.frame_vox == b.frame_vox
        for f in ("keys", "offsets", "counts", "perm"):
            assert torch.equal(getattr(a, f), getattr(b, f)), f
        tight.close()


def test_structure_loss_of_few_points(env):  # noqa: F811
    torch, vgpr, ctx = env
    r = np.random.default_rng(4)
    g = np.zeros((1000, 8), np.float32)
    g[:, :3] = r.uniform(-2, 2, (1000, 3))
    g[:, 4:7] = 0.01
    x, g = dev(torch, r.uniform(-2, 2, (1000, 3))), dev(torch, g)
    say("loss budget")
    tight = vgpr.Context(0, hbm_budget=1262016)  # about 170 bytes a Gaussian, 12 a point and 1.1 MB
    a, b = (c.structure_loss(x, g, 0.2) for c in (tight, ctx))
    assert a[:2] == b[:2] and torch.equal(a[2], b[2]) and torch.equal(a[3], b[3])
    tight.close()
