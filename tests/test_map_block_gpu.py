"""Memory of destroyed maps, taken again by the context's next map."""
import struct

import numpy as np
import pytest

from paper_2410_17084_amd import configs
from tests import parity
from tests.test_parity_gpu import dev, env, say  # noqa: F401

pytestmark = pytest.mark.gpu


def _params(vgpr):
    return parity.gpu_params(vgpr, dict(configs.params_for("paper_stream"), max_pts=20, min_pts=4))


def _records(params, data):
    """An export's voxels by key: (stored, total, converged, has rows, stored points, rows)."""
    mode, = struct.unpack_from("<i", data, 12)
    nv, = struct.unpack_from("<q", data, 16)
    cap, m = params.max_pts, params.grid_side ** 2
    at = len(data) - nv * (8 + 4 + 4 + 1 + mode + 12 * cap + 16 * m * mode)
    out = []
    for dtype, width in ((np.uint64, 1), (np.int32, 1), (np.int32, 1), (np.uint8, 1), (np.uint8, mode),
                         (np.float32, 3 * cap), (np.float32, 4 * m * mode)):
        out.append(np.frombuffer(data, dtype, nv * width, at).reshape(nv, width))
        at += out[-1].nbytes
    assert at == len(data)
    key, stored, total, conv, pred, pool, rows = out
    return {int(key[v, 0]): (int(stored[v, 0]), int(total[v, 0]), int(conv[v, 0]), pred[v].tolist(),
                             pool[v, :3 * stored[v, 0]].tobytes(), rows[v].tobytes() if pred[v].any() else b"")
            for v in range(nv)}


def _session(vgpr, ctx, params, frames, size, feedback):
    m = vgpr.Map(ctx, params, max_voxels=size, feedback=feedback)
    got = []
    for x in frames:
        got += [t.cpu().numpy().copy() for t in m.update(x)]
    got.append(_records(params, m.export()))
    m.close()
    return got


def _same(a, b):
    return len(a) == len(b) and all(
        e == g if isinstance(e, dict) else np.array_equal(e, g, equal_nan=e.dtype.kind == "f") for e, g in zip(a, b))


def _frames(torch, seed, n, k):
    r = np.random.default_rng(seed)
    return [dev(torch, r.uniform(-3, 3, (n, 3)) * [1, 1, 0.1]) for _ in range(k)]


@pytest.mark.parametrize("feedback", [False, True])
def test_map_closed_on_another_stream(env, feedback):  # noqa: F811
    """A map whose last update ran on one stream, closed with the context on another: the next map,
    on the other stream, holds what it holds in a context of its own."""
    torch, vgpr, _ = env
    p = _params(vgpr)
    before, after = _frames(torch, 5, 60000, 2), _frames(torch, 6, 5000, 3)
    say("map closed on another stream", feedback)
    fresh = vgpr.Context(0)
    expect = _session(vgpr, fresh, p, after, 8000, feedback)
    fresh.close()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s1):
        ctx = vgpr.Context(0)
        for k in range(4):
            ctx.set_stream(s1)
            with torch.cuda.stream(s1):
                m = vgpr.Map(ctx, p, max_voxels=8000, feedback=feedback)
                kept = [m.update(x) for x in before]
            ctx.set_stream(s2)
            m.close()
            with torch.cuda.stream(s2):
                got = _session(vgpr, ctx, p, after, 8000, feedback)
            assert _same(expect, got), k
            del kept
            torch.cuda.synchronize()
        ctx.close()


@pytest.mark.parametrize("feedback", [False, True])
def test_map_in_a_kept_block(env, feedback):  # noqa: F811
    """Two sessions of several updates in one context, the second in the first's (larger) block: what
    the second returns and exports equals a new context's, voxel by voxel."""
    torch, vgpr, _ = env
    p = _params(vgpr)
    say("map in a kept block", feedback)
    first, second = _frames(torch, 7, 9000, 4), _frames(torch, 8, 5000, 4)
    fresh = vgpr.Context(0)
    expect = _session(vgpr, fresh, p, second, 6000, feedback)
    fresh.close()
    ctx = vgpr.Context(0)
    _session(vgpr, ctx, p, first, 9000, feedback)
    held = ctx.workspace_bytes()
    m = vgpr.Map(ctx, p, max_voxels=6000, feedback=feedback)
    assert ctx.workspace_bytes() == held  # the map is in the kept block
    m.close()
    assert _same(expect, _session(vgpr, ctx, p, second, 6000, feedback))
    assert ctx.workspace_bytes() == held
    ctx.close()


def test_kept_blocks_are_counted_and_bounded(env):  # noqa: F811
    torch, vgpr, _ = env
    p = _params(vgpr)
    say("kept blocks")
    ctxs = [vgpr.Context(0) for _ in range(4)]
    none = [c.workspace_bytes() for c in ctxs]
    free = torch.cuda.mem_get_info()[0]
    for c in ctxs:  # about 200 MB each
        vgpr.Map(c, p, max_voxels=600000).close()
    kept = [c.workspace_bytes() - b for c, b in zip(ctxs, none)]
    assert kept[0] > (128 << 20) and sum(kept) <= (512 << 20)
    assert free - torch.cuda.mem_get_info()[0] <= sum(kept) + (64 << 20)
    # a map that would leave most of the block unused does not keep it from the others
    vgpr.Map(ctxs[0], p, max_voxels=1000).close()
    assert ctxs[0].workspace_bytes() - none[0] < (8 << 20)
    # one that does not fit takes its place
    vgpr.Map(ctxs[0], p, max_voxels=20000).close()
    small = ctxs[0].workspace_bytes()
    m = vgpr.Map(ctxs[0], p, max_voxels=20000)
    assert ctxs[0].workspace_bytes() == small
    m.close()
    # over the bound, and with an HBM budget, nothing is kept
    m = vgpr.Map(ctxs[3], p, max_voxels=2000000)
    assert ctxs[3].workspace_bytes() - none[3] > (512 << 20)
    m.close()
    assert ctxs[3].workspace_bytes() == none[3]
    own = vgpr.Context(0, hbm_budget=1 << 30)
    vgpr.Map(own, p, max_voxels=1000).close()
    assert own.workspace_bytes() == 0
    own.close()
    for c in ctxs:
        c.close()
