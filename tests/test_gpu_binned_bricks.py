"""The brick-binned scatter: channel counts, contractions, light and crowded bricks, points on their faces (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from parity import GRAD, close  # noqa: E402

pytestmark = pytest.mark.gpu


def _scene(rng, n, C, warp, b):
    """A grid and points: scattered ones, a crowd of 3000 in a few bricks, and points on vertices, thus on the
    faces between bricks; for a contraction world points, of all three kinds, out to 1000."""
    lim = 1.0 + b if warp else 1.0
    g = synth.normal_grid(rng, n, C, -lim, lim)
    g.warp, g.warp_b = warp, b
    faces = (rng.integers(0, n, (1500, 3)) / (n - 1) * 2 - 1) * lim
    xyz = np.concatenate([rng.uniform(-1.1, 1.1, (4000, 3)) * lim, 0.3 + 0.05 * rng.standard_normal((3000, 3)), faces])
    if warp:
        d = rng.standard_normal((4000, 3))
        far = d / np.abs(d).max(1, keepdims=True) * 10.0 ** rng.uniform(-1.0, 3.0, (4000, 1))
        # the crowd once more, seen through the contraction: a cone far outside
        xyz = np.concatenate([xyz, far, (np.float64([0.9, 0.2, -0.4]) + 0.01 * rng.standard_normal((2000, 3))) * 40.0])
    return g, xyz.astype(np.float32)


@pytest.mark.parametrize("n", [20, 49, 70])           # 27, 216 and 729 bricks
@pytest.mark.parametrize("C,cs", [(1, 1), (1, 3), (2, 2), (3, 3), (3, 4), (4, 4), (5, 5)])
@pytest.mark.parametrize("warp,b", [(0, 1.0), (1, 1.0), (1, 0.4), (2, 1.0), (2, 2.5)])
def test_binned_bricks(n, C, cs, warp, b):
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(100 * n + 10 * C + warp)
    g, xyz = _scene(rng, n, C, warp, b)
    S = xyz.shape[0]
    y = rng.standard_normal((S, C)).astype(np.float32)
    y[::97] = 0.0
    print(f"[case] binned bricks n={n} C={C} cs={cs} warp={warp} b={b}", flush=True)
    data = np.zeros((n, n, n, cs), np.float32)
    before = rng.standard_normal(data.shape).astype(np.float32)
    dg = ops.DeviceGrid(torch.from_numpy(data).cuda(), g.xyz_min, g.xyz_max, grad=torch.from_numpy(before.copy()).cuda(),
                        channels=C, warp=warp, warp_b=b)
    t = torch.from_numpy(xyz).cuda()
    ws = ops.bin_samples(dg, t)
    ops.grid_scatter_binned(dg, t, torch.from_numpy(y).cuda(), ws)
    torch.cuda.synchronize()
    got = dg.grad.cpu().numpy()
    want = oracle.scatter(g, xyz, y.astype(np.float64)).reshape(n, n, n, C)
    close(got[..., :C], before[..., :C].astype(np.float64) + want, **GRAD, name="binned scatter")
    assert np.array_equal(got[..., C:], before[..., C:])
