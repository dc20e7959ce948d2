"""The scatter's slot walk at the edges of its rounds, runs and channel groups (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from parity import GRAD, close  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,cs", [(1, 1), (1, 5), (2, 2), (3, 4), (4, 4), (6, 6), (8, 8), (11, 12), (12, 12), (16, 16)])
@pytest.mark.parametrize("S", [1, 7, 8, 61, 1023, 4097, 140001])
def test_slot_walk_edges(C, cs, S):
    # points along jittered lines (shared vertices, both directions along each axis), with jumps; padded
    # rows keep their padding.  float32 sums of at most a few thousand terms against the FP64 oracle.
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(1000 * C + S)
    n = 21
    g = synth.normal_grid(rng, n, C)
    t = np.arange(S)[:, None]
    step = rng.uniform(-0.06, 0.06, (S // 37 + 1, 3))[t[:, 0] // 37]
    start = rng.uniform(-1.1, 1.1, (S // 37 + 1, 3))[t[:, 0] // 37]
    xyz = (start + step * (t % 37)).astype(np.float32)
    y = rng.standard_normal((S, C)).astype(np.float32)
    y[S // 3: S // 3 + 40] = 0.0
    print(f"[case] slot walk C={C} cs={cs} S={S}", flush=True)
    data = np.zeros((n, n, n, cs), np.float32)
    data[..., :C] = g.data
    before = rng.standard_normal(data.shape).astype(np.float32)
    grad = torch.from_numpy(before.copy()).cuda()
    dg = ops.DeviceGrid(torch.from_numpy(data).cuda(), g.xyz_min, g.xyz_max, grad=grad, channels=C)
    ops.grid_scatter(dg, torch.from_numpy(xyz).cuda(), torch.from_numpy(y).cuda())
    torch.cuda.synchronize()
    got = grad.cpu().numpy()
    want = before[..., :C].astype(np.float64) + oracle.scatter(g, xyz, y.astype(np.float64)).reshape(n, n, n, C)
    close(got[..., :C], want, **GRAD, name="scatter")
    assert np.array_equal(got[..., C:], before[..., C:])


@pytest.mark.parametrize("n,S,crowd", [(9, 64, 0), (9, 65, 0), (40, 3000, 0), (40, 3000, 2500), (180, 20001, 6000)])
def test_binned_scatter_crowded_bricks(n, S, crowd):
    # bricks of at most 64 samples (one wave, global atomics) beside crowded ones (the block's LDS tile),
    # one and several bricks per block, more than one block of the prefix sum (180^3: 12,167 bricks)
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(n + S)
    g = synth.normal_grid(rng, n, 1)
    xyz = rng.uniform(-1.05, 1.05, (S, 3)).astype(np.float32)
    if crowd:
        xyz[:crowd] = (0.31 + 0.0007 * np.arange(crowd)[:, None] * rng.uniform(-0.1, 0.1, 3)).astype(np.float32)
    y = rng.standard_normal((S, 1)).astype(np.float32)
    print(f"[case] crowded bricks n={n} S={S} crowd={crowd}", flush=True)
    dg = ops.DeviceGrid(torch.from_numpy(g.data).cuda(), g.xyz_min, g.xyz_max,
                        grad=torch.zeros(n, n, n, 1, device="cuda"))
    t = torch.from_numpy(xyz).cuda()
    ws = ops.bin_samples(dg, t)
    for _ in range(2):  # the bins serve several scatters
        ops.grid_scatter_binned(dg, t, torch.from_numpy(y).cuda(), ws)
    torch.cuda.synchronize()
    close(dg.grad.cpu().numpy(), 2.0 * oracle.scatter(g, xyz, y.astype(np.float64)), **GRAD, name="binned scatter")
