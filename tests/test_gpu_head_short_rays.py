"""The colour head on batches of many rays with few samples each, which have no bias rows (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from parity import FWD, close  # noqa: E402
from test_gpu_parity import FWD16  # noqa: E402

pytestmark = pytest.mark.gpu


def _dev(x, dt=torch.float32):
    return torch.as_tensor(x).to("cuda", dt).contiguous()


def _exact(mlp, ray, dirs, feat, F):
    """The head in float64 and the magnitude its logits' sums are conditioned on."""
    d = dirs.double()
    t = torch.cat([d * 2.0 ** k for k in range(F)] or [d[:, :0]], 1)
    x = torch.cat([feat.double(), torch.cat([d, t.sin(), t.cos()], 1)[ray]], 1)
    a = x.abs()
    for i in range(3):
        W, b = (_dev(v, torch.float64) for v in (mlp.W[i], mlp.b[i]))
        x, a = x @ W.T + b, a @ W.abs().T + b.abs()
        x = x.relu() if i < 2 else x
    y = x.sigmoid()
    return y, a * y * (1 - y)


# around the rule: 8,192 rays, and 24 samples a ray of more rays
@pytest.mark.parametrize("R,S,C,F", [(9001, 18003, 12, 4), (9001, 2500, 12, 4), (20011, 20011, 12, 3), (9001, 9001, 4, 2),
                                     (9001, 30000, 5, 1), (9001, 18003, 11, 0), (8192, 8192, 12, 4), (8193, 8193, 12, 4),
                                     (8193, 24 * 8193, 12, 4), (8193, 24 * 8193 - 1, 12, 4)])
@pytest.mark.parametrize("half", [False, True])
def test_head_of_short_rays(R, S, C, F, half):
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(R + S)
    lengths = np.full(R, S // R) if S % R == 0 else np.bincount(rng.integers(0, R, S), minlength=R)
    offs = _dev(np.concatenate([[0], np.cumsum(lengths)]), torch.int32)
    ray = _dev(np.repeat(np.arange(R), lengths), torch.int64)
    mlp = synth.mlp_weights(rng, C, n_freq=F, bias_std=0.3)
    dirs = _dev(synth.scenes._unit(rng.standard_normal((R, 3))))
    n = 16
    grid = ops.DeviceGrid(_dev(rng.standard_normal((n, n, n, C))), (-1.0,) * 3, (1.0,) * 3)
    xyz = _dev(rng.uniform(-1, 1, (S, 3)))
    feat = ops.grid_gather(grid, xyz)
    W, b = [_dev(w) for w in mlp.W], [_dev(v) for v in mlp.b]
    gW, gb = [torch.zeros_like(w) for w in W], [torch.zeros_like(v) for v in b]
    P = ops.MLPParams(W, b, gW, gb, in_feat=C, n_freq=F, precision=ops.MLP_F16 if half else ops.MLP_SPLIT_F16)
    print(f"[case] short rays R={R} S={S} C={C} F={F} half={half}", flush=True)
    rgb = ops.mlp_forward(P, offs, dirs, feat)
    want, mag = _exact(mlp, ray, dirs, feat, F)
    torch.cuda.synchronize()
    close(rgb.cpu().numpy(), want.cpu().numpy(), **(FWD16 if half else FWD), name="rgb", scale=mag.cpu().numpy())
    # any call's preparation serves the others, and the fused lookup sees the same features
    ws = torch.empty(ops.mlp_workspace_size(P, R, S), dtype=torch.uint8, device="cuda")
    ops.mlp_backward(P, offs, dirs, feat, torch.ones_like(rgb), ws=ws)
    assert torch.equal(rgb, ops.mlp_forward(P, offs, dirs, feat, ws=ws, prepared=True))
    if C % 4 == 0:
        assert torch.equal(rgb, ops.mlp_forward_gather(P, offs, dirs, grid, xyz, ws=ws, prepared=True))
