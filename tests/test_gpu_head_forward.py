"""The colour head's forward at the edges of its tiles, ray windows and input groups (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from parity import FWD, close  # noqa: E402

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lengths,C,F", [
    ([1], 12, 4), ([31], 12, 4), ([32], 12, 4), ([33], 12, 4), ([0, 0, 5, 0], 12, 4),
    ([1] * 200, 12, 4),                      # 32 rays start in a tile
    ([3] + [0] * 100 + [60], 12, 4),         # a tile whose rays lie beyond the 64-entry window
    ([0] * 62 + [16, 16] + [0] * 70 + [1, 40], 12, 4),
    ([40, 7], 1, 0), ([40, 7], 4, 2), ([40, 7], 5, 1), ([40, 7], 8, 3), ([40, 7], 11, 4)])
def test_head_forward_edges(lengths, C, F):
    # directions that are not unit vectors and large biases move the bound that scales layer 1's output
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(len(lengths) + 100 * C + F)
    mlp = synth.mlp_weights(rng, C, n_freq=F, bias_std=1.0)
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    S, R = int(offs[-1]), len(lengths)
    dirs = (1.5 * rng.standard_normal((R, 3))).astype(np.float32)
    feat = (rng.standard_normal((S, C)) * 10.0 ** rng.uniform(-3, 0.5, (S, 1))).astype(np.float32)
    print(f"[case] head forward S={S} R={R} C={C} F={F}", flush=True)

    def dev(x, dt=torch.float32):
        return torch.as_tensor(x).to("cuda", dt).contiguous()

    P = ops.MLPParams([dev(w) for w in mlp.W], [dev(v) for v in mlp.b], in_feat=C, n_freq=F)
    got = ops.mlp_forward(P, dev(offs, torch.int32), dev(dirs), dev(feat))
    torch.cuda.synchronize()
    ref = oracle.mlp_forward(mlp, offs, dirs, feat.astype(np.float64), F=F)
    # elementwise against the magnitude each colour is conditioned on (the head over absolute values)
    mag = oracle.mlp_magnitudes(mlp, offs, dirs, feat.astype(np.float64), np.zeros((S, 3)), F=F)[0]
    close(got.cpu().numpy(), ref, **FWD, name="rgb", scale=mag)
