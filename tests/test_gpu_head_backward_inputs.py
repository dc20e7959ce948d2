"""The colour head's backward over its input widths and over many tiles a block, against 64 bits (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from parity import GRAD, close  # noqa: E402
from test_gpu_parity import GRAD16  # noqa: E402

pytestmark = pytest.mark.gpu


def _dev(x, dt=torch.float32):
    return torch.as_tensor(x).to("cuda", dt).contiguous()


def _batch(rng, lengths, C, F):
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    R, S = len(lengths), int(offs[-1])
    mlp = synth.mlp_weights(rng, C, n_freq=F, bias_std=0.3)
    dirs = synth.scenes._unit(rng.standard_normal((R, 3))).astype(np.float32)
    feat = rng.standard_normal((S, C)).astype(np.float32)
    grgb = (rng.standard_normal((S, 3)) * 10.0 ** rng.uniform(-4, 1, (S, 1))).astype(np.float32)
    return mlp, offs, dirs, feat, grgb


def _run(mlp, offs, dirs, feat, grgb, F, half=False):
    from paper_2206_05085_amd import ops
    W, b = [_dev(w) for w in mlp.W], [_dev(v) for v in mlp.b]
    gW, gb = [torch.zeros_like(w) for w in W], [torch.zeros_like(v) for v in b]
    P = ops.MLPParams(W, b, gW, gb, in_feat=feat.shape[1], n_freq=F, precision=ops.MLP_F16 if half else ops.MLP_SPLIT_F16)
    gf = ops.mlp_backward(P, _dev(offs, torch.int32), _dev(dirs), _dev(feat), _dev(grgb))
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in [gf] + gW + gb]


def _exact(mlp, offs, dirs, feat, grgb, F):
    """Gradients in float64, and how far each moves if the ReLU units within rounding (1e-5 of the magnitude of
    their sums) of zero take the other side: (feat, W1..W3, b1..b3) and the same for the slack."""
    f64 = torch.float64
    ray = torch.repeat_interleave(torch.arange(len(offs) - 1, device="cuda"), _dev(np.diff(offs), torch.int64))
    d = _dev(dirs, f64)
    t = torch.cat([d * 2.0 ** k for k in range(F)] or [d[:, :0]], 1)
    x = torch.cat([_dev(feat, f64), torch.cat([d, t.sin(), t.cos()], 1)[ray]], 1)
    (W1, W2, W3), (b1, b2, b3) = [_dev(w, f64) for w in mlp.W], [_dev(v, f64) for v in mlp.b]
    z1 = x @ W1.T + b1
    a1 = z1.abs() <= 1e-5 * (x.abs() @ W1.abs().T + b1.abs())
    h1 = z1.relu()
    z2 = h1 @ W2.T + b2
    a2 = z2.abs() <= 1e-5 * (h1 @ W2.abs().T + b2.abs())
    h2 = z2.relu()
    y = (h2 @ W3.T + b3).sigmoid()
    d3 = _dev(grgb, f64) * y * (1 - y)
    u2 = d3 @ W3
    d2 = u2 * (z2 > 0)
    u1 = d2 @ W2
    d1 = u1 * (z1 > 0)
    s2 = u2.abs() * a2
    s1 = u1.abs() * a1 + s2 @ W2.abs()
    C = feat.shape[1]
    grads = [d1 @ W1[:, :C], d1.T @ x, d2.T @ h1, d3.T @ h2, d1.sum(0), d2.sum(0), d3.sum(0)]
    slack = [s1 @ W1[:, :C].abs(), s1.T @ x.abs(), s2.T @ h1, 0 * W3, s1.sum(0), s2.sum(0), 0 * b3]
    return [[t.cpu().numpy() for t in v] for v in (grads, slack)]


NAMES = ["d feat", "dW1", "dW2", "dW3", "db1", "db2", "db3"]


# one tile, the edges of the ray window's refresh (64 tiles a block), and past it; rays of many lengths there,
# so that a wrong first ray of a tile gives a wrong view encoding
@pytest.mark.parametrize("tiles", [1, 2, 63, 64, 65, 66, 130])
def test_many_tiles_per_block(tiles):
    rng = np.random.default_rng(tiles)
    S = 256 * 32 * tiles - 5
    lengths = rng.integers(0, 400, S // 190)
    lengths = np.append(lengths[np.cumsum(lengths) < S], 0)
    lengths[-1] = S - lengths[:-1].sum()
    print(f"[case] head backward, {tiles} tiles a block, S={S} R={len(lengths)}", flush=True)
    case = _batch(rng, lengths, 12, 4)
    got, (want, slack) = _run(*case, 4), _exact(*case, 4)
    for x, y, s, name in zip(got, want, slack, NAMES):
        close(x, y, **GRAD, name=name, slack=s)


LENGTHS = [0, 5, 1, 64, 100, 0, 130] + [0] * 70 + [3] * 40 + [200, 31]


@pytest.mark.parametrize("C", [1, 4, 5, 8, 11, 12])
@pytest.mark.parametrize("F", [0, 1, 2, 3, 4])
def test_input_widths(C, F):
    rng = np.random.default_rng(10 * C + F)
    print(f"[case] head backward C={C} F={F}", flush=True)
    case = _batch(rng, LENGTHS, C, F)
    got, (want, slack) = _run(*case, F), _exact(*case, F)
    for x, y, s, name in zip(got, want, slack, NAMES):
        close(x, y, **GRAD, name=name, slack=s)


@pytest.mark.parametrize("C,F", [(1, 2), (4, 4), (5, 0), (8, 3), (11, 1), (12, 2)])
def test_input_widths_half(C, F):
    rng = np.random.default_rng(10 * C + F)
    print(f"[case] FP16 head backward C={C} F={F}", flush=True)
    mlp, offs, dirs, feat, grgb = _batch(rng, LENGTHS, C, F)
    got = _run(mlp, offs, dirs, feat, grgb, F, half=True)
    args = (mlp, offs, dirs, feat.astype(np.float64), grgb.astype(np.float64))
    rf, rW, rb = oracle.mlp_backward(*args, F=F, half=True)
    sf, sW, sb = oracle.mlp_kink_slack(*args, thr=1e-4, F=F, half=True)
    _, mf, mW, mb = oracle.mlp_magnitudes(*args, F=F, half=True)
    for x, y, s, m, name in zip(got, [rf, *rW, *rb], [sf, *sW, *sb], [mf, *mW, *mb], NAMES):
        close(x, y, **GRAD16, name=name, slack=s, scale=m)
