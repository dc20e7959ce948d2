"""The colour head's backward at the edges of its tile pipeline and on its general input path (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from parity import GRAD, close  # noqa: E402

pytestmark = pytest.mark.gpu


# 256 blocks of 32-sample tiles: the last block count at which every block has one tile, blocks with one tile
# beside blocks with two, three tiles, and 65 (the first rays of a block's tiles are read 64 at a time)
@pytest.mark.parametrize("S,longest", [(1, 1), (32, 5), (33, 40), (8192, 3), (8193, 60), (16384 + 31, 9),
                                       (24576 + 8192 * 62, 200)])
def test_head_backward_pipeline(S, longest):
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(S + longest)
    lengths = []
    while sum(lengths) < S:
        lengths.append(min(int(rng.integers(0, longest + 1)), S - sum(lengths)) if S < 1e5 else longest)
        if lengths[-1] == 0 and rng.random() < 0.5:
            lengths += [0] * 70  # beyond the 64-entry window of ray starts
    lengths[-1] -= sum(lengths) - S
    offs = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    R = len(lengths)
    mlp = synth.mlp_weights(rng, bias_std=0.3)
    dirs = synth.scenes._unit(rng.standard_normal((R, 3))).astype(np.float32)
    feat = rng.standard_normal((S, 12)).astype(np.float32)
    grgb = (rng.standard_normal((S, 3)) * 10.0 ** rng.uniform(-4, 1, (S, 1))).astype(np.float32)
    print(f"[case] head backward S={S} R={R}", flush=True)

    def dev(x, dt=torch.float32, shift=0):
        x = torch.as_tensor(x).to("cuda", dt).contiguous()
        buf = torch.empty(x.numel() + shift, dtype=dt, device="cuda")
        out = buf[shift:].view(x.shape)
        out.copy_(x)
        return out

    W, b = [dev(w) for w in mlp.W], [dev(v) for v in mlp.b]

    def run(shift):
        gW, gb = [torch.zeros_like(w) for w in W], [torch.zeros_like(v) for v in b]
        P = ops.MLPParams(W, b, gW, gb)
        gf = ops.mlp_backward(P, dev(offs, torch.int32), dev(dirs), dev(feat, shift=shift), dev(grgb))
        torch.cuda.synchronize()
        return [gf] + gW + gb

    got = run(0)
    # features off the 16-byte grid take the general loads and stores: the same arithmetic, so the same bits
    for x, y in zip(got, run(1)):
        assert torch.equal(x, y)
    if S > 20000:
        return  # the oracle's comparison at this length is that of the full-size workloads
    f64, g64 = feat.astype(np.float64), grgb.astype(np.float64)
    rgf, rgW, rgb = oracle.mlp_backward(mlp, offs, dirs, f64, g64)
    sf, sW, sb = oracle.mlp_kink_slack(mlp, offs, dirs, f64, g64, thr=1e-5)
    close(got[0].cpu().numpy(), rgf, **GRAD, name="d feat", slack=sf)
    for i in range(3):
        close(got[1 + i].cpu().numpy(), rgW[i], **GRAD, name=f"dW{i + 1}", slack=sW[i])
        close(got[4 + i].cpu().numpy(), rgb[i], **GRAD, name=f"db{i + 1}", slack=sb[i])
