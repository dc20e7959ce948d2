"""The dense total-variation update that walks columns along x, at the edges of its walks (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(2, 2, 2, 4), (3, 2, 5, 8), (4, 3, 70, 12), (5, 33, 2, 16), (9, 17, 19, 4),
                                   (130, 6, 5, 12), (7, 24, 31, 12)])
@pytest.mark.parametrize("delta", [0.3, 1e30])
def test_dense_tv(shape, delta):
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(sum(shape))
    v = rng.standard_normal(shape).astype(np.float32)
    g = (1e-3 * rng.standard_normal(shape)).astype(np.float32)
    g[rng.random(shape[:3]) < 0.5] = 0.0
    weight = 0.05
    coef = 2.0 * weight / v.size
    print(f"[case] dense tv {shape} delta {delta}", flush=True)
    p, q = torch.as_tensor(v).cuda(), torch.as_tensor(g).cuda()
    ops.tv_add_grad(ops.DeviceGrid(p, (-1.0,) * 3, (1.0,) * 3, grad=q), weight, delta, True)
    torch.cuda.synchronize()
    d = v.astype(np.float64)
    total, mag = np.zeros(shape), np.zeros(shape)
    for a in range(3):
        lo, hi = [slice(None)] * 4, [slice(None)] * 4
        lo[a], hi[a] = slice(0, -1), slice(1, None)
        step = np.clip(d[tuple(lo)] - d[tuple(hi)], -delta, delta)
        total[tuple(lo)] += step
        total[tuple(hi)] -= step
        mag[tuple(lo)] += np.abs(step)
        mag[tuple(hi)] += np.abs(step)
    # six differences, five sums, the coefficient (rounded once), a product and a sum, each within 2^-24
    bound = 16 * 2.0 ** -24 * (np.abs(g) + coef * mag)
    assert (np.abs(q.cpu().numpy() - (g + coef * total)) <= bound).all()
