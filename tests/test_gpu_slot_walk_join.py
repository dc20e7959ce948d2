"""Slot walks whose groups end on the same vertices and join their sums (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle  # noqa: E402
import synth  # noqa: E402
from parity import GRAD, close  # noqa: E402

pytestmark = pytest.mark.gpu


def _points(rng, kind, S):
    """one: every point in one cell; halves: two cells, changing within a wave; alternate: neighbouring groups
    in different cells; behind: lines that have left the box and stay in the cells of its faces"""
    at = np.float32([[0.31, -0.42, 0.13], [-0.55, 0.2, 0.7]])
    k = np.arange(S)
    which = {"one": 0 * k, "halves": k * 2 // max(S, 1), "alternate": k // 8 % 2}.get(kind)
    if which is None:
        return (rng.uniform(-1, 1, (S // 100 + 1, 3))[k // 100] + (k % 100)[:, None] * rng.uniform(-0.2, 0.2, (S // 100 + 1, 3))[k // 100]).astype(np.float32)
    return (at[which] + rng.uniform(-0.01, 0.01, (S, 3))).astype(np.float32)


@pytest.mark.parametrize("kind", ["one", "halves", "alternate", "behind"])
@pytest.mark.parametrize("C", [1, 2, 3, 4, 7, 8, 12, 16])
@pytest.mark.parametrize("S", [2, 63, 700, 20003])
def test_joined_sums(kind, C, S):
    # float32 sums of S terms in another order than the oracle's: within the gradients' bound
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(C + S)
    g = synth.normal_grid(rng, 8, C)
    xyz = _points(rng, kind, S)
    y = rng.uniform(0.1, 1.0, (S, C)).astype(np.float32)
    print(f"[case] joined sums {kind} C={C} S={S}", flush=True)
    dg = ops.DeviceGrid(torch.from_numpy(g.data).cuda(), g.xyz_min, g.xyz_max, grad=torch.zeros(8, 8, 8, C, device="cuda"))
    ops.grid_scatter(dg, torch.from_numpy(xyz).cuda(), torch.from_numpy(y).cuda())
    torch.cuda.synchronize()
    close(dg.grad.cpu().numpy(), oracle.scatter(g, xyz, y.astype(np.float64)), **GRAD, name="scatter")


@pytest.mark.parametrize("kind", ["one", "halves", "alternate", "behind"])
@pytest.mark.parametrize("mode", ["grid", "samples"])
def test_joined_sums_of_a_render_backward(kind, mode):
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(5)
    N, R, n = 130, 24, 8
    S = N * R
    xyz = _points(rng, kind, S)
    offs = (np.arange(R + 1) * N).astype(np.int32)
    mid = np.tile(((np.arange(N) + 0.5) / N).astype(np.float32), R)
    smp = synth.scenes.Samples(offs, xyz, np.full(S, 0.02, np.float32), mid, np.full(S, 1.0 / N, np.float32))
    dens, col = synth.normal_grid(rng, n, 1), synth.normal_grid(rng, n, 3)
    srgb = rng.random((S, 3)).astype(np.float32)
    GC = rng.standard_normal((R, 3)).astype(np.float32)
    shift = float(np.float32(-2.0))
    print(f"[case] joined sums, render backward {kind} {mode}", flush=True)

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda()

    b = ops.SampleBatch.from_arrays(offs, xyz, smp.delta, mid, smp.s_len)
    d = ops.DeviceGrid(dev(dens.data), dens.xyz_min, dens.xyz_max, grad=torch.zeros(n, n, n, 1, device="cuda"))
    c = ops.DeviceGrid(dev(col.data), col.xyz_min, col.xyz_max, grad=torch.zeros(n, n, n, 3, device="cuda")) if mode == "grid" else None
    s = None if mode == "grid" else dev(srgb)
    rgb, T, dist, state = ops.render_forward(b, d, c, s, act_shift_=shift)
    ops.render_backward(b, d, c, s, T, state, dev(GC), act_shift_=shift)
    torch.cuda.synchronize()
    want = oracle.render_backward(smp, dens, GC, color=col if mode == "grid" else None, srgb=None if mode == "grid" else srgb, shift=shift)
    close(d.grad.cpu().numpy(), want["grad_density"], **GRAD, name="grad density")
    if mode == "grid":
        close(c.grad.cpu().numpy(), want["grad_color"], **GRAD, name="grad colour")
