"""The C++ autograd nodes against the Python Functions they stand in for (GPU)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import synth  # noqa: E402
from parity import GRAD, close  # noqa: E402

pytestmark = pytest.mark.gpu


def _dev(x, dt=torch.float32):
    return torch.as_tensor(x).to("cuda", dt).contiguous()


def _call(kind, mod, node, seed=0):
    """(function of the leaves, leaves) through the module's entry point or through its Function."""
    from paper_2206_05085_amd import ops
    rng = np.random.default_rng(seed)
    wl = synth.config2(R=40, N=48, n=24)
    smp = wl.samples
    b = ops.SampleBatch.from_arrays(smp.ray_offsets, smp.xyz, smp.delta, smp.s_mid, smp.s_len)
    box = (wl.density.xyz_min, wl.density.xyz_max)
    S = smp.n_samples
    if kind in ("render_grid", "render_samples", "render_nodist"):
        grid = kind == "render_grid"
        leaves = [_dev(wl.density.data), _dev(rng.random((24, 24, 24, 3) if grid else (S, 3)))]
        a = (grid, mod.ops.act_shift(), 1e-3 if grid else 0.0, (0.2, 0.5, 1.0), kind != "render_nodist")
        if node:
            return (lambda d, c: mod.render(d, c, b, box, grid_color=a[0], act_shift=a[1], halt_T=a[2], bg=a[3],
                                            want_dist=a[4])), leaves
        return (lambda d, c: mod.RenderFn.apply(d, c, b, box, *a)), leaves
    if kind == "distortion":
        rest = (b.ray_offsets, b.s_mid, b.s_len)
        return (lambda w: (mod.distortion if node else mod.DistortionFn.apply)(w, *rest)), [_dev(rng.random(S) / 40)]
    if kind == "gather":
        return (lambda g: mod.gather(g, b.xyz, box) if node else mod.GatherFn.apply(g, b.xyz, box)), [_dev(wl.feat.data)]
    mlp = synth.mlp_weights(rng, bias_std=0.3)
    leaves = [_dev(rng.standard_normal((S, 12)))] + [_dev(w) for w in mlp.W] + [_dev(v) for v in mlp.b]
    dirs = _dev(wl.rays.dirs)
    if node:
        return (lambda f, *p: mod.color_mlp(f, p[:3], p[3:], b.ray_offsets, dirs)), leaves
    return (lambda f, a1, a2, a3, b1, b2, b3: mod.ColorMLPFn.apply(f, a1, b1, a2, b2, a3, b3, b.ray_offsets, dirs, 4)), leaves


KINDS = ["render_grid", "render_samples", "render_nodist", "distortion", "gather", "head"]


def _run(kind, node, which=None, hooks=False):
    from paper_2206_05085_amd import autograd as mod
    fn, leaves = _call(kind, mod, node)
    leaves = [t.requires_grad_() for t in leaves]
    saved = []
    if hooks:
        with torch.autograd.graph.saved_tensors_hooks(lambda t: (saved.append(t.shape), t.cpu())[1], lambda t: t.cuda()):
            out = fn(*leaves)
        assert saved
    else:
        out = fn(*leaves)
    out = list(out) if isinstance(out, (tuple, list)) else [out]
    assert all(o.grad_fn is not None for o in out)
    ups = [torch.linspace(-1, 1, 2 * o.numel(), device="cuda").view(*o.shape, 2)[..., 0] for o in out]  # not contiguous
    use = range(len(out)) if which is None else which
    args = ([out[i] for i in use], leaves, [ups[i] for i in use])
    grads = torch.autograd.grad(*args, retain_graph=True)
    again = torch.autograd.grad(*args)
    for x, y in zip(grads, again):
        close(x.cpu().numpy(), y.cpu().numpy(), **GRAD, name="second backward")
    return out, grads


@pytest.mark.parametrize("kind,which,hooks", [(k, None, False) for k in KINDS] + [(k, None, True) for k in KINDS] +
                         [("render_samples", [i], False) for i in range(3)] + [("render_grid", [0], False)])
def test_nodes_match_functions(kind, which, hooks):
    # forward bit for bit; gradients to the order of their atomic sums; missing upstream gradients, upstream
    # gradients that are not contiguous, saved-tensor hooks, a second backward of the same graph
    print("[case] autograd node", kind, which, hooks, flush=True)
    a, ga = _run(kind, True, which, hooks)
    b, gb = _run(kind, False, which)
    assert type(a[0].grad_fn) is not type(b[0].grad_fn)  # not the same path twice
    for x, y in zip(a, b):
        assert x.shape == y.shape and torch.equal(x, y)
    for x, y in zip(ga, gb):
        assert x.shape == y.shape
        close(x.cpu().numpy(), y.cpu().numpy(), **GRAD, name="gradient")


@pytest.mark.parametrize("kind", KINDS)
def test_refused_calls_raise_as_before(kind):
    from paper_2206_05085_amd import autograd as mod

    def error(node, spoil):
        fn, leaves = _call(kind, mod, node)
        try:
            fn(*spoil(leaves))
        except Exception as e:  # noqa: BLE001
            return type(e), str(e)
        return None

    for spoil in (lambda t: [t[0].double()] + t[1:], lambda t: [t[0].cpu()] + t[1:],
                  lambda t: [t[0][:-1]] + t[1:] if kind == "distortion" else [t[0].transpose(0, 1)] + t[1:]):
        assert error(True, spoil) == error(False, spoil) and error(False, spoil) is not None


def test_transforms_take_the_function():
    from paper_2206_05085_amd import autograd as mod
    for kind in KINDS:
        fn, leaves = _call(kind, mod, True)
        with pytest.raises(RuntimeError):  # a Function without a vmap rule says so
            torch.func.vmap(fn)(*[t[None] for t in leaves])
    fn, leaves = _call("gather", mod, True)
    x = leaves[0].requires_grad_()
    out = fn(x)
    with torch.no_grad():
        x.mul_(2.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        out.sum().backward()


def test_nodes_on_a_side_stream():
    from paper_2206_05085_amd import autograd as mod
    fn, leaves = _call("head", mod, True)
    leaves = [t.requires_grad_() for t in leaves]
    want = torch.autograd.grad(fn(*leaves).sum(), leaves)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        got = torch.autograd.grad(fn(*leaves).sum(), leaves)
    torch.cuda.current_stream().wait_stream(side)
    for x, y in zip(got, want):
        assert torch.equal(x, y)
