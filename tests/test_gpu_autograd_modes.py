"""The autograd entry points under the modes and call forms that their Functions serve (GPU)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_autograd_nodes import KINDS, _call  # noqa: E402

pytestmark = pytest.mark.gpu


def _first(out):
    return out[0] if isinstance(out, (tuple, list)) else out


def _outcome(fn):
    try:
        return fn()
    except Exception as e:  # noqa: BLE001
        return type(e), str(e)


@pytest.mark.parametrize("kind", KINDS)
def test_forward_mode_takes_the_function(kind):
    from torch.autograd import forward_ad

    from paper_2206_05085_amd import autograd as mod

    def dual(node):
        fn, leaves = _call(kind, mod, node)
        with forward_ad.dual_level():
            return fn(forward_ad.make_dual(leaves[0], torch.ones_like(leaves[0])), *leaves[1:])

    def plain(node):  # a level is active, but no tensor has a tangent
        fn, leaves = _call(kind, mod, node)
        with forward_ad.dual_level():
            out = _first(fn(*[t.requires_grad_() for t in leaves]))
        return out, type(out.grad_fn).__name__

    print("[case] forward mode", kind, flush=True)
    want = _outcome(lambda: dual(False))
    assert want[0] is NotImplementedError and _outcome(lambda: dual(True)) == want
    (x, name), (y, want) = plain(True), plain(False)
    assert name == want and torch.equal(x, y)


class _NoGradient(torch.autograd.Function):
    """A consumer whose backward has nothing to pass on."""

    @staticmethod
    def forward(ctx, x):
        return x.clone()

    @staticmethod
    def backward(ctx, g):
        return None


@pytest.mark.parametrize("kind", KINDS)
def test_undefined_upstream_gradients_are_zeros(kind):
    from paper_2206_05085_amd import autograd as mod
    print("[case] undefined upstream", kind, flush=True)
    for node in (True, False):
        fn, leaves = _call(kind, mod, node)
        leaves = [t.requires_grad_() for t in leaves]
        out = fn(*leaves)
        out = list(out) if isinstance(out, (tuple, list)) else [out]
        grads = torch.autograd.grad(sum(_NoGradient.apply(o).sum() for o in out), leaves)
        assert all(g.shape == t.shape and not g.any() for g, t in zip(grads, leaves)), node


def test_library_errors_of_a_backward_are_dvgo_errors():
    # a batch spoilt after the forward, which debug mode finds on the device before anything is launched
    from paper_2206_05085_amd import _lib, autograd as mod, ops
    import synth
    wl = synth.config2(R=40, N=48, n=24)
    smp = wl.samples
    errors = []
    for node in (True, False):
        b = ops.SampleBatch.from_arrays(smp.ray_offsets, smp.xyz, smp.delta, smp.s_mid.copy(), smp.s_len)
        d = torch.as_tensor(wl.density.data).cuda().requires_grad_()
        c = torch.rand(smp.n_samples, 3, device="cuda")
        box = (wl.density.xyz_min, wl.density.xyz_max)
        before = ops.set_debug(True)
        try:
            args = (False, -4.0, 0.0, (1.0, 1.0, 1.0), True)
            if node:
                out = mod.render(d, c, b, box, grid_color=args[0], act_shift=args[1])
            else:
                out = mod.RenderFn.apply(d, c, b, box, *args)
            b.s_mid.copy_(b.s_mid.flip(0))
            with pytest.raises(_lib.DvgoError) as e:
                out[0].sum().backward()
            errors.append((e.value.code, str(e.value)))
        finally:
            ops.set_debug(before)
    assert errors[0] == errors[1] and _lib.ERRORS[errors[0][0]] == "ERR_UNSORTED"


FORMS = {
    "list": list, "ints": lambda v: [int(x) if x == int(x) else x for x in v], "array": lambda v: __import__("numpy").array(v),
    "tensor": torch.tensor, "device tensor": lambda v: torch.tensor(v).cuda(), "iterator": iter, "text": lambda v: [str(x) for x in v],
    "two": lambda v: v[:2], "four": lambda v: [*v, 1.0], "none": lambda v: None,
}


@pytest.mark.parametrize("form", FORMS)
def test_box_and_background_forms(form):
    # every form the Functions take gives what a tuple gives; the others raise the same error
    import synth
    from paper_2206_05085_amd import autograd as mod, ops
    wl = synth.config2(R=40, N=48, n=24)
    smp, f = wl.samples, FORMS[form]
    b = ops.SampleBatch.from_arrays(smp.ray_offsets, smp.xyz, smp.delta, smp.s_mid, smp.s_len)
    d, c = torch.as_tensor(wl.density.data).cuda(), torch.rand(smp.n_samples, 3, device="cuda")
    bg, lo, hi = (0.25, 0.5, 1.0), (-1.0, -1.0, -1.0), (1.0, 1.0, 1.0)
    args = (False, -4.0, 0.0)

    def same(node, function, plain):
        x, y = _outcome(node), _outcome(function)
        if isinstance(y, tuple) and isinstance(y[0], type):
            assert form in ("two", "four", "none") and x == y
        else:
            assert torch.equal(_first(x), _first(y)) and torch.equal(_first(x), _first(plain()))

    same(lambda: mod.render(d, c, b, (lo, hi), grid_color=False, act_shift=-4.0, bg=f(bg)),
         lambda: mod.RenderFn.apply(d, c, b, (lo, hi), *args, tuple(f(bg)), True),
         lambda: mod.render(d, c, b, (lo, hi), grid_color=False, act_shift=-4.0, bg=bg))
    same(lambda: mod.render(d, c, b, (f(lo), f(hi)), grid_color=False, act_shift=-4.0),
         lambda: mod.RenderFn.apply(d, c, b, (f(lo), f(hi)), *args, (1.0, 1.0, 1.0), True),
         lambda: mod.render(d, c, b, (lo, hi), grid_color=False, act_shift=-4.0))
    same(lambda: mod.gather(d, b.xyz, (f(lo), f(hi))), lambda: mod.GatherFn.apply(d, b.xyz, (f(lo), f(hi))),
         lambda: mod.gather(d, b.xyz, (lo, hi)))
