"""What the autograd entry points do with tensors that saved-tensor hooks hand back (GPU)."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_autograd_nodes import _call  # noqa: E402

pytestmark = pytest.mark.gpu


def _permuted(t):
    # the same values and sizes, other strides: what the hooks' contract allows
    return t.permute(*reversed(range(t.dim()))).contiguous().permute(*reversed(range(t.dim())))


# (kind, place of the tensor among the saved ones, what the hook hands back instead)
CASES = [(kind, at, "strides") for kind, n in (("render_grid", 2), ("render_samples", 2), ("gather", 2)) for at in range(n)]
CASES += [("head", at, "strides") for at in (0, 1, 3, 5, 8)]
CASES += [("distortion", at, "strides") for at in (2, 3)]
CASES += [(kind, at, change) for kind, n in (("render_grid", 2), ("gather", 2), ("head", 9), ("distortion", 4))
          for at in range(n) for change in ("cpu", "type")]


@pytest.mark.parametrize("kind,at,change", CASES)
def test_changed_saved_tensors_are_refused(kind, at, change):
    from paper_2206_05085_amd import autograd as mod
    print("[case] saved tensor", kind, at, change, flush=True)
    fn, leaves = _call(kind, mod, True)
    leaves = [t.requires_grad_() for t in leaves]
    seen = []

    def pack(t):
        seen.append(t)
        return len(seen) - 1, t

    def unpack(x):
        i, t = x
        if i != at:
            return t
        if change == "cpu":
            return t.cpu()
        if change == "type":
            return t.double()
        return _permuted(t) if t.dim() > 1 else torch.stack([t, t], 1)[:, 0]

    with torch.autograd.graph.saved_tensors_hooks(pack, unpack):
        out = fn(*leaves)
    out = out[0] if isinstance(out, (tuple, list)) else out
    want = {"cpu": (ValueError, "must live on the GPU"), "type": (TypeError, "must be torch.*, got torch.(float64|double)"),
            "strides": (ValueError, "must be contiguous")}[change]
    with pytest.raises(want[0], match=want[1]):
        torch.autograd.grad(out.sum(), leaves)
    torch.cuda.synchronize()


def test_weights_of_other_strides_are_read_by_value():
    # the one saved tensor whose strides are free: both paths take a contiguous copy of it
    from paper_2206_05085_amd import autograd as mod
    fn, (w,) = _call("distortion", mod, True)
    w.requires_grad_()
    want = torch.autograd.grad(fn(w).sum(), w)[0]
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, lambda t: torch.stack([t, t], 1)[:, 0] if t.data_ptr() == w.data_ptr() else t):
        out = fn(w)
    assert torch.equal(torch.autograd.grad(out.sum(), w)[0], want)
