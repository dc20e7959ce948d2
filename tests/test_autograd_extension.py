"""The package without the C++ autograd nodes: libdvgo.so alone serves every call."""
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2206_05085_amd import _lib, autograd, build  # noqa: E402


def test_entry_points_take_the_functions_without_the_extension(monkeypatch):
    monkeypatch.setattr(_lib, "lib", lambda: None)
    monkeypatch.setattr(autograd, "_nodes", None)
    monkeypatch.setattr(autograd, "_eager", lambda *t: True)
    monkeypatch.setitem(sys.modules, "paper_2206_05085_amd._dvgo_autograd", None)  # import raises ImportError
    monkeypatch.delattr(sys.modules["paper_2206_05085_amd"], "_dvgo_autograd", raising=False)
    taken = []
    for name in ("RenderFn", "DistortionFn", "GatherFn", "ColorMLPFn"):
        monkeypatch.setattr(autograd, name, type(name, (), {"apply": staticmethod(lambda *a, n=name: taken.append(n))}))
    x, box = torch.zeros(1), ((0.0,) * 3, (1.0,) * 3)
    with pytest.warns(RuntimeWarning, match="not built"):
        autograd.render(x, x, None, box, grid_color=True, act_shift=0.0)
    autograd.distortion(x, x, x, x)
    autograd.gather(x, x, box)
    autograd.color_mlp(x, [x] * 3, [x] * 3, x, x)
    assert taken == ["RenderFn", "DistortionFn", "GatherFn", "ColorMLPFn"]


@pytest.mark.parametrize("cxx", ["/nonexistent/c++", "/bin/false"])
def test_build_goes_on_without_a_host_compiler(monkeypatch, tmp_path, capfd, cxx):
    lib, nodes = tmp_path / "libdvgo.so", tmp_path / "_dvgo_autograd.so"
    nodes.write_text("of an older build")
    monkeypatch.setattr(build, "LIB", str(lib))
    monkeypatch.setattr(build, "NATIVE", str(nodes))
    monkeypatch.setattr(build, "HERE", str(tmp_path))
    monkeypatch.setenv("CXX", cxx)
    real = subprocess.check_call

    def compile_(cmd):
        if cmd[0] != build.HIPCC:
            return real(cmd)
        (tmp_path / "libdvgo.so.tmp").write_text("library")

    monkeypatch.setattr(subprocess, "check_call", compile_)
    assert build.build() == str(lib) and lib.read_text() == "library" and not nodes.exists()
    assert "autograd nodes were not built" in capfd.readouterr().err
