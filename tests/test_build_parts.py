"""What the build makes without torch, and what serves without the binding's native calls (CPU)."""

import os

import pytest

import paper_2606_01813_amd as pkg
from paper_2606_01813_amd import Plan, _build, _lib


@pytest.fixture
def steps(monkeypatch, tmp_path):
    """The build with its compiles and links recorded and none made."""
    done = []
    monkeypatch.setattr(_build, "PKG", str(tmp_path))
    monkeypatch.setattr(_build, "BINDING", str(tmp_path / "_binding.so"))
    monkeypatch.setattr(_build, "_compile", lambda src, obj_dir, verbose: src)
    monkeypatch.setattr(_build, "_link", lambda objs, out, verbose, libs=(): done.append((os.path.basename(out), objs)))
    return done


def test_everything_is_built(steps):
    _build.build()
    assert [n for n, _ in steps] == ["libcaddtree.so", "libcaddtree_probe.so", "_binding.so"]
    assert steps[0][1] == _build.SOURCES and steps[2][1] == ["binding.cpp"]


def test_the_library_is_built_without_torch(steps, monkeypatch):
    real = _build.importlib.util.find_spec
    monkeypatch.setattr(_build.importlib.util, "find_spec", lambda name: None if name == "torch" else real(name))
    with open(_build.BINDING, "w") as f:
        f.write("of another source")
    _build.build()
    assert [n for n, _ in steps] == ["libcaddtree.so", "libcaddtree_probe.so"]
    assert not os.path.exists(_build.BINDING)


def test_the_library_is_built_without_python_headers(steps, monkeypatch):
    paths = dict(_build.sysconfig.get_paths(), include="/nonexistent")
    monkeypatch.setattr(_build.sysconfig, "get_paths", lambda: paths)
    _build.build()
    assert [n for n, _ in steps] == ["libcaddtree.so", "libcaddtree_probe.so"]


def test_a_binding_that_does_not_compile_is_an_error_after_the_library(steps, monkeypatch):
    def compile_(src, obj_dir, verbose):
        if src == "binding.cpp":
            raise RuntimeError("hipcc failed on binding.cpp")
        return src
    monkeypatch.setattr(_build, "_compile", compile_)
    with pytest.raises(RuntimeError, match="binding.cpp"):
        _build.build()
    assert [n for n, _ in steps] == ["libcaddtree.so", "libcaddtree_probe.so"]


class _Library:
    """Stands in for the library: plans are made, and a build's arguments are recorded."""

    def __init__(self):
        self.builds = []

    def caddtree_plan_create(self, cfg, h):
        return 0

    def caddtree_plan_destroy(self, h):
        pass

    def caddtree_build(self, *args):
        self.builds.append(args)
        return 0


def test_plans_serve_without_the_native_calls(monkeypatch, tmp_path):
    import torch
    lib = _Library()
    monkeypatch.setattr(_lib, "_HERE", str(tmp_path))
    monkeypatch.setattr(_lib, "_BINDING", None)
    monkeypatch.setattr(_lib, "lib", lambda: lib)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(pkg, "_on_device", lambda t, device: t.device.type == "cpu")
    monkeypatch.setattr(pkg, "_stream", lambda stream, device: 0x1234)
    plan = Plan(L=2, V=16, K=2, cap=4, t_draft=1.0, t_verify=[1.0, 1.1, 1.2, 1.3, 1.4], dtype="f32")
    out = plan.new_outputs(1, device="cpu")
    plan.build(torch.zeros((1, 2, 16)), out)
    assert len(lib.builds) == 1
    with pytest.raises(ValueError):
        plan.build(torch.zeros((1, 3, 16)), out)
    assert len(lib.builds) == 1
