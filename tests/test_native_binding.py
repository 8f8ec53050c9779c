"""The native calls of the binding against the Python checks (CPU, no GPU needed).

Over forms of every argument (types, shapes, strides, None, other objects), a native call either passes the
library exactly what the Python path passes it, or returns None and leaves the call to the Python path; what the
Python path refuses it never passes on.  Host tensors stand in for device ones, and recording functions for the
library's.
"""

import ctypes
import os
import shutil
import subprocess
import sys

import numpy as np
import pytest
import torch

import paper_2606_01813_amd as pkg
from paper_2606_01813_amd import Plan, TreeOutputs, _lib

B, K, V = 3, 4, 64
STREAM = 0x1234


class _Recorder:
    """Stands in for the library: every function records its arguments and returns 0."""

    def __init__(self):
        self.calls = []
        real = _lib.lib()
        for name in ("build", "build_noalloc", "reduce_topk", "expand", "emit", "accept"):
            types = getattr(real, "caddtree_" + name).argtypes
            f = ctypes.CFUNCTYPE(ctypes.c_int, *types)(self._make(name))
            f.argtypes = types
            setattr(self, "caddtree_" + name, f)

    def _make(self, name):
        def record(*args):
            flat = []
            for a in args:
                if isinstance(a, ctypes.POINTER(_lib.Outputs)):
                    flat += [getattr(a.contents, f) for f, _ in _lib.Outputs._fields_]
                else:
                    flat.append(a)
            self.calls.append((name, tuple(flat)))
            return 0
        return record


def _plans(monkeypatch, L, cap, mask, dtype):
    monkeypatch.setattr(pkg, "_on_device", lambda t, device: t.device.type == "cpu")
    monkeypatch.setattr(pkg, "_stream", lambda stream, device: STREAM)
    rec = _Recorder()
    plans = []
    for native in (False, True):
        p = object.__new__(Plan)
        p.L, p.V, p.K, p.cap, p.dtype, p.mask, p.device = L, V, K, cap, dtype, mask, 0
        p._lib, p._h = rec, ctypes.c_void_p(0x10)
        p.close = lambda: None
        if native:
            p._native = _lib.binding()
            p._fast = _lib.call_spec(rec, 0x10, -1, L, V, K, cap, dtype, mask)
            p._raw_stream = lambda stream: STREAM
        plans.append(p)
    return rec, plans[0], plans[1]


def _state(L, cap, mask, dtype):
    i32, f32, f64 = dict(dtype=torch.int32), dict(dtype=torch.float32), dict(dtype=torch.float64)
    c = max(cap, 1)
    m = {"u8": lambda: torch.zeros((B, c, c), dtype=torch.uint8),
         "bits": lambda: torch.zeros((B, c, (c + 31) // 32), **i32), "none": lambda: None}[mask]()
    out = TreeOutputs(token_ids=torch.zeros((B, c), **i32), parent=torch.zeros((B, c), **i32),
                      depth=torch.zeros((B, c), **i32), path_prob=torch.zeros((B, c), **f32),
                      n_star=torch.zeros((B,), **i32), phi=torch.zeros((B,), **f32), theta=torch.zeros((B,), **f32),
                      mask=m, pos_ids=torch.zeros((B, c), **i32), topk_ids=torch.zeros((B, L, K), **i32),
                      topk_logit=torch.zeros((B, L, K), **f32), topk_lq=torch.zeros((B, L, K), **f32),
                      lse=torch.zeros((B, L), **f64))
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    return {"logits": torch.zeros((B, L, V), dtype=dt), "out": out, "pos_offset": 7, "workspace":
            torch.zeros(4096, dtype=torch.uint8), "ctx_len": torch.zeros(B, dtype=torch.int64),
            "u": torch.zeros((B, L), **f64), "accept_len": torch.zeros(B, **i32), "round_cost": torch.zeros(B, **f64)}


CALLS = {
    "build": lambda p, s: p.build(s["logits"], s["out"], s["pos_offset"], s["workspace"], None, s["ctx_len"]),
    "build_noalloc": lambda p, s: p.build_noalloc(s["logits"], s["out"], s["pos_offset"], None, s["ctx_len"]),
    "reduce_topk": lambda p, s: p.reduce_topk(s["logits"], s["out"].topk_ids, s["out"].topk_logit, s["out"].lse,
                                              s["out"].topk_lq),
    "expand": lambda p, s: p.expand(s["out"].topk_ids, s["out"].topk_logit, s["out"].lse, s["out"], None,
                                    s["ctx_len"]),
    "emit": lambda p, s: p.emit(s["out"], s["pos_offset"]),
    "accept": lambda p, s: p.accept(s["out"], s["out"], s["u"], s["accept_len"], s["round_cost"], s["ctx_len"]),
}


def _forms(t):
    """Other forms of a tensor argument."""
    yield None
    yield "text"
    yield np.zeros(3)
    yield torch.nn.Parameter(t.clone(), requires_grad=False)
    for dt in (torch.int32, torch.int64, torch.float32, torch.float64, torch.bfloat16, torch.uint8, torch.uint32):
        yield torch.zeros(t.shape, dtype=dt)
    yield torch.zeros((t.shape[0] + 2,) + tuple(t.shape[1:]), dtype=t.dtype)         # a longer batch
    yield torch.zeros((t.shape[0] - 1,) + tuple(t.shape[1:]), dtype=t.dtype)         # a shorter one
    yield torch.zeros((0,) + tuple(t.shape[1:]), dtype=t.dtype)
    yield torch.zeros((2 * t.shape[0],) + tuple(t.shape[1:]), dtype=t.dtype)[::2]    # every other row
    yield torch.zeros(tuple(t.shape) + (1,), dtype=t.dtype)
    yield torch.zeros(tuple(t.shape) + (2,), dtype=t.dtype)[..., 0]                  # strided elements
    yield torch.zeros(tuple(t.shape[:-1]) + (t.shape[-1] + 3,), dtype=t.dtype)
    yield torch.zeros(tuple(t.shape[:-1]) + (t.shape[-1] + 3,), dtype=t.dtype)[..., : t.shape[-1]]
    yield torch.zeros(t.shape[::-1], dtype=t.dtype).permute(*range(t.dim() - 1, -1, -1))
    yield torch.zeros(t.numel() + 1, dtype=t.dtype)[1:].view(t.shape)                # an offset into its storage
    yield torch.zeros((1,) * t.dim(), dtype=t.dtype).expand(t.shape)
    yield torch.zeros(t.shape, dtype=t.dtype, device="meta")
    yield torch.zeros((), dtype=t.dtype)
    if t.dtype.is_floating_point:
        yield torch.zeros(t.shape, dtype=t.dtype, requires_grad=True)
        yield torch.zeros(t.shape, dtype=t.dtype).to_sparse()


def _outcome(rec, plan, call, s):
    rec.calls.clear()
    try:
        CALLS[call](plan, s)
    except Exception as e:
        assert not rec.calls
        return type(e), str(e)
    assert len(rec.calls) == 1
    return rec.calls[0]


@pytest.mark.parametrize("L,cap,mask,dtype", [(4, 40, "u8", "bf16"), (1, 1, "bits", "f32"), (5, 70, "bits", "bf16"),
                                              (3, 0, "none", "f32")])
@pytest.mark.parametrize("call", list(CALLS))
def test_native_calls_pass_what_the_python_path_passes(call, L, cap, mask, dtype, monkeypatch):
    rec, slow, fast = _plans(monkeypatch, L, cap, mask, dtype)
    native = []
    for name in ("build", "reduce_topk", "expand", "emit", "accept"):
        def spy(*a, f=getattr(fast._native, name)):
            r = f(*a)
            native.append(r)
            return r
        monkeypatch.setattr(fast._native, name, spy)
    s = _state(L, cap, mask, dtype)
    if call == "accept":
        assert s["out"].token_ids.shape[1] == max(cap, 1)

    def both(what, expect_native=False):
        a = _outcome(rec, slow, call, s)
        native.clear()
        b = _outcome(rec, fast, call, s)
        assert a == b, (call, what, a, b)
        assert len(native) == 1
        if expect_native:
            assert native[0] == 0, (call, what)
        if isinstance(a[0], type):
            assert native[0] is None, (call, what)

    both("as it is", expect_native=True)
    for key in ("logits", "workspace", "ctx_len", "u", "accept_len", "round_cost"):
        keep = s[key]
        for i, form in enumerate(_forms(keep)):
            s[key] = form
            both((key, i))
        s[key] = keep
    for f, _ in _lib.Outputs._fields_:
        keep = getattr(s["out"], f)
        if keep is None:
            continue
        for i, form in enumerate(_forms(keep)):
            setattr(s["out"], f, form)
            both((f, i))
        setattr(s["out"], f, keep)
    for pos in (0, -5, 2 ** 31 - 1, 2 ** 31, True, np.int64(3), 2.0, "x", None):
        s["pos_offset"] = pos
        both(("pos_offset", pos))
    s["pos_offset"] = 7
    dt = s["logits"].dtype
    wide = torch.zeros((B, L, V + 9), dtype=dt)                       # rows padded, longer batches, one round
    for i, form in enumerate((wide[:, :, :V], wide, torch.zeros((2 * B, L, V), dtype=dt)[::2],
                              torch.zeros((B, 2 * L, V), dtype=dt)[:, ::2], torch.zeros((B, L + 1, V), dtype=dt)[:, :L],
                              wide[:1], wide[:2, :, 3:], torch.zeros((1, L, 2 * V), dtype=dt)[:, :, ::2])):
        s["logits"] = form
        s["ctx_len"] = torch.zeros(form.shape[0], dtype=torch.int64)
        both(("rows", i))
    if call not in ("reduce_topk", "expand", "accept"):
        s["out"] = object()
        both("no outputs")


_THROWS = r"""
import ctypes, sys
import torch
from paper_2606_01813_amd import _lib
f = ctypes.cast(ctypes.CDLL(sys.argv[1]).throws, ctypes.c_void_p).value
native = _lib.binding()
spec = native.spec(0x10, -1, 2, 16, 2, 4, 0, 0, f, f, f, f, f, f)
i32 = torch.zeros((1, 2, 2), dtype=torch.int32)
try:
    native.reduce_topk(spec, torch.zeros((1, 2, 16)), i32, torch.zeros((1, 2, 2)), torch.zeros((1, 2), dtype=torch.float64),
                       None, 0)
except RuntimeError as e:
    print("raised", e, sum(range(1000)))
"""


def test_an_exception_out_of_the_library_is_raised_with_the_lock_held(tmp_path):
    """Raised once, and not passed to the Python path, which would make the call again."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ is not available")
    (tmp_path / "throws.cpp").write_text("#include <new>\nextern \"C\" int throws() { throw std::bad_alloc(); }\n")
    so = str(tmp_path / "throws.so")
    subprocess.run([gxx, "-shared", "-fPIC", "-o", so, str(tmp_path / "throws.cpp")], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(pkg.__file__)))
    r = subprocess.run([sys.executable, "-c", _THROWS, so], capture_output=True, text=True, cwd=root, timeout=300)
    assert r.returncode == 0 and "raised the caddtree library threw" in r.stdout, r.stdout + r.stderr
