"""Builds libcaddtree.so (gfx950) in-tree with hipcc, and the Python binding's native calls where torch's
and Python's headers are there (the library needs neither).

Every HIP translation unit is compiled with packed fp32 instructions disabled
(``-target-feature -packed-fp32-ops``).
"""

from __future__ import annotations

import concurrent.futures as cf
import importlib.util
import os
import shutil
import subprocess
import sys
import sysconfig

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libcaddtree.so")
# the benchmark's read-bandwidth probe: a library of its own, outside the CaDDTree interface
PROBE_LIB = os.path.join(PKG, "libcaddtree_probe.so")
PROBE_SOURCES = ["probe.hip"]
SOURCES = ["api.cpp", "reduce_topk.hip", "expand.hip", "expand_level.hip", "expand_wide.hip", "emit.hip", "accept.hip",
           "scratch.hip", "costfit.cpp"]
# the Python binding's native calls (host code, against torch's headers): an extension module
BINDING = os.path.join(PKG, "_binding.so")
BINDING_SOURCE = "binding.cpp"
ARCH = os.environ.get("CADDTREE_ARCH", "gfx950")


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found (ROCm is required to build libcaddtree.so)")


def common_flags():
    return ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-I", INCLUDE, "-I", CSRC,
            "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
            "-Wall", "-Wno-unused-function", "-Wno-unused-command-line-argument"]


def torch_dir() -> str:
    spec = importlib.util.find_spec("torch")
    return "" if spec is None else os.path.dirname(spec.origin)


def binding_lacks() -> str:
    """What the binding's native calls cannot be built without and is not there ("" if all is)."""
    need = [os.path.join(torch_dir(), "include", "torch", "csrc", "autograd", "python_variable.h"),
            os.path.join(sysconfig.get_paths()["include"], "Python.h")]
    if not torch_dir():
        return "torch"
    return ", ".join(f for f in need if not os.path.exists(f))


def binding_flags():
    inc = os.path.join(torch_dir(), "include")
    return ["-D__HIP_PLATFORM_AMD__=1", "-I", sysconfig.get_paths()["include"], "-isystem", inc,
            "-isystem", os.path.join(inc, "torch", "csrc", "api", "include")]


def _compile(src: str, obj_dir: str, verbose: bool) -> str:
    obj = os.path.join(obj_dir, os.path.splitext(src)[0] + ".o")
    lang = ["-x", "hip"] if src.endswith(".hip") else []
    extra = binding_flags() if src == BINDING_SOURCE else []
    cmd = [hipcc()] + common_flags() + extra + lang + ["-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    if verbose and r.stderr.strip():
        print(r.stderr, file=sys.stderr)
    return obj


def _link(objs, out: str, verbose: bool, libs=()) -> None:
    tmp = out + ".tmp"
    cmd = [hipcc(), "-shared", "-fPIC", f"--offload-arch={ARCH}", "-o", tmp] + objs + list(libs)
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"link failed:\n{r.stdout}\n{r.stderr}")
    os.replace(tmp, out)


def build(verbose: bool = False) -> str:
    obj_dir = os.path.join(PKG, "_build")
    os.makedirs(obj_dir, exist_ok=True)
    lacks = binding_lacks()
    srcs = SOURCES + PROBE_SOURCES + ([] if lacks else [BINDING_SOURCE])
    with cf.ThreadPoolExecutor(max_workers=len(srcs)) as ex:
        objs = {s: ex.submit(_compile, s, obj_dir, verbose) for s in srcs}
    _link([objs[s].result() for s in SOURCES], LIB, verbose)
    _link([objs[s].result() for s in PROBE_SOURCES], PROBE_LIB, verbose)
    if lacks:                # the Python path serves without it; none of another source may stay
        print(f"the binding's native calls are not built: {lacks} not found", file=sys.stderr)
        if os.path.exists(BINDING):
            os.remove(BINDING)
    else:
        _link([objs[BINDING_SOURCE].result()], BINDING, verbose,
              ["-L" + os.path.join(torch_dir(), "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10"])
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
