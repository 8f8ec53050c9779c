"""The reduction's streaming loads stay inside their segment (CPU: reads the assembly that the build's own
compile of reduce_topk.hip makes for gfx950).

A load of the ring may lie past the segment's end; it then returns zeros without touching memory, because the
descriptor's size covers the segment and the hardware holds the load's offset against it.  That check covers the
lane's offset register and the instruction's 12-bit offset, not the scalar offset, so no load may have one.
"""

import os
import re
import subprocess

import pytest

from paper_2606_01813_amd import _build


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "reduce_topk.txt")
    cmd = [_build.hipcc()] + _build.common_flags() + ["--offload-device-only", "-S", "-x", "hip",
                                                      os.path.join(_build.CSRC, "reduce_topk.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        return f.read()


def test_every_buffer_load_offset_is_range_checked(assembly):
    loads = re.findall(r"^\s*(buffer_load_\S+)\s+(v\S+), (v\S+|off), (s\[\d+:\d+\]), (\S+)(.*)$", assembly, re.M)
    assert len(loads) == len(re.findall(r"^\s*buffer_load_", assembly, re.M)) > 0
    for op, _, lane, _, scalar, rest in loads:
        assert op == "buffer_load_dwordx4" and lane != "off" and " offen" in rest
        assert scalar == "0", "the scalar offset is not part of the range check: " + scalar
        at = re.search(r"offset:(\d+)", rest)
        assert at is None or int(at.group(1)) % 1024 == 0 and int(at.group(1)) < 4096
