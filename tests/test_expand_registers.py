"""Registers of the several-wavefront expansion (CPU: reads the assembly that the build's own compile of
expand_wide.hip makes for gfx950).

With more rounds than compute units the kernel runs eight wavefronts a round so that two rounds share a compute
unit: sixteen wavefronts on four SIMDs of 512 registers a lane, at most 128 each.
"""

import os
import re
import subprocess

from paper_2606_01813_amd import _build


def test_two_rounds_of_eight_wavefronts_share_a_compute_unit(tmp_path):
    out = str(tmp_path / "expand_wide.txt")
    cmd = [_build.hipcc()] + _build.common_flags() + ["--offload-device-only", "-S", "-x", "hip",
                                                      os.path.join(_build.CSRC, "expand_wide.hip"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    with open(out) as f:
        text = f.read()
    used = {}
    for name, body in re.findall(r"^(_Z\w*expand_wide_kernel\w*):(.*?)^; Occupancy:", text, re.M | re.S):
        used[name] = int(re.search(r"; TotalNumVgprs: (\d+)", body).group(1))
    assert len(used) == 2 and all(n <= 128 for n in used.values()), used
