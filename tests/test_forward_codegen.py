"""What the layer output's kernels are built around, checked on the generated assembly (no GPU: hipcc cross-compiles gfx950).

The combine waits for memory and little else: it lives from eight waves per SIMD, which 64 vector registers a lane leave, with
parts of K to add or without.
"""
import os
import re
import shutil
import subprocess

import pytest


def test_combine_leaves_eight_waves_per_simd(tmp_path):
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not found")
    from paper_2508_02322_amd import build
    out = tmp_path / "forward.s"
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    res = subprocess.run([build.hipcc(), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "forward.hip"), "-o", str(out)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    registers = {name: int(n) for name, n in re.findall(r"\.name:\s+(\S*combine_kernel\S*).*?\.vgpr_count:\s+(\d+)", out.read_text(), re.S)}
    assert len(registers) == 3 and max(registers.values()) <= 64, registers
