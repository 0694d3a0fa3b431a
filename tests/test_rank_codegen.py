"""What the ranking kernels assume of their launch, checked on the generated assembly (no GPU: hipcc cross-compiles
gfx950).

The 128 KiB histogram of the first select pass is LDS of the kernel itself.  As dynamic LDS it would need a function
attribute, which is set per device: a context on a second GPU of the process would have to set it again, and a note of
having done so would be shared by host threads.
"""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_select_histogram_is_static_lds(tmp_path):
    if shutil.which("hipcc") is None and not os.path.exists("/opt/rocm/bin/hipcc"):
        pytest.skip("hipcc not found")
    from paper_2508_02322_amd import build
    out = tmp_path / "rank.s"
    flags = [f for f in build.FLAGS if f != "-fPIC"]
    res = subprocess.run([build.hipcc(), *flags, "--cuda-device-only", "-S", os.path.join(build.CSRC, "rank.hip"), "-o", str(out)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    sizes = {name: int(lds) for lds, name in
             re.findall(r"\.group_segment_fixed_size:\s+(\d+).*?\.name:\s+(\S+)", out.read_text(), re.S)}
    top = [lds for name, lds in sizes.items() if "rank_top_kernel" in name]
    assert top == [2 * (1 << 16) + 4 * (1 << 8)]      # 2^16 counters of 16 bits, 2^8 of 32
