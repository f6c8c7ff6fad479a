"""What one step of an adaptive-volume update hands to the next goes through a
launch of its own, read from the compiled kernels.  A counter by which a job's
last block takes over from the others is sound only if every wave waits for its
global stores and atomics at agent scope before the block reports, since neither
a barrier nor another wave's fence does; there is none."""
import os
import re
import subprocess

import pytest

from paper_2505_11655_amd import build


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "k_av.s")
    cmd = [build.hipcc()] + build.COMMON + ["-S", "--cuda-device-only", os.path.join(build.CSRC, "k_av.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return open(out).read()


@pytest.mark.parametrize("name", ["k_av_histIf", "k_av_histId", "k_av_count"])
def test_no_block_waits_for_the_others(listing, name):
    m = re.search(r"^(\w*" + name + r"\w*):.*?^\s*\.end_amdhsa_kernel", listing, re.S | re.M)
    assert m, "kernel not found"
    code = [l.split(";")[0].strip() for l in m.group(0).splitlines()]
    # an arrival: a 32-bit add whose old value comes back
    assert not [t for t in code if re.match(r"(global|flat)_atomic_(add|inc) v\d+, .*sc0", t)]
