"""The hand-over to a job's last block (adaptive volume), read from the compiled
kernels: every wave has to wait for its own global stores and atomics before the
barrier that precedes the block's arrival, since neither the barrier nor
another wave's fence waits for them."""
import os
import re
import subprocess

import pytest

from paper_2505_11655_amd import build

KERNELS = ["k_av_histIfE", "k_av_histIdE", "k_av_countE"]


@pytest.fixture(scope="module")
def listing(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("asm") / "k_av.s")
    cmd = [build.hipcc()] + build.COMMON + ["-S", "--cuda-device-only", os.path.join(build.CSRC, "k_av.hip"), "-o", out]
    subprocess.run(cmd, check=True, capture_output=True)
    return open(out).read()


@pytest.mark.parametrize("name", KERNELS)
def test_every_wave_drains_before_the_arrival(listing, name):
    m = re.search(r"^(\w*" + name + r"\w*):.*?^\s*\.end_amdhsa_kernel", listing, re.S | re.M)
    assert m, "kernel not found"
    code = [t for t in (l.split(";")[0].strip() for l in m.group(0).splitlines()) if t and not t.startswith(".")]
    # the arrival: the only 32-bit add whose old value comes back
    arrive = [i for i, t in enumerate(code) if re.match(r"(global|flat)_atomic_add v\d+, .*sc0", t)]
    assert len(arrive) == 1, arrive
    barrier = max(i for i in range(arrive[0]) if code[i].startswith("s_barrier"))
    drained = released = False
    for t in reversed(code[:barrier]):
        if t.startswith("s_waitcnt") and "vmcnt(0)" in t:
            drained = True
        if drained and t.startswith("buffer_wbl2"):
            released = True
            break
        assert not re.match(r"(global|flat|buffer)_(store|atomic)", t), f"in flight at the barrier: {t}"
        assert not t.startswith("s_barrier"), "no release between the barriers"
    assert drained and released
