"""The batch's phase end waits where it has to, in the code built for gfx950; no GPU.

An L2 write-back (buffer_wbl2) is over only when a vmcnt(0) wait behind it is:
counting a phase's items before that lets a block of another XCD read the links
of the phase before.  The compiler may leave a release fence's wait out, so the
emitted instructions are looked at.
"""

import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
WAIT = re.compile(r"s_waitcnt\b.*vmcnt\(0\)")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of each persistent kernel, in program order."""
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not installed")
    out = str(tmp_path_factory.mktemp("asm") / "batched.s")
    r = subprocess.run([HIPCC, "-O3", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-x", "hip", "--cuda-device-only", "-S",
                        os.path.join(ROOT, "paper_1105_2279_amd", "csrc", "batched.hip"), "-o", out],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    found, name = {}, None
    for line in open(out):
        line = line.split(";")[0].strip()
        m = re.match(r"(\w*k_ape_batched\w*):", line)
        if m:
            name = m.group(1)
            found[name] = []
        elif line.startswith(".Lfunc_end"):
            name = None
        elif name and line and not line.startswith("."):
            found[name].append(line)
    assert found
    return found


def test_write_back_is_waited_for(kernels):
    for name, ins in kernels.items():
        backs = [i for i, x in enumerate(ins) if x.startswith("buffer_wbl2")]
        assert backs, name
        for i in backs:
            after = next(x for x in ins[i + 1:] if WAIT.match(x) or x.startswith(("global_", "flat_", "s_barrier",
                                                                                  "s_endpgm")))
            assert WAIT.match(after), (name, after)


def test_invalidation_follows_an_arrived_count(kernels):
    for name, ins in kernels.items():
        invs = [i for i, x in enumerate(ins) if x.startswith("buffer_inv")]
        assert invs, name
        for i in invs:  # the poll's load has arrived before the caches are dropped
            before = next(x for x in reversed(ins[:i]) if WAIT.match(x) or x.startswith(("global_load", "flat_load")))
            assert WAIT.match(before), (name, before)
