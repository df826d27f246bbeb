"""The library's device memory: the pool's rules on made-up devices
(tests/devpool_harness.cpp), and every allocation going through it."""
from __future__ import annotations

import os
import re
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1505_07855_amd", "csrc")


def test_pool_rules(tmp_path):
    exe = str(tmp_path / "devpool_harness")
    subprocess.check_call(["g++", "-O1", "-g", "-std=c++17", "-pthread", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(ROOT, "tests", "devpool_harness.cpp"),
                           os.path.join(CSRC, "devpool.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "all checks passed" in r.stdout, r.stdout


def test_every_allocation_goes_through_the_pool():
    """A block taken around the pool would fail while the pool holds memory."""
    for name in sorted(os.listdir(CSRC)):
        if name != "devpool.cpp":
            with open(os.path.join(CSRC, name)) as f:
                assert not re.findall(r"\bhip(?:Malloc|Free)\(", f.read()), name
