"""Moving a plan to another stream, on the host: the helper itself, and that
nothing else in the library assigns a plan's stream after its creation."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2304_12597_amd", "csrc")


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
def test_inner_plan_follows(tmp_path):
    exe = tmp_path / "plan_stream"
    src = os.path.join(HERE, "native", "plan_stream.cpp")
    r = subprocess.run(["hipcc", "-std=c++17", "-O0", "-x", "hip", "--offload-arch=gfx950",
                        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                        src, "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "ok" in r.stdout, r.stdout + r.stderr


def test_one_place_moves_a_plan():
    found = []
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".h", ".hip")):
            continue
        with open(os.path.join(CSRC, name)) as fh:
            for line in fh:
                if re.search(r"->stream\s*=[^=]", line):
                    found.append((name, line.strip()))
    # the creation (plan and options) and the helper, the plan and its inner plan
    assert [f for f in found if f[0] not in ("plan.hip", "pd_internal.h")] == []
    assert len([f for f in found if f[0] == "plan.hip"]) == 2
    assert len([f for f in found if f[0] == "pd_internal.h"]) == 2
