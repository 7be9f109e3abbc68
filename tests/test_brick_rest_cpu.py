"""After a launch of bricks that did not find its workgroups together a context
rests from them for a while, not for good (host check of the rule)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc to build the host check")
def test_rests(tmp_path):
    exe = str(tmp_path / "brick_rest_check")
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-I", os.path.join(ROOT, "paper_1302_3663_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                           "-x", "hip", os.path.join(HERE, "brick_rest_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(out.stdout)
    assert out.returncode == 0 and out.stdout.startswith("0 mismatches"), out.stdout + out.stderr
