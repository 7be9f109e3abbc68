"""The bricks of a V-cycle exchange values through mailboxes without locks:
every workgroup's posts and reads of a launch of several cycles are walked
on the CPU, on the library's own plans, and no entry may be posted again by
a workgroup that does not know of all reads of it.  The same walk must find
the reads out of order of a tail level whose right-hand side is kept once
and read by every workgroup there."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc to build the host check")
def test_mailbox_entries_are_read_before_they_are_posted_again(tmp_path):
    exe = str(tmp_path / "brick_order_check")
    # the kernels' launchers are never called
    subprocess.check_call(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-Wl,--unresolved-symbols=ignore-all",
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                           "-I", os.path.join(ROOT, "paper_1302_3663_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                           "-x", "hip", os.path.join(HERE, "brick_order_check.cpp"), "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    print(out.stdout)
    assert out.returncode == 0 and " 0 mismatches" in out.stdout, out.stdout + out.stderr
