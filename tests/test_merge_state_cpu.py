"""CPU check of merged-adapter state over failing HIP calls:
`tests/merge_state_check.cpp` builds the library's host runtime
(`csrc/model.cpp`) against stand-ins for its HIP calls and kernel launchers."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def test_failed_merges_never_leave_weights_to_build_on(tmp_path):
    hipcc = shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not available")
    exe = str(tmp_path / "merge_state_check")
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-fuse-cuid=none", "-O1", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "paper_2503_17707_amd", "csrc"),
           os.path.join(HERE, "merge_state_check.cpp"), "-o", exe, "-lpthread"]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and r.stdout.endswith("0 failures\n"), r.stdout[-4000:]
