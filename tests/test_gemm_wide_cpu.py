"""CPU check of the GEMM launches beside the square tiles (plan_wide and the
streaming kernel's block map in `csrc/gemm_plan.h`, built for the host):
`tests/gemm_wide_check.cpp` over ragged row counts, widths and workspaces."""
import os
import shutil
import subprocess

import pytest

from wide_cases import CASES, WORKSPACE

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    hipcc = shutil.which("hipcc")
    if not hipcc:
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("wide") / "gemm_wide_check")
    cmd = [hipcc, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2503_17707_amd", "csrc"),
           os.path.join(HERE, "gemm_wide_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-4000:]
    return exe


def test_wide_launches_cover_every_product_once(exe):
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    print(r.stdout)
    assert r.returncode == 0 and " 0 failures" in r.stdout, r.stdout[-4000:]


def test_plans_of_the_compared_products(exe):
    for M, N, K, _, plan in CASES:
        r = subprocess.run([exe] + [str(v) for v in (M, N, K, WORKSPACE)], capture_output=True, text=True, timeout=60)
        assert r.stdout.strip() == plan, (M, N, K)
