"""Every kernel of the built library has a kind in the profile summaries, and the
GEMM kernels a row of their own in the stall tables."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2503_17707_amd import profsum

LIB = os.path.join(os.path.dirname(os.path.abspath(profsum.__file__)), "lib", "libpipeboost.so")


def test_every_kernel_has_a_kind():
    if not shutil.which("nm") or not os.path.exists(LIB):
        pytest.skip("no nm, or the library is not built")
    out = subprocess.run(["nm", LIB], capture_output=True, text=True, timeout=120, check=True).stdout
    names = sorted(set(re.findall(r"\S*__device_stub__\S*", out)))
    assert len(names) > 300
    assert [n for n in names if profsum.kind_of(n) is None] == []
    kinds = {profsum._base(profsum.kind_of(n)) for n in names}
    assert {"gemm_qkv", "gemm_o", "gemm_fc1", "gemm_fc2", "lora_shrink", "lm_head", "attention", "layernorm"} <= kinds
    gemms = [n for n in names if "gemm_kernel" in n or "pingpong" in n or "stream_kernel" in n]
    assert all("?" not in profsum._gemm_key(n) for n in gemms if profsum.kind_of(n) != "lora_shrink")


def test_kinds_of_traced_names():
    # as a kernel trace names them
    for name, kind, key in [
            ("_ZN2pb12_GLOBAL__N_120gemm_pingpong_kernelIDF16_Li1ELi4ELi2EEEvNS_10GemmParamsENS0_9SplitArgsE", "gemm_fc1",
             "this library 256x256 ping-pong, 8 waves, fc1"),
            ("_ZN2pb12_GLOBAL__N_113stream_kernelIDF16bLi2ELi32ELi64ELi1ELi4ELi256ELi3ELi1EEEvNS_10GemmParamsENS0_9SplitArgsEi",
             "gemm_o", "this library 32x64 streaming, 4 waves, o"),
            ("_ZN2pb12_GLOBAL__N_111gemm_kernelIDF16_Li0ELi128ELi128ELi2ELi4ELi0ELi3EEEvNS_10GemmParamsENS0_9SplitArgsE",
             "gemm_qkv", "this library 128x128, 8 waves, qkv"),
            ("_ZN2pb12_GLOBAL__N_118split_terms_kernelIDF16_EEvPKfiiiPT_Pf", "lm_head terms", None),
            ("_ZN2pb12_GLOBAL__N_117row_shrink_kernelIDF16_Li4ELi4EEEvPKT_iNS_9RowShrinkE", "lora_shrink", None)]:
        assert profsum.kind_of(name) == kind and profsum._gemm_key(name) == key
