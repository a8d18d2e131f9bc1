"""The host side of the library names no processor outside spin.h, whose waiting hint compiles for several."""
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_12013_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"


@pytest.mark.skipif(not os.path.exists(CLANG), reason="no clang")
@pytest.mark.parametrize("target", ["x86_64-linux-gnu", "aarch64-linux-gnu", "powerpc64le-linux-gnu",
                                    "riscv64-linux-gnu"])
def test_waiting_hint_compiles(target):
    out = subprocess.run([CLANG, f"--target={target}", "-std=c++17", "-fsyntax-only", "-Wall", "-Werror", "-x", "c++",
                          os.path.join(CSRC, "spin.h"), "-Wno-pragma-once-outside-header"],
                         capture_output=True, text=True)
    if "unknown target" in out.stderr or "No available targets" in out.stderr:
        pytest.skip("target not built into this compiler")
    assert out.returncode == 0, out.stderr


def test_no_other_processor_intrinsics():
    for f in os.listdir(CSRC):
        if f != "spin.h" and f.endswith((".h", ".hip", ".cpp")):
            assert not re.search(r"__builtin_ia32|_mm_|immintrin", open(os.path.join(CSRC, f)).read()), f
