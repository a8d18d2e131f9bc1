"""The rating-table rule of the clustering: one function that the host (which lays out the tables in scratch)
and the device (which decides whether a vertex has one there) both compile, and one LDS limit."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12013_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def want(d, n):
    if d <= 0:
        return 0
    t = 16
    while t < 2 * min(d, n):
        t *= 2
    return t


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no HIP compiler")
def test_host_rule(tmp_path):
    src, exe = tmp_path / "rule.hip", tmp_path / "rule"
    src.write_text('#include <stdio.h>\n#include "jet_internal.h"\n'
                   "int main() {\n"
                   "  long long d, n;\n"
                   '  while (scanf("%lld %lld", &d, &n) == 2) printf("%lld\\n", (long long)jet::co_table(d, n));\n'
                   "}\n")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    sizes = sorted({0, 1, 3, 7, 1 << 40} | {(1 << b) + o for b in range(3, 31) for o in (-1, 0, 1)})
    pairs = [(d, n) for d in sizes for n in sizes if 1 <= n < 1 << 31]
    out = subprocess.run([str(exe)], input="".join(f"{d} {n}\n" for d, n in pairs), check=True, capture_output=True,
                         text=True).stdout.split()
    assert [int(x) for x in out] == [want(d, n) for d, n in pairs]


def test_one_definition():
    text = {f: open(os.path.join(CSRC, f)).read() for f in os.listdir(CSRC) if f.endswith((".h", ".hip", ".cpp"))}
    defs = [f for f, s in text.items() for _ in re.finditer(r"__host__ __device__ inline int64_t co_table\(", s)]
    assert defs == ["jet_internal.h"]
    assert len(re.findall(r"kCoLds\w+ = ", "".join(text.values()))) == 2  # the LDS limit, the small form's
