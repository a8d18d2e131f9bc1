"""The grid of a move application on the host: the workgroups that sum the block weights of a list stride by
a fixed count, so no grid may be smaller, however few workgroups a card or a partition of one holds."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12013_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no HIP compiler")
def test_grid_holds_the_weight_blocks(tmp_path):
    src, exe = tmp_path / "grid.hip", tmp_path / "grid"
    src.write_text('#include <stdio.h>\n#include "jet_internal.h"\n'
                   "int main() {\n"
                   "  long long fits, groups;\n"
                   '  printf("%u\\n", jet::kWeightBlocks);\n'
                   '  while (scanf("%lld %lld", &fits, &groups) == 2)\n'
                   '    printf("%lld\\n", (long long)jet::apply_grid(fits, groups));\n'
                   "}\n")
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-host-only", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(exe)], check=True, capture_output=True)
    pairs = [(f, g) for f in (8, 32, 63, 64, 65, 1024, 2048, 4096) for g in (0, 1, 3000, 1 << 30)]
    out = subprocess.run([str(exe)], input="".join(f"{f} {g}\n" for f, g in pairs), check=True, capture_output=True,
                         text=True).stdout.split()
    blocks = int(out[0])
    assert [int(x) for x in out[1:]] == [max(min(f, 2048), min(g, 1 << 20), blocks) for f, g in pairs]


def test_the_kernel_strides_by_that_count():
    text = open(os.path.join(CSRC, "k_iter.hip")).read()
    assert re.search(r"blockIdx\.x < kWeightBlocks", text) and "apply_grid(" in text
