"""Hand-overs between workgroups of one launch are ordered by the language's memory model, not by what
a GPU happens to do: in the intermediate code of the hub pass, compiled here, a workgroup's arrival is
a release at device scope, and an acquire fence follows it."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no HIP compiler")
def test_hub_rows_are_handed_over_by_release_and_acquire(tmp_path):
    src = tmp_path / "probe.hip"
    src.write_text('#include "hub.h"\n'
                   "__global__ __launch_bounds__(jet::kHubBlock) void probe(jet::HubArgs a) {\n"
                   "  jet::hub_work<1, 1, true, false>(a, (int32_t)blockIdx.x, (int32_t)gridDim.x);\n"
                   "}\n")
    out = tmp_path / "probe.ll"
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-device-only", "-S", "-emit-llvm",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                    "-I", os.path.join(ROOT, "paper_2504_12013_amd", "csrc"), "-I", os.path.join(ROOT, "include"),
                    str(src), "-o", str(out)], check=True, capture_output=True)
    code = out.read_text()
    body = code[code.index("@_Z5probeN3jet7HubArgsE"):]
    arrival = re.search(r'= atomicrmw add ptr addrspace\(1\) .* i32 1 syncscope\("agent"\) (release|acq_rel)', body)
    assert arrival
    assert arrival.group(1) == "acq_rel" or 'fence syncscope("agent") acquire' in body[arrival.end():]
    assert "s_waitcnt" not in body
