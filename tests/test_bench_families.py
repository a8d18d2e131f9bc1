"""The benchmark's kernel families follow the kernels: every name it sums exists, a kernel belongs to one
family, and the hub pass is booked with the pass it serves."""
import csv
import os
import re
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402

CSRC = os.path.join(ROOT, "paper_2504_12013_amd", "csrc")
OLDER = {"k_apply_chunks", "k_apply_nets"}  # in traces of older builds


def kernels():
    names = set()
    for f in os.listdir(CSRC):
        if f.endswith(".hip"):
            names |= set(re.findall(r"__global__\s+(?:__launch_bounds__\((?:[^()]|\([^()]*\))*\)\s*)?void (k_\w+)\(",
                                    open(os.path.join(CSRC, f)).read()))
    return names


def test_families_name_kernels_once():
    seen = [k for heads, rest in bench.FAMILIES.values() for k in heads + rest]
    assert len(seen) == len(set(seen))
    assert set(seen) - OLDER <= kernels()


def test_loop_kernels_are_booked():
    phase = {k for k in kernels() if re.match(r"k_(candidates|hub|ab_|rg_|select_moves|apply|rb_)", k)}
    phase -= {"k_rb_prepare", "k_rb_prepare_union"}  # before the marks of the round
    booked = {k for heads, rest in bench.FAMILIES.values() for k in heads + rest}
    assert phase <= booked


def test_hub_passes_are_told_apart(tmp_path, capsys):
    with open(tmp_path / "t_kernel_stats.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Name", "Calls", "TotalDurationNs", "AverageNs"])
        w.writerow(["void jet::(anonymous namespace)::k_hub<1, 2, true>(jet::HubArgs)", 3, 30e6, 10e6])
        w.writerow(["void jet::(anonymous namespace)::k_rb_hub<1, 2, true>(jet::HubArgs)", 5, 100e6, 20e6])
        w.writerow(["jet::(anonymous namespace)::k_rb_list(int*)", 5, 5e6, 1e6])
    bench.summarize(str(tmp_path), 0)
    rows = {line.split()[0]: line.split() for line in capsys.readouterr().out.splitlines()[1:]}
    assert rows["candidates_hub"][1] == "3" and float(rows["candidates_hub"][2]) == pytest.approx(30.0)
    assert rows["rebalance_gain"][1] == "5" and float(rows["rebalance_gain"][2]) == pytest.approx(105.0)
