"""Hand-overs between workgroups of one launch hold by the language's memory model, not by what a GPU happens
to do.  The hub pass passes sums through words that only relaxed atomics at device scope touch and that
need no order between them (csrc/hand_over.h): the compiled pass is looked at here, and the words are run by
host threads under ThreadSanitizer."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2504_12013_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


@pytest.mark.skipif(not shutil.which(HIPCC), reason="no HIP compiler")
@pytest.mark.parametrize("rb", ["false", "true"])
def test_hub_words_are_touched_by_atomics_only(tmp_path, rb):
    src = tmp_path / "probe.hip"
    src.write_text('#include "hub.h"\n'
                   "__global__ __launch_bounds__(jet::kHubBlock) void probe(jet::HubArgs a) {\n"
                   f"  jet::hub_work<1, 1, true, {rb}>(a, (int32_t)blockIdx.x, (int32_t)gridDim.x);\n"
                   "}\n")
    out = tmp_path / "probe.ll"
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-device-only", "-S", "-emit-llvm",
                    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", CSRC,
                    "-I", os.path.join(ROOT, "include"), str(src), "-o", str(out)], check=True, capture_output=True)
    code = out.read_text()
    body = code[code.index("@_Z5probeN3jet7HubArgsE"):]
    agent = r'syncscope\("agent"\) monotonic'
    word = re.findall(rf"= load atomic i64, ptr addrspace\(1\) (%\S+) {agent}", body)
    assert len(word) == 1
    w = re.escape(word[0])
    assert len(re.findall(rf"store atomic i64 0, ptr addrspace\(1\) {w} {agent}", body)) == 1
    assert len(re.findall(rf"addrspace\(1\) {w}\b", body)) == 2  # the loop that takes the word
    assert re.search(rf"= atomicrmw add ptr addrspace\(1\) %\S+, i64 %\S+ {agent}", body)
    assert "s_waitcnt" not in body


DRIVER = r"""
#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
#include "hand_over.h"
#include <pthread.h>
#include <stdio.h>
#include <stdlib.h>
#include <thread>
#include <vector>
int main(int, char **argv) {
  const int shares = atoi(argv[1]), columns = atoi(argv[2]), launches = atoi(argv[3]);
  std::vector<unsigned long long> words(columns, 0ull);
  std::vector<int> took(launches, 0), wrong(shares, 0);
  pthread_barrier_t end;  // a launch ends before the next one begins
  pthread_barrier_init(&end, nullptr, shares);
  auto value = [](int l, int s, int c) { return (int32_t)((unsigned)(l * 7919 + s * 104729 + c * 31) % 50000000u); };
  std::vector<std::thread> th;
  for (int s = 0; s < shares; ++s)
    th.emplace_back([&, s] {
      for (int l = 0; l < launches; ++l) {
        bool last = false;
        for (int x = 0; x < columns; ++x) {  // from another column each: the last column is not added last
          const int c = (x + s * 5 + l) % columns;
          const bool all = jet::word_add(&words[c], value(l, s, c), shares);
          if (c == columns - 1) last = all;
        }
        if (last) {
          __atomic_fetch_add(&took[l], 1, __ATOMIC_RELAXED);
          for (int c = 0; c < columns; ++c) {
            int32_t sum = -1;
            int64_t want = 0;
            for (int q = 0; q < shares; ++q) want += value(l, q, c);
            if (!jet::word_take(&words[c], shares, &sum) || sum != want) ++wrong[s];
          }
        }
        pthread_barrier_wait(&end);
      }
    });
  for (auto &t : th) t.join();
  int bad = 0;
  for (int w : wrong) bad += w;
  for (int t : took) bad += t != 1;
  for (unsigned long long w : words) bad += w != 0ull;
  printf("%d\n", bad);
  return bad != 0;
}
"""


@pytest.mark.parametrize("shares,columns,launches", [(2, 1, 400), (2, 129, 60), (5, 33, 100), (16, 65, 30)])
def test_words_hand_over_under_thread_sanitizer(tmp_path, shares, columns, launches):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-I", CSRC, str(src), "-o", str(exe),
                    "-lpthread"], check=True, capture_output=True)
    run = subprocess.run([str(exe), str(shares), str(columns), str(launches)], capture_output=True, text=True,
                         timeout=120)
    assert run.returncode == 0 and run.stdout.strip() == "0", run.stdout + run.stderr
