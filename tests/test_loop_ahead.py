"""Which pieces the host keeps in flight ahead of the device loop (csrc/ahead.h, host C++), run against
sequences of phases: never more than asked for, as many as asked for once the pattern of the rebalancing
rounds is known, and always the piece the loop waits for."""
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# phases: J R(ebalance) L(rollback); reads "lead slots rb_only phases", prints
# "pieces launched, most reports in flight, pieces whose phase the loop was not in"
DRIVER = r"""
#include "ahead.h"
#include <stdio.h>
#include <string.h>
#include <deque>
#include <vector>
int main() {
  char text[1 << 16];
  int lead, slots, rb_only;
  while (scanf("%d %d %d %65535s", &lead, &slots, &rb_only, text) == 4) {
    jet::Ahead a(rb_only != 0, lead);
    std::vector<int> want;
    for (char *c = text; *c; ++c) want.push_back(*c == 'J' ? jet::kPhJet : *c == 'R' ? jet::kPhRb : jet::kPhRoll);
    std::deque<int> queue = {jet::kPhAny};
    size_t at = 0;          // the phase the loop is in
    int rounds = 0, pieces = 0, most = 0, idle = 0;
    uint32_t seq = 0;
    bool ok = true;
    while (ok && !a.done()) {
      const int add = a.want();
      if (add >= 0 && a.room(add == jet::kPhRb ? slots : 1)) {
        const int n = add == jet::kPhRb ? slots : 1;
        a.launched(add, n);
        for (int i = 0; i < n; ++i) queue.push_back(add);
        ++pieces;
        if (a.in_flight() > most) most = a.in_flight();
        if (pieces > 1000000) ok = false;
        continue;
      }
      if (queue.empty()) { ok = false; break; }  // nothing runs and nothing is launched
      const int ph = queue.front();
      queue.pop_front();
      ++seq;
      if (ph == jet::kPhAny) {
      } else if (at < want.size() && want[at] == ph) {
        if (ph == jet::kPhJet) rounds = 0;
        if (ph == jet::kPhRb) ++rounds;
        ++at;
      } else {
        ++idle;
      }
      jet::LoopMail m{};
      m.seq = seq & jet::kMailSeqMask;
      m.phase = at < want.size() ? want[at] : (int)jet::kPhDone;
      m.rb_rounds = rounds;
      a.report(m);
    }
    printf("%d %d %d %d\n", ok ? 1 : 0, pieces, most, idle);
  }
}
"""


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    d = tmp_path_factory.mktemp("ahead")
    (d / "driver.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I",
                    os.path.join(ROOT, "paper_2504_12013_amd", "csrc"), str(d / "driver.cpp"), "-o", str(d / "driver")],
                   check=True)

    def go(lead, phases, slots=1, rb_only=0):
        out = subprocess.run([str(d / "driver")], input=f"{lead} {slots} {rb_only} {phases}\n", check=True,
                             capture_output=True, text=True).stdout.split()
        ok, pieces, most, idle = map(int, out)
        assert ok
        return pieces, most, idle
    return go


def need(phases):
    return len(phases)


@pytest.mark.parametrize("pattern", ["J", "JRR", "JR", "JRRJR"])
def test_one_in_flight_launches_what_runs(run, pattern):
    phases = pattern * 40 + "L"
    pieces, most, idle = run(1, phases)
    assert pieces == need(phases) and idle == 0 and most <= 2  # the set-up's report beside the first piece


@pytest.mark.parametrize("lead", [2, 3, 4, 8, 64, 1024])
@pytest.mark.parametrize("pattern", ["J", "JRR", "JRRR"])
def test_as_many_in_flight_as_asked_for(run, lead, pattern):
    phases = pattern * 200 + "L"
    pieces, most, idle = run(lead, phases)
    assert most >= min(lead, 256)  # pieces ahead, not only the current one
    assert most <= min(lead, 256) + 1
    assert pieces - need(phases) == idle
    assert idle <= 4 * lead + 8    # while the pattern is learnt, and where the round ends


@pytest.mark.parametrize("seed", range(40))
def test_any_sequence_is_followed(run, seed):
    rng = random.Random(seed)
    phases = "".join("J" + "R" * rng.choice([0, 0, 1, 2, rng.randint(0, 20)]) + "L" * (rng.random() < 0.05)
                     for _ in range(150)) + "L"
    for lead in (1, 2, 5, 300):
        for slots in (1, 3, 64):
            pieces, most, _ = run(lead, phases, slots)
            assert most <= max(lead, 2) + 2 * slots
    run(2, "R" * 30, 1, 1)
    run(16, "R" * 30, 1, 1)
