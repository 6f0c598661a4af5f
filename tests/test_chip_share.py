"""The rule that keeps the group launches of a process from holding CUs that each other's workgroups wait for
(csrc/nmfa_share.h), on the CPU: streams enqueue launches of random widths, each behind the waits that the rule
gives it; a device starts any launch whose stream predecessor and waits are complete, and completes started ones in
random order. At no time may the widths of the started launches exceed the CUs, and all must end. Without the
waits the same schedules do exceed them."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1806_08422_amd", "csrc")

PROGRAM = r"""
#include "nmfa_share.h"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <set>
using namespace nmfa;
struct L { int width, prev; std::vector<int> waits; bool started, done; };
int main(int, char** argv) {
  const bool obey = atoi(argv[1]);
  const int cus = 256, streams = atoi(argv[2]);
  std::mt19937 g(atoi(argv[3]));
  auto pick = [&](int n) { return (int)(g() % n); };
  ChipShare s;
  std::vector<L> all;
  std::vector<int> ev_launch;             // event -> the launch it was last recorded behind
  std::vector<size_t> pool;
  std::vector<int> last(streams, -1);
  int over = 0, most = 0, events = 0;
  auto key = [](int st) { return (void*)(size_t)(st + 1); };
  auto check = [&] {
    int sum = 0;
    for (auto& l : all) sum += l.started && !l.done ? l.width : 0;
    most = std::max(most, sum);
    over += sum > cus;
  };
  auto device = [&](bool drain) {  // start all that may start, complete one or more
    do {
      for (auto& l : all) {
        bool ok = !l.started && (l.prev < 0 || all[l.prev].done);
        for (int w : l.waits) ok = ok && all[w].done;
        if (ok) l.started = true;
      }
      check();
      std::vector<int> run;
      for (int k = 0; k < (int)all.size(); ++k) if (all[k].started && !all[k].done) run.push_back(k);
      if (run.empty()) break;
      all[run[pick(run.size())]].done = true;
    } while (drain);
  };
  for (int step = 0; step < 400; ++step) {
    const int st = pick(streams), width = ChipShare::rounded(1 + pick(pick(3) ? 64 : 256));
    auto release = [&](void* e) { pool.push_back((size_t)e - 1); };
    s.reap([&](void* e) { return (bool)all[ev_launch[(size_t)e - 1]].done; }, release);
    L l{width, last[st], {}, false, false};
    if (obey) for (void* e : s.waits(key(st), width, cus)) l.waits.push_back(ev_launch[(size_t)e - 1]);
    size_t ev;
    if (pool.empty()) { ev = ev_launch.size(); ev_launch.push_back(0); ++events; }
    else { ev = pool.back(); pool.pop_back(); }
    ev_launch[ev] = (int)all.size();
    s.add(key(st), width, (void*)(ev + 1), release);
    last[st] = (int)all.size();
    all.push_back(l);
    while (pick(3)) device(false);
  }
  device(true);
  int left = 0;
  for (auto& l : all) left += !l.done;
  s.reap([&](void*) { return true; }, [](void*) {});
  int held = 0;
  printf("%d %d %d %d %d", over, left, most, events, s.others(nullptr, &held) + held);
}
"""


@pytest.fixture(scope="module")
def simulate(tmp_path_factory):
    d = tmp_path_factory.mktemp("share")
    (d / "sim.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", CSRC, str(d / "sim.cpp"), "-o", str(d / "sim")])
    return lambda *a: [int(x) for x in subprocess.check_output([str(d / "sim"), *map(str, a)], text=True).split()]


@pytest.mark.parametrize("streams", [1, 2, 3, 8, 40])
@pytest.mark.parametrize("seed", [1, 2, 3])
def test_running_launches_fit(simulate, streams, seed):
    over, left, most, events, rest = simulate(1, streams, seed)
    assert over == 0 and left == 0 and most <= 256 and rest == 0
    assert events <= 32 * streams + 1  # unfinished launches kept per stream: one per width
    if streams > 1:
        assert simulate(0, streams, seed)[0] > 0


def test_reservations(tmp_path_factory):
    d = tmp_path_factory.mktemp("reserve")
    (d / "r.cpp").write_text(r"""
#include "nmfa_share.h"
#include <cstdio>
int main() {
  nmfa::ChipShare s;
  int a = 0, b = 0;
  s.reserve(&a, 64); s.reserve(&a, 32); s.reserve(&b, 8);
  printf("%d %d %d ", s.reserved_by_others(&a), s.reserved_by_others(&b), s.reserved_by_others(nullptr));
  s.unreserve(&a);
  printf("%d %d", s.reserved_by_others(&b), nmfa::ChipShare::rounded(41));
}""")
    subprocess.check_call(["g++", "-std=c++17", "-I", CSRC, str(d / "r.cpp"), "-o", str(d / "r")])
    assert subprocess.check_output([str(d / "r")], text=True).split() == ["8", "64", "72", "0", "48"]
