"""The barrier of the workgroups that serve one frame cache together, on the
host: its counter only grows during a call and wraps after 2^32 arrivals
(256 workgroups, eight barriers a chunk: two million chunks), which must not
open a barrier early or keep it shut."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2609_09800_amd", "csrc")

PROGRAM = r"""
#include "hbf_group.h"
#include <cstdio>
int main() {
  const uint32_t nb = NB;
  // 4,096 barriers ending 2,048 past the wrap; `done` counts arrivals without wrapping
  uint64_t done = (uint64_t(1) << 32) - 2048ull * nb;
  for (int b = 0; b < 4096; b++) {
    const uint32_t target = (uint32_t)(done + nb);
    for (uint32_t a = 0; a <= nb; a++)  // a workgroups have arrived
      if (hbf::counter_reached((uint32_t)(done + a), target) != (a == nb)) {
        std::printf("barrier %d of %u: %u arrived\n", b, nb, a);
        return 1;
      }
    // the last to look may see arrivals at the next barrier
    for (uint32_t a = 0; a < nb; a++)
      if (!hbf::counter_reached((uint32_t)(done + nb + a), target)) return 2;
    done += nb;
  }
  return 0;
}
"""


@pytest.mark.parametrize("nb", [1, 3, 256])
def test_barrier_counter_wraps(tmp_path, nb):
    src, exe = tmp_path / "b.cpp", tmp_path / "b"
    src.write_text(PROGRAM.replace("NB", str(nb)))
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


JOIN = r"""
#include "hbf_group.h"
#include <atomic>
#include <cstdio>
#include <random>
#include <thread>
#include <vector>
struct Shared { std::atomic<uint32_t> arrived{0}, members{0}; };
struct Words {
  Shared &s;
  int patience;
  uint32_t arrive() { return s.arrived.fetch_add(1); }
  uint32_t close() { return s.arrived.fetch_or(hbf::GROUP_CLOSED); }
  uint32_t count() { return s.members.load(); }
  void set_count(uint32_t n) { s.members.store(n); }
  bool wait() { std::this_thread::yield(); return patience-- > 0; }
};
int main() {
  std::mt19937 rng(SEED);
  for (int round = 0; round < 400; round++) {
    const uint32_t want = 1 + rng() % 8, room = 1 + rng() % want;  // `room` run at a time
    const int patience = rng() % 3 ? 200 : 0;
    Shared s;
    std::atomic<uint32_t> next{0}, barrier{0};
    std::vector<hbf::Member> got(want);
    auto slot = [&] {  // takes one workgroup after another, each to its end
      for (uint32_t g; (g = next.fetch_add(1)) < want;) {
        Words w{s, patience};
        const hbf::Member m = hbf::group_join(w, want);
        got[g] = m;
        uint32_t target = 0;
        for (int b = 0; m.count && b < 3; b++) {  // members meet, and only they
          target += m.count;
          barrier.fetch_add(1);
          while (!hbf::counter_reached(barrier.load(), target)) std::this_thread::yield();
        }
      }
    };
    std::vector<std::thread> t;
    for (uint32_t i = 0; i < room; i++) t.emplace_back(slot);
    for (auto &x : t) x.join();
    uint32_t n = 0, seen = 0;
    for (auto &m : got)
      if (m.count) {
        if (n && m.count != n) return std::printf("round %d: counts %u and %u\n", round, n, m.count), 1;
        n = m.count;
        if (m.id >= n || (seen >> m.id & 1)) return std::printf("round %d: id %u\n", round, m.id), 1;
        seen |= 1u << m.id;
      }
    if (!n || seen != (1u << n) - 1) return std::printf("round %d: members %x of %u\n", round, seen, n), 1;
  }
  return 0;
}
"""


@pytest.mark.parametrize("seed", range(3))
def test_members_never_wait_for_workgroups_without_room(tmp_path, seed):
    """Threads as workgroups, fewer of them at a time than the launch has:
    the members agree on their number, each has a number of its own, all
    meet at barriers, and the workgroups that start later leave."""
    src, exe = tmp_path / "j.cpp", tmp_path / "j"
    src.write_text(JOIN.replace("SEED", str(seed)))
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
