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
