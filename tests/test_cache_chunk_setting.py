"""A saved chunk setting put back leaves the cache as it was: the length a new
cache reports stands for lengths chosen by the solve, any other is fixed
(compiled from the library's header and run on the host)."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include "hbf_internal.h"
int main() {
  const uint64_t R[] = {64, 20000, uint64_t(1) << 26};
  const uint32_t F[] = {64, 10000, 1000000, 1u << 23};
  for (uint64_t r : R)
    for (uint32_t f : F) {
      const uint32_t saved = hbf::chunk_default(f, r);
      if (saved == 0 || hbf::chunk_asked(saved, f, r) != 0) return 1;
      for (uint32_t set : {1u, 1000u, saved - 1, saved + 1, hbf::CHUNK_MAX})
        if (set != saved && hbf::chunk_asked(set, f, r) != set) return 2;
    }
  return 0;
}
"""


def test_a_saved_setting_put_back(tmp_path):
    src, exe = tmp_path / "c.cpp", tmp_path / "c"
    src.write_text(PROGRAM)
    inc = [os.path.join(ROOT, "include"), os.path.join(ROOT, "paper_2609_09800_amd", "csrc"), "/opt/rocm/include"]
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", *[f"-I{i}" for i in inc], str(src), "-o", str(exe)],
                   check=True)
    assert subprocess.run([str(exe)]).returncode == 0
    api = open(os.path.join(inc[1], "hbf_api.cpp")).read()
    assert "chunk_asked(c->chunk, c->F, c->R)" in api
