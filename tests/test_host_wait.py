"""The one wait between workgroups in the library ends, also if what it waits for never comes (qg_wait.h on the CPU)."""
import os
import re
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2504_12984_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "qg_wait.h"
int main() {
  unsigned looks = 0, pauses = 0, count = 0;
  auto pause = [&] { ++pauses; };
  const bool came = qg::wait_for([&] { return ++looks == 5 ? count = 2 : count; }, 2u, pause);         // at the fifth look
  std::printf("%d %u %u\n", came, looks, pauses);
  looks = pauses = 0;
  const bool beyond = qg::wait_for([&] { ++looks; return 3u; }, 2u, pause);                              // another call's counts
  std::printf("%d %u %u\n", beyond, looks, pauses);
  looks = pauses = 0;
  const bool never = qg::wait_for([&] { ++looks; return 1u; }, 2u, pause);
  std::printf("%d %d %d\n", never, looks == qg::WAIT_LIMIT, pauses == qg::WAIT_LIMIT);
}
"""


def test_the_wait_ends(tmp_path):
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++20", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout
    assert out.splitlines() == ["1 5 4", "1 1 0", "0 1 1"]


def test_no_kernel_waits_in_a_loop_of_its_own():
    # a loop whose condition reads a counter of other workgroups would be a wait without an end
    for name in sorted(os.listdir(CSRC)):
        text = open(os.path.join(CSRC, name)).read()
        assert not re.search(r"\bwhile\s*\([^;{]*__hip_atomic", text), name
        assert not re.search(r"\bfor\s*\([^;]*;[^;]*__hip_atomic", text), name
