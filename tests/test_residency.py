"""Which passes keep a state in the last-level cache (the host's rule, compiled
by itself)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2609_19147_amd", "csrc")
MIB = 1 << 20

MAIN = r"""
#include "layout.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  const unsigned long long b = std::strtoull(argv[1], 0, 10), o = std::strtoull(argv[2], 0, 10);
  std::printf("%u %u\n", qs::keep_resident(b, o), qs::keep_resident(b, o, 128ull << 20));
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("residency")
    src, exe = d / "main.cpp", d / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src), "-o", str(exe)],
                   check=True)
    return lambda b, o: tuple(int(v) for v in subprocess.run(
        [str(exe), str(b), str(o)], check=True, capture_output=True, text=True).stdout.split())


@pytest.mark.parametrize("bytes_,others,want", [
    (16, 0, (0, 0)), (32, 0, (1, 0)), (64, 0, (1, 0)), (128, 0, (1, 1)), (256, 0, (1, 1)), (512, 0, (0, 0)),
    # a second state (an adjoint sweep): both have to fit
    (64, 64, (1, 0)), (128, 128, (1, 1)), (256, 256, (0, 0)),
    # the states of a batch: 16 of 32 MiB, 8 and 2 of 128 MiB
    (32, 15 * 32, (0, 0)), (128, 7 * 128, (0, 0)), (128, 128, (1, 1))])
def test_states_that_take_turns_fit_together(rule, bytes_, others, want):
    assert rule(bytes_ * MIB, others * MIB) == want
