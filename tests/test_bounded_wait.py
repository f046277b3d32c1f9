"""A block's wait for words that other blocks write (csrc/bounded_wait.h): it ends whatever the words hold.  Compiled for the host, with
words that never come; on the GPU every wait ends well (test_gpu_chain.py)."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1904_07421_amd", "csrc")

PROGRAM = r"""
#include "bounded_wait.h"
#include <cstdio>
int main() {
    int rests = 0, at = 0, looks = 3, word = 7;
    auto rest = [&] { ++rests; };
    auto look = [&](int least) { return word >= least; };
    auto say = [&](bool ok) { std::printf("%d %d %d\n", ok, rests, looks); };
    say(jitdb::wait_bounded(7, looks, look, rest));                              // there at once: one look is used
    looks = 10;
    say(jitdb::wait_bounded(8, looks, [&](int least) { word += ++at == 4; return look(least); }, rest));   // comes late
    word = -2147483647 - 1; rests = 0;
    say(jitdb::wait_bounded(8, looks, look, rest));                              // never comes: what is left of the looks
    looks = 0;
    say(jitdb::wait_bounded(8, looks, look, rest));                              // ... and nothing is left for the next
    word = 8; looks = 0;
    say(jitdb::wait_bounded(8, looks, look, rest));
}
"""


def test_the_wait_ends(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "wait.cpp", tmp_path / "wait"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=20).stdout.split("\n")
    assert out[:5] == ["1 1 2", "1 5 6", "0 7 -1", "0 8 -1", "0 9 -1"], out
