"""CPU check of the tags a polling host waits for: none is 0, none repeats, and
consecutive ones stay one apart, across the powers of two at which a counter
of fewer bits would wrap."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = r"""
#include <cstdio>
#include <cstdlib>
#include "bmg_tags.h"
int main(int, char **argv)
{
    hbmg::Tags t;
    t.last = std::strtoull(argv[1], nullptr, 10);
    double prev = (double)t.last;
    int bad = 0;
    for (int solve = 0; solve < 64; ++solve) {
        const double norm = t.next();              // ||b||'s tag
        const double first = t.take(500);          // then a cycle's each
        bad += norm == 0.0 || norm != prev + 1.0 || first != norm + 1.0 || first + 1.0 == first;
        prev = first + 499.0;
        bad += prev != (double)t.last;
    }
    std::printf("bad %d\n", bad);
    return bad != 0;
}
"""


@pytest.mark.parametrize("start", [0, 2**20 - 250, 2**31 - 250, 2**32 - 250, 2**52 - 250])
def test_tags_neither_repeat_nor_vanish(tmp_path, start):
    (tmp_path / "tags.cpp").write_text(SRC)
    exe = tmp_path / "tags"
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_1803_02481_amd", "csrc"),
                    str(tmp_path / "tags.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe), str(start)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
