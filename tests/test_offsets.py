"""Walks through entry offsets near the largest entry count, 2^31 - 2: the
kernels' step counter compiled for the host with the undefined-behaviour
sanitizer, which ends the run at a signed overflow, and a look at the sources
for loops that step an int32 offset past a range's end."""
import glob
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2011_08879_amd", "csrc")

DRIVER = r"""
#include "offsets.hpp"
#include <cstdio>
#include <initializer_list>

template <int32_t S>
int check(int32_t b, int32_t e, int32_t first) {
    int64_t want = (int64_t)b + first;
    for (gko::entry_steps<S> k(b, e, first); k.more(); k.next(), want += S) {
        if (k.at() != want || k.left() != e - want) return 1;
        if (k.count() != (e - want < S ? e - want : S)) return 1;
    }
    return want >= e ? 0 : 1;  // every step was taken
}

template <int32_t S>
int all() {
    const int32_t top = 2147483646;
    const int32_t lens[] = {0, 1, 2, 63, 64, 65, 255, 256, 1023, 2047, 2048, 2049, 4095, 4096, 4097, 10000};
    const int32_t ends[] = {10000, top - 4097, top - 1, top};
    int bad = 0;
    for (int32_t e : ends)
        for (int32_t len : lens)
            for (int32_t first : {0, 1, 63, 255, 319}) bad += check<S>(e - len, e, first);
    return bad;
}

int main() {
    const int bad = all<1>() + all<4>() + all<16>() + all<64>() + all<256>() + all<1024>() + all<2048>() + all<4096>();
    std::printf("bad %d\n", bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host C++ compiler")
def test_steps_near_the_largest_offset(tmp_path):
    src = tmp_path / "steps.cpp"
    src.write_text(DRIVER)
    exe = str(tmp_path / "steps")
    cc = subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                         "-I", CSRC, str(src), "-o", exe], capture_output=True, text=True)
    assert cc.returncode == 0, cc.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout == "bad 0\n", run.stdout + run.stderr[-2000:]


def test_no_int32_offset_is_stepped_past_its_range():
    """for (int32_t k = ...; k < e; k += S) over matrix offsets (rows' begins
    and ends from rp) overflows when e is within S of 2^31."""
    loop = re.compile(r"for \(int32_t (\w+) = (?:b|kb|b\[u\])\b[^;]*; \1 < (?:e|ke|e\[u\]); \1 \+= ")
    bad = []
    for path in sorted(glob.glob(os.path.join(CSRC, "*.h*"))):
        for k, line in enumerate(open(path), 1):
            if loop.search(line):
                bad.append("%s:%d %s" % (os.path.basename(path), k, line.strip()))
    assert not bad, bad
