"""The library's host helpers, compiled on their own."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2003_03931_amd", "csrc")


def _run(tmp_path, body):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host compiler")
    src = tmp_path / "t.cpp"
    src.write_text('#include "hostutil.h"\n#include <cstdio>\n#include <vector>\nusing namespace cube;\n'
                   "int main() {\n" + body + "\nreturn 0;\n}\n")
    exe = str(tmp_path / "t")
    subprocess.run([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", exe], check=True)
    return subprocess.run([exe], check=True, capture_output=True, text=True).stdout.split("\n")


def test_key_bits_hold_every_cell_and_no_more(tmp_path):
    """A power-of-two number of cells needs no spare bit: 24 bits (three sort passes) at 256 cells a side."""
    sides = [12, 16, 48, 80, 112, 128, 160, 256, 384, 512, 1024]
    out = _run(tmp_path, "".join(f'printf("%d\\n", key_bits({s}LL * {s} * {s}));' for s in sides))
    assert [int(x) for x in out if x] == [(s ** 3 - 1).bit_length() for s in sides]


def test_copies_run_together_within_an_allocation_only(tmp_path):
    """Arrays that follow each other on both sides are one copy, but not across allocations that are
    neighbours, after a gap on either side, or past an error."""
    out = _run(tmp_path, r'''
static char from[64], to[64];
// allocations of the source: [0, 24) and [24, 64); the destination is one
auto one = [](const void*, const void* s, size_t n) {
    const long at = (const char*)s - from;
    return at + (long)n <= (at < 24 ? 24 : 64);
};
int fail = 0;
auto copy = [&](void* d, const void* s, size_t n) {
    printf("%ld %ld %d;", (long)((char*)d - to), (long)((const char*)s - from), (int)n);
    return fail;
};
auto run = [&](std::vector<std::vector<int>> parts) {
    CopyRuns<decltype(copy), decltype(one)> c(copy, one);
    int e = 0;
    for (auto& p : parts)
        if ((e = c.add(to + p[0], from + p[1], p[2]))) break;
    if (!e) e = c.flush();
    printf(" %d\n", e);
};
run({{0, 0, 8}, {8, 8, 8}, {16, 16, 8}});
run({{0, 0, 8}, {8, 8, 16}, {24, 24, 8}, {32, 32, 8}});
run({{0, 0, 8}, {9, 8, 8}, {17, 17, 7}});
run({{8, 8, 8}, {0, 0, 8}});
run({});
fail = 3;
run({{0, 0, 8}, {24, 24, 8}, {32, 32, 8}});''')
    assert out[:6] == ["0 0 24; 0", "0 0 24;24 24 16; 0", "0 0 8;9 8 8;17 17 7; 0", "8 8 8;0 0 8; 0", " 0", "0 0 8; 3"]
