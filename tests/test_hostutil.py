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
