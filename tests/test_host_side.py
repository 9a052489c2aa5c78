"""Host code of the library that no call reaches without a GPU, compiled on its own with the host
compiler: the split of a launch over the grid's dimensions."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _run(tmp_path, source, *args):
    """Output lines of a C++ program that sees the library's headers and links nothing of HIP."""
    src, exe = tmp_path / "prog.cpp", tmp_path / "prog"
    src.write_text(source)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2604_18556_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe), *args], check=True, capture_output=True, text=True)
    return r.stdout.splitlines()


SPLIT = r"""
#include "gsq_internal.h"
#include <cstdio>
#include <cstdlib>
int main(int argc, char** argv) {
  for (int i = 1; i + 1 < argc; i += 2) {
    const gsq::RowSplit s = gsq::split_rows(std::atoll(argv[i]), std::atoll(argv[i + 1]));
    std::printf("%d %u %u\n", s.rows_x, s.gx, s.gy);
  }
}
"""
EDGE = (1 << 24) - 1   # workgroups of 256 threads in one dimension: 2^32 - 256 threads


def test_rows_split_over_the_grid(tmp_path):
    """(rows, workgroups per row): every row has its place (y rows_x + x / cols covers 0 .. rows - 1,
    each once), and no dimension holds 2^32 threads; layers that fit one dimension keep one."""
    cases = [(1, 1), (7, 3), (EDGE, 1), (EDGE + 1, 1), (1 << 24, 2), (17_000_015, 1), (1 << 30, 1),
             (EDGE // 2, 2), (EDGE // 2 + 1, 2), (5, EDGE // 5), (6, EDGE // 5), (70_000, 256),
             (1, 65536), (255, 65536), (256, 65536), (2000, 65536)]
    lines = _run(tmp_path, SPLIT, *(str(x) for c in cases for x in c))
    assert len(lines) == len(cases)
    for (rows, cols), line in zip(cases, lines):
        rows_x, gx, gy = map(int, line.split())
        assert gx == rows_x * cols and 0 < gx <= EDGE, (rows, cols, line)
        assert (gy - 1) * rows_x < rows <= gy * rows_x and 0 < gy <= 65535, (rows, cols, line)
        assert gy == 1 or (rows_x + 1) * cols > EDGE, (rows, cols, line)
