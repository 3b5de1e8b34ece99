"""CPU-only check of the tile loader's per-lane offsets (csrc/row_offset.hpp) at the largest row
stride the strided entry points accept: the exact value, with no signed overflow on the way."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER_DIR = os.path.join(ROOT, "paper_2510_04212_amd", "csrc")

MAIN = r"""
#include "row_offset.hpp"
#include <cstdio>
int main(int argc, char**) {
  const int strides[] = {32, 256, 8454664, (int)kRowStrideLimit - 8};
  for (int sn : strides)
    for (int row = argc - 1; row < kMaxTileRows; ++row)
      printf("%lld %u\n", (long long)row * 2 * sn + 48, row_offset(row, sn, 48));
  return 0;
}
"""


def test_offsets_are_exact_up_to_the_largest_stride(tmp_path):
    src, exe = tmp_path / "main.cpp", tmp_path / "main"
    src.write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all", "-I", HEADER_DIR,
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    lines = [tuple(map(int, l.split())) for l in r.stdout.splitlines()]
    assert len(lines) == 4 * 128 and all(a == b for a, b in lines)
