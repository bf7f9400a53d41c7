"""Which bytes the projection's loads touch, enumerated on the CPU from the functions that the kernel
uses (csrc/qkv_tile.h): every lane of every load of every k-tile, for tiles of any row count.

A buffer load compares the lane's offset with the buffer's size and adds the scalar offset behind that
comparison, so a load touches [lane + scalar, lane + scalar + 16) whenever lane < size."""
from __future__ import annotations

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include <vector>
#include "qkv_tile.h"
using namespace d2o::qkv;

// argv: hidden, rows of the tile, 1: the step of a load in the scalar offset (a planted mistake).
// Rows beyond kMaxBufferHidden go by clamped 64-bit offsets; of their k-tiles the first and last three are taken.
int main(int argc, char** argv) {
  const int hidden = atoi(argv[1]), rows = atoi(argv[2]);
  const bool scalar_step = argc > 3 && atoi(argv[3]);
  const bool wide = hidden > kMaxBufferHidden;
  const int64_t row_bytes = int64_t(hidden) * 2, size = wide ? rows * row_bytes : buffer_bytes(rows, uint32_t(row_bytes));
  const int nkt = (hidden + kBK - 1) / kBK;
  long outside = 0, wrong = 0;
  for (int kt = 0; kt < nkt; ++kt) {
    if (wide && kt >= 3 && kt < nkt - 3) continue;
    std::vector<int64_t> lds(kBM * kLd / 8, -2);  // per 16 bytes of the stage: the offset loaded there (-1: zero)
    for (int w = 0; w < kThreads / 64; ++w)
      for (int i = 0; i < kLoads; ++i)
        for (int lane = 0; lane < 64; ++lane) {
          if (wide) {
            const int64_t off = wide_offset(w, lane, i, kt, rows, row_bytes);
            if (off < 0 || off + 16 > size) ++outside;
            lds[(lds_start(w, i) + lane * 8) / 8] = off;
            continue;
          }
          uint32_t at = lane_offset(w, lane, i & 1, row_bytes), scalar = load_step(i, kt, row_bytes);
          if (!scalar_step) {
            at += scalar;
            scalar = 0;
          }
          if (at >= (1u << 31)) ++outside;
          if (at < size && int64_t(at) + scalar + 16 > size) ++outside;
          lds[(lds_start(w, i) + lane * 8) / 8] = at < size ? int64_t(at) + scalar : -1;
        }
    // the stage holds what the operand reads expect: chunk k of row r at position k ^ ((r >> 1) & 7)
    for (int r = 0; r < kBM; ++r)
      for (int k = 0; k < kBK / 8; ++k) {
        const int64_t got = lds[(r * kLd) / 8 + (k ^ ((r >> 1) & 7))];
        const int col = kt * kBK + k * 8;
        if (got == -2) ++wrong;
        if (r < rows && col < hidden && got != int64_t(r) * row_bytes + col * 2) ++wrong;
      }
  }
  printf("%ld %ld\n", outside, wrong);
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("qkv")
    src, exe = d / "loads.cpp", d / "loads"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", os.path.join(ROOT, "paper_2406_13035_amd", "csrc"), "-o", str(exe), str(src)],
                   check=True)
    return lambda *args: tuple(int(x) for x in subprocess.run([str(exe), *map(str, args)], check=True, capture_output=True,
                                                              text=True).stdout.split())


@pytest.mark.parametrize("hidden", [32, 64, 96, 160, 1024, 4096, 4128, (1 << 22) - 64, (1 << 22) - 32, 1 << 22, (1 << 31) - 32])
@pytest.mark.parametrize("rows", [0, 1, 7, 8, 9, 44, 63, 64, 65, 128, 200, 255, 256])
def test_no_load_leaves_its_buffer_and_every_element_arrives(program, hidden, rows):
    if hidden == (1 << 22) - 64 and rows not in (1, 65, 255, 256):
        pytest.skip("65535 k-tiles: at four row counts")
    if hidden > (1 << 22) - 64 and rows == 0:
        pytest.skip("past the last output tile these rows load the last tile again")
    assert program(hidden, rows) == (0, 0)


def test_the_enumeration_sees_steps_behind_the_comparison(program):
    """The mistake this guards against, planted: a load's row and k-tile step as scalar offset."""
    for hidden, rows in ((4096, 1), (4096, 200), (96, 256)):  # ragged tiles, and a last half k-tile
        outside, _ = program(hidden, rows, 1)
        assert outside > 0
    assert program(4096, 256, 1)[0] == 0                       # (a full tile of whole k-tiles stays inside either way)
