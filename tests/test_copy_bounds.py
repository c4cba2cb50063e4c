"""CPU-only: the copies of the products that walk their tiles read nothing but their operands' rows, and all of a tile's.

The kernel's address arithmetic (csrc/faar_copies.h) is compiled for the host and walked copy by copy and lane by lane: no read ends
beyond the last row that the matrix has, whatever is left of it for the tile, and the rows and chunks lie in LDS where the main loop
takes its fragments from."""
import os
import shutil
import subprocess

import pytest

from paper_2603_22370_amd import build as fbuild

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "faar_copies.h"
constexpr int BM = 256, WN = 64, TN = 4, COPIES = 64;
typedef faar::RoundsCopy<BM, WN, TN> R;
#define CHECK(x) do { if (!(x)) { std::printf("%s: rows %u pitch %u copy %d lane %d\n", #x, rows, pitch, u, lane); std::exit(1); } } while (0)
int main() {
  const uint32_t inputs[] = {192, 256, 1088, 2048, 4096};
  for (uint32_t kd : inputs)
    for (uint32_t pitch : {2u * kd, 2u * kd + 16u, 1u << 23})           // bytes a row
      for (uint32_t rows = 1; rows <= BM; ++rows)
        for (int u = 0; u < COPIES; ++u)
          for (int lane = 0; lane < 64; ++lane) {
            const uint32_t off = R::offset(u, lane, rows, pitch), last = off + (kd / 64 - 1) * 128 + 16;
            CHECK((uint64_t)last <= (uint64_t)(rows - 1) * pitch + 2 * kd);   // the last slice too
            const bool of_a = u < BM / 8;
            const int p = of_a ? 8 * u + lane / 8 : 8 * u - BM + lane / 8, slot = lane % 8;       // LDS row of the operand, 16-byte slot
            const uint32_t row = of_a ? p : WN * (p / WN) + TN * (p % 16) + p % WN / 16, chunk = slot ^ (p / 2 % 8);
            CHECK(R::row(u, lane) == row && R::chunk(u, lane) == chunk);
            if (row < rows) CHECK(off == row * pitch + chunk * 16);
          }
  std::puts("ok");
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_copies_stay_within_the_operands(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", fbuild.CSRC, str(src), "-o", str(exe)], check=True, timeout=120)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout == "ok\n", r.stdout
