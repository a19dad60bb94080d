"""CPU check of the encoder's addresses of single rows: it steps between the
bricks of a row's window with signed 24-bit products, so single rows are only
taken where the 24-bit product of a step equals the whole one, on every sensor
a context accepts (the rule is the library's own, compiled from its header).
"""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <cstdio>
#include "veckm_internal.h"
using namespace veckm;
// the signed 24-bit product of the vector ALU (operands cut to their low 24 bits)
static long mul24(long a, long b) {
  auto cut = [](long v) { v &= 0xffffff; return v >= 0x800000 ? v - 0x1000000 : v; };
  return cut(a) * cut(b);
}
int main() {
  const Brick bricks[] = {{32, 32, 8}, {32, 16, 16}, {32, 16, 8}, {32, 16, 4}, {16, 16, 8}, {16, 16, 4},
                          {16, 8, 4},  {8, 8, 4},    {8, 8, 2},   {8, 4, 2},   {4, 4, 1}};
  const int sides[][2] = {{346, 260},     {1280, 720},   {12288, 12288}, {8192, 8192}, {11584, 11588},
                          {1 << 25, 4},   {1 << 25, 5},  {1 << 26, 8},   {4, 1 << 26}, {1 << 30, 1},
                          {23170, 23170}, {11585, 11585}};
  int refused = 0;
  for (const Brick& b : bricks)
    for (const auto& s : sides) {
      const long nbx = (s[0] + b.bx - 1) / b.bx, nby = (s[1] + b.by - 1) / b.by;
      bool exact = true;
      for (long k = -64; k <= 64; ++k)
        exact = exact && mul24(k, nbx * nby) == k * nbx * nby && mul24(k, nbx) == k * nbx;
      if (single_rows_fit(s[0], s[1], b) != exact) {
        std::printf("sensor %dx%d brick %d,%d,%d: rule %d, products exact %d\n", s[0], s[1], b.bx, b.by, b.bt,
                    (int)single_rows_fit(s[0], s[1], b), (int)exact);
        return 1;
      }
      refused += !exact;
    }
  std::printf("refused %d\n", refused);
  return refused > 0 ? 0 : 1;
}
"""


def test_window_steps_fit_24_bits(tmp_path):
    src, exe = tmp_path / "steps.cpp", tmp_path / "steps"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2504_19417_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], stdout=subprocess.PIPE, text=True)
    assert r.returncode == 0, r.stdout
