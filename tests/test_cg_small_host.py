"""The rule that sends a pad's CG to one block admits no more rows than the
kernel's arrays, sized by the same constant, hold."""
import subprocess

from paper_2606_20426_amd import build

MAIN = r"""
#define __host__
#define __device__
#include "tc_device.h"
template <typename R> constexpr int beyond() {
  int bad = 0;
  for (int W = 1; W <= 64; ++W)
    for (int V = 1; V <= 2048; ++V)
      bad += tc::cg_small_rows(V, W, sizeof(R) == 8) != (W <= 16 && V <= tc::CG_SMALL_ROWS<R>);
  return bad;
}
int main() { return beyond<double>() + beyond<float>(); }
"""


def test_rule_and_capacity_agree(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "rows")
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(tmp_path / "main.cpp"), "-o", exe], check=True)
    assert subprocess.run([exe]).returncode == 0
