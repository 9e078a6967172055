"""The autotuner's choice of CG block sizes from probe times, on the host: a
probe that ran solves in one block is compared by all of its CG time."""
import os
import subprocess

import pytest

from paper_2606_20426_amd import build

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "tune.h"
int main(int argc, char** argv) {
  tc::CgProbe p[16];
  int n = 0;
  for (int i = 1; i + 4 < argc; i += 5, ++n)
    p[n] = {atoi(argv[i]), atof(argv[i + 1]), atof(argv[i + 2]), atof(argv[i + 3]), atoll(argv[i + 4])};
  const tc::CgChoice c = tc::choose_cg_blocks(p, n, {64, 64});
  printf("%d %d\n", c.vertex_block, c.spmv_block);
}
"""


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("tune")
    (d / "main.cpp").write_text(MAIN)
    exe = str(d / "tune")
    subprocess.run(["g++", "-std=c++17", "-I", build.CSRC, str(d / "main.cpp"), "-o", exe], check=True)
    return lambda *probes: tuple(
        int(v) for v in subprocess.check_output([exe, *[str(v) for p in probes for v in p]]).split())


# block, ms of products, of updates, of solves in one block, iterations
LAUNCHED = [(128, 6.0, 2.0, 0.0, 1000), (512, 5.0, 3.0, 0.0, 1000), (1024, 9.0, 4.0, 0.0, 1000)]


@pytest.mark.parametrize("own,want", [
    ((256, 4.0, 1.0, 0.0, 1000), (256, 256)),       # launched and best at both
    ((256, 4.0, 9.0, 0.0, 1000), (128, 256)),       # each kernel for itself
    ((256, 0.0, 0.0, 20.0, 1000), (128, 512)),      # small pads only, slower in one block
    ((256, 0.0, 0.0, 5.0, 1000), (256, 256)),       # and faster
    ((256, 2.0, 1.0, 8.0, 1000), (128, 512)),       # a part in one block, slower as a whole
    ((256, 2.0, 1.0, 3.0, 1000), (256, 256)),       # and faster
    ((256, 0.0, 0.0, 0.0, 0), (128, 512)),          # nothing measured
    ((256, 0.0, 1.0, 0.0, 1000), (256, 512)),       # one kernel not measured
    ((256, 4.0, 1.0, 0.0, 2000), (256, 256)),       # per iteration
])
def test_choice_by_measured_times(choose, own, want):
    for at in range(4):
        assert choose(*LAUNCHED[:at], own, *LAUNCHED[at:]) == want


def test_only_small_probes(choose):
    assert choose((256, 0.0, 0.0, 5.0, 1000)) == (256, 256)
    assert choose() == (64, 64)
