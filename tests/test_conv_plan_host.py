"""The small-grid conv plan (csrc/plan.hpp): tiles and K splits whose blocks
do not all fit on the GPU at once against the next best, measured on MI355X."""

import os
import subprocess

import pytest

from paper_2606_19163_amd import build as B

MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include "plan.hpp"
using namespace pulse;

int main(int argc, char** argv) {
  const long p = std::atol(argv[1]);
  const int n = std::atoi(argv[2]), k = std::atoi(argv[3]);
  const int hw = std::atoi(argv[4]), want = std::atoi(argv[5]);
  const ConvPlan c = conv_plan_small(p, n, k, hw, TILE2_C64x128S3, 16, -1, (ConvWant)want);
  const TileInfo t = tile2_info(c.tile);
  std::printf("%d %d %d\n", t.bm, t.bn, c.ks);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    if not os.path.exists(B.LIB):
        B.build()
    d = tmp_path_factory.mktemp("plan")
    src, obj, exe = d / "plan.hip", d / "plan.o", d / "plan"
    src.write_text(MAIN)
    subprocess.run([B.HIPCC, *B.CFLAGS, "-c", str(src), "-o", str(obj)], check=True,
                   capture_output=True)
    subprocess.run([B.HIPCC, str(obj), B.LIB, f"-Wl,-rpath,{os.path.dirname(B.LIB)}", "-o",
                    str(exe)], check=True, capture_output=True)

    def run(p, n, k, hw=1, want=0):  # want: a ConvWant
        r = subprocess.run([str(exe), *map(str, (p, n, k, hw, want))], check=True,
                           capture_output=True, text=True, timeout=60)
        return tuple(map(int, r.stdout.split()))

    return run


# rows, columns, K -> tile and K splits; us of that plan and of the one the
# model takes without counting the rounds past the resident blocks
@pytest.mark.parametrize("p,n,k,want", [
    (13056, 128, 128, (64, 128, 1)),   # 6.5, 32 x 64 in 816 blocks 7.9
    (2304, 768, 192, (64, 128, 1)),    # 6.9, 32 x 64 in 864 blocks 8.7
    (4480, 384, 128, (64, 128, 1)),    # 6.4, 32 x 64 in 840 blocks 7.9
    (1472, 1024, 9216, (64, 128, 2)),  # 48.1, five splits, 920 blocks, 50.1
    (12288, 128, 128, (32, 64, 1)),    # 6.2 in 768 blocks, all of them resident, 64 x 128 6.3
    (8192, 128, 128, (32, 64, 1)),     # 5.2 in 512 blocks, 64 x 128 6.2
])
def test_rounds_past_the_resident_blocks_count(plan, p, n, k, want):
    assert plan(p, n, k) == want


# a 3x3 conv of 32 x 32 images whose output's statistics are wanted too
def test_small_tiles_in_several_rounds(plan):
    # 15.1 us, 32 x 64 in four K groups and 768 blocks, one per CU, 22.7
    assert plan(24576, 64, 1152, 1024, 1) == (64, 128, 1)
