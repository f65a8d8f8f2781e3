"""The start position of a conv-mode GEMM's K range (csrc/kpos.hpp), built
for the CPU with UndefinedBehaviorSanitizer: every block and K group against
a walk over K, and groups past the end of K."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

MAIN = r"""
#include <cstdio>
#include <initializer_list>
#include "kpos.hpp"
using namespace pulse;

struct KSeg {
  int taps, C;
};

// segment, tap and channel of K-step kt, found by walking there
static KStart walk(int kt, int bk, const KSeg (&s)[3]) {
  for (int seg = 0; seg < 3; ++seg)
    for (int cb = 0; cb < s[seg].C; cb += bk)
      for (int tap = 0; tap < s[seg].taps; ++tap)
        if (kt-- == 0) return KStart{seg, tap, cb};
  return KStart{-1, 0, 0};
}

int main() {
  const KSeg cases[][3] = {{{9, 64}, {0, 0}, {0, 0}},  {{1, 64}, {0, 0}, {0, 0}},
                           {{1, 128}, {0, 0}, {0, 0}}, {{9, 128}, {1, 192}, {0, 0}},
                           {{9, 64}, {9, 64}, {1, 128}}, {{1, 192}, {1, 64}, {0, 0}}};
  int past = 0;
  for (const auto& s : cases)
    for (int bk : {32, 64}) {
      int all = 0;
      for (const KSeg& g : s) all += g.taps * (g.C / bk);
      for (int steps : {all, (all + 1) / 2, (all + 2) / 3})  // K splits
        for (int ktb = 0; ktb < all; ktb += steps)
          for (int kg = 1; kg <= 4; ++kg) {
            const int n = steps < all - ktb ? steps : all - ktb, len = (n + kg - 1) / kg;
            for (int g = 0; g < kg; ++g) {
              const int kt0 = ktb + g * len;
              KSeg cur = s[0];
              const KStart a = k_start(kt0, bk, cur, [&](KSeg& c, int i) { c = s[i]; });
              if (kt0 >= all) {
                ++past;
                continue;
              }
              const KStart b = walk(kt0, bk, s);
              if (a.seg != b.seg || a.tap != b.tap || a.cb != b.cb) {
                std::printf("step %d: %d %d %d, not %d %d %d\n", kt0, a.seg, a.tap, a.cb, b.seg,
                            b.tap, b.cb);
                return 1;
              }
            }
          }
    }
  std::printf("%d groups past the end\n", past);
  return past > 0 ? 0 : 2;
}
"""


def test_k_start_of_every_block_and_group(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "kpos.cpp", tmp_path / "kpos"
    src.write_text(MAIN)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-fsanitize=undefined",
                    "-fno-sanitize-recover=all", "-I",
                    os.path.join(ROOT, "paper_2606_19163_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
