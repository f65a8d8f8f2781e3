// Where a block or K group of a conv-mode GEMM starts along K.  Plain C++.
#pragma once

namespace pulse {

// taps x C columns of one source range of the implicit operand
struct KSeg {
  int taps, C;
};

// segment, tap and first channel of a K-step
struct KStart {
  int seg, tap, cb;
};

// K-step q of up to three segments (unused ones: 0 taps), bk channels per
// step, chunk-major: the taps of one chunk run back to back.  K groups share
// the steps of a block out, and where K is shorter than the groups (a 1x1
// conv of few channels) the last ones start at or past its end: any position
// will do for them, since they load nothing, but they must not divide by the
// 0 taps of an unused segment.
constexpr KStart k_start(int q, int bk, KSeg s0, KSeg s1, KSeg s2) {
  int seg = 0;
  KSeg s = s0;
  while (seg < 2 && q >= s.taps * (s.C / bk)) {
    q -= s.taps * (s.C / bk);
    ++seg;
    s = seg == 1 ? s1 : s2;
  }
  if (s.taps == 0) return KStart{seg, 0, 0};
  const int chunk = q / s.taps;
  return KStart{seg, q - chunk * s.taps, chunk * bk};
}

}  // namespace pulse
