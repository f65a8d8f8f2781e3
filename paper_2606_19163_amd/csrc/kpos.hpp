// Where a block or K group of a conv-mode GEMM starts along K.  Plain C++.
#pragma once

namespace pulse {

// segment, tap and first channel of a K-step
struct KStart {
  int seg, tap, cb;
};

// K-step q of up to three segments of taps x C columns, bk channels per step,
// chunk-major: the taps of one chunk run back to back.  s: the first segment
// on entry, the step's on return; next(s, i) moves it on to segment i (unused
// ones: 0 taps).  K groups share the steps of a block out, and where K is
// shorter than the groups (a 1x1 conv of few channels) the last ones start at
// or past its end: any position will do for them, since they load nothing,
// but they must not divide by the 0 taps of an unused segment.
template <class S, class Next>
constexpr KStart k_start(int q, int bk, S& s, Next next) {
  int seg = 0;
  while (seg < 2 && q >= s.taps * (s.C / bk)) {
    q -= s.taps * (s.C / bk);
    next(s, ++seg);
  }
  const int taps = s.taps > 0 ? s.taps : 1;
  const int chunk = q / taps;
  return KStart{seg, q - chunk * taps, chunk * bk};
}

}  // namespace pulse
