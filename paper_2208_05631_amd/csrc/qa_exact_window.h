// Where the fine bins of the exact threshold's one pass over a long bucket lie (qa_exact_wide.hip).  constexpr and
// without headers of the GPU: the probe's last work-group and the tests on the CPU run the same lines.
#ifndef QA_EXACT_WINDOW_H
#define QA_EXACT_WINDOW_H

#include <stdint.h>

namespace qa {

// 32 bins per binade, 8192 to 512 around the bracket.  (Half of what a level has: the scan is bound by its
// instructions, and with 64 per binade and 4096 bins in all it took 13 us.)
constexpr int kFarShift = 18, kNearShift = 10, kWidestNear = 14;
constexpr int kNearBins = 2 << (kFarShift - kNearShift), kMostNear = kNearBins >> (kFarShift - kWidestNear);

// kNearBins bins of 2^shift patterns in the place of the bins of 2^18 from near0 on; shift 0: there are none.
struct NearWindow {
  uint32_t near0, shift;
};

// The finest bins whose window, centred on `mid`, holds the bracket [below, above) with four of them to spare at
// either end.  (Of a bracket that lies outside in part the proof may fail, and every level reads the gradient: 2^24 x 4
// 10 %-dense Laplace components 192 us, 150 with a window that holds it.)  Patterns of positive finite floats,
// below < mid < above.
constexpr NearWindow near_window(uint32_t below, uint32_t mid, uint32_t above) {
  for (int shift = kNearShift; shift <= kWidestNear; ++shift) {
    const uint32_t near = (uint32_t)kNearBins >> (kFarShift - shift), spare = 4u << shift;
    const uint32_t near0 = (mid - ((near - 1u) << (kFarShift - 1))) >> kFarShift;
    const uint32_t from = near0 << kFarShift, to = (near0 + near) << kFarShift;
    if (below > from + spare && above + spare < to) return NearWindow{near0, (uint32_t)shift};
  }
  return NearWindow{0u, 0u};
}

}  // namespace qa

#endif
