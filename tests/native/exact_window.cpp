// qa_exact_window.h for tests/test_exact_window.py
#include "qa_exact_window.h"

extern "C" void near_window(uint32_t below, uint32_t mid, uint32_t above, uint32_t* near0, uint32_t* shift) {
  const qa::NearWindow w = qa::near_window(below, mid, above);
  *near0 = w.near0;
  *shift = w.shift;
}
extern "C" void near_window_shape(uint32_t* out) {
  out[0] = qa::kFarShift; out[1] = qa::kNearShift; out[2] = qa::kWidestNear; out[3] = qa::kNearBins;
}
