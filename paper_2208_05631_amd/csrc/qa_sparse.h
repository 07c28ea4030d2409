// Device helpers shared by the kernels that read or write the sparse encoding (indicator bits +
// compact per-bucket code stream; Section 3.2, Encode paragraph).  Internal to libqadagrad.
#pragma once
#include "qa_common.h"

namespace qa {

// Deposit table: entry [nib][s] spreads the low 2-bit codes of s to the 2-bit fields of a byte
// whose positions are the set bits of the 4-bit mask nib (first code to the lowest set bit).
struct DepositLut { uint8_t v[16 * 256]; };
constexpr DepositLut make_deposit_lut() {
  DepositLut t{};
  for (int nib = 0; nib < 16; ++nib)
    for (int s = 0; s < 256; ++s) {
      uint32_t w = (uint32_t)s, out = 0;
      for (int b = 0; b < 4; ++b)
        if ((nib >> b) & 1) { out |= (w & 3u) << (2 * b); w >>= 2; }
      t.v[nib * 256 + s] = (uint8_t)out;
    }
  return t;
}
static __device__ const DepositLut kDepositLut = make_deposit_lut();

}  // namespace qa
