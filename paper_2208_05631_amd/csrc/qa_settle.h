// The settling pass of the quantizers that read a long gradient once: code words in which the pattern 10
// stands for a component inside the bracket around the threshold get the codes of those components.
// Internal to libqadagrad.
#pragma once
#include "qa_common.h"

namespace qa {

constexpr int kSettleTiles = 8;            // consecutive tiles per work-group, thread t holds word t of each
constexpr int kSettleList = 4096;          // open components that are looked up; more: the tiles are coded again

struct SettleLds {
  uint32_t words[kSettleTiles * kTileWords];
  uint16_t list[kSettleList];              // word of the eight tiles << 4 | field
  uint32_t wave_total[kWaves];
};

// w[u]: word t of tile tile0 + u (0 where there is none; such words are not open).  On return w[] holds
// the settled words, and s, c have grown by what the open components of this thread's share keep.
// The open components are listed first and then looked up one per thread: their cache lines are
// requested together instead of one field of every word after the other (54 M x 8 components of two
// tensors: 160 -> 139 us).  Contains barriers.  Returns false, with w[], s and c as they were, if more than
// an eighth of the components are open: magnitudes that grow along the vector put all of them into few
// work-groups, whose lists took longer than the rest of the call (2^24 x 4 rising magnitudes 243 -> 78 us).
// *changed: whether this thread's words did.
__device__ __forceinline__ bool settle_words(const float* __restrict__ g, int64_t tile0, float D,
                                             uint32_t (&w)[kSettleTiles], SettleLds& lds, double& s, uint32_t& c,
                                             bool* changed) {
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  uint32_t open[kSettleTiles], mine = 0;
#pragma unroll
  for (int u = 0; u < kSettleTiles; ++u) {
    open[u] = (w[u] >> 1) & ~w[u] & 0x55555555u;         // low bit of every field 10
    mine += (uint32_t)__popc(open[u]);
  }
  const uint32_t incl = wave_scan_u32(mine);
  if (lane == kWave - 1) lds.wave_total[wave] = incl;
#pragma unroll
  for (int u = 0; u < kSettleTiles; ++u) lds.words[u * kTileWords + t] = w[u];
  __syncthreads();
  uint32_t before = incl - mine, total = 0;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) {
    if (v < wave) before += lds.wave_total[v];
    total += lds.wave_total[v];
  }
  *changed = mine != 0;
  if (total > (uint32_t)kSettleList) return false;       // uniform
  if (total == 0) return true;
  if (mine) {
    uint32_t at = before;
#pragma unroll
    for (int u = 0; u < kSettleTiles; ++u)
      for (uint32_t left = open[u]; left; left &= left - 1u, ++at)
        lds.list[at] = (uint16_t)(((u * kTileWords + t) << 4) | ((__ffs((int)left) - 1) >> 1));
  }
  __syncthreads();
  for (uint32_t i = t; i < total; i += kThreads) {
    const uint32_t e = lds.list[i], word = e >> 4, field = e & 15u;
    const float x = g[(tile0 + (word >> 8)) * kTile + 16 * (int64_t)(word & 255u) + field];
    const float av = fabsf(x);
    const bool keep = av > D;
    s += keep ? (double)av : 0.0;
    c += keep ? 1u : 0u;
    // the field holds 10; exclusive or with 10 ^ code
    atomicXor(&lds.words[word], (2u ^ ternary_field(x, D)) << (2 * field));
  }
  __syncthreads();
  if (mine) {
#pragma unroll
    for (int u = 0; u < kSettleTiles; ++u) w[u] = lds.words[u * kTileWords + t];
  }
  return true;
}

}  // namespace qa
