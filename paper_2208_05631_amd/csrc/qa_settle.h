// The quantizers that read a long gradient once, with a bracket around the threshold: codes and sums of what lies
// outside it, the components inside it ("open") and their codes once the threshold is known.
// Internal to libqadagrad.
#pragma once
#include "qa_common.h"
#include "qa_open_group.h"

namespace qa {

constexpr int kSettleTiles = 8;            // consecutive tiles whose kept sum becomes one partial sum
constexpr uint32_t kOpenSlots = 16;        // float4 groups with open components that a wave of the one pass can list
constexpr uint32_t kOpenMany = 15;         // what stands for more: the tile is coded again then
// A tile's count of what is certainly kept (4096 at most) and the lengths of its four lists share a word.
__device__ __forceinline__ uint32_t tile_counts(const uint32_t (&wave)[kWaves]) {
  uint32_t kept = 0, open = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    kept += wave[w] & 0xFFFFu;
    open |= (wave[w] >> 16) << (4 * w);
  }
  return kept | open << 16;
}
__device__ __forceinline__ bool too_many_open(uint32_t counts) {   // one of the four fields is 15
  const uint32_t o = counts >> 16;
  return ((o & (o >> 1) & (o >> 2) & (o >> 3)) & 0x1111u) != 0u;
}

// Did the sample's bracket hold the threshold?  (NaN compares false.)
__device__ __forceinline__ bool bracket_held(float2 band, float D) {
  return band.x >= 0.0f && D >= band.x && D <= band.y;
}

// The one pass over a tile: the sum of |v| in the order of the passes that form only that, the sum and (of the whole
// wave) the number of what is certainly kept, the lanes whose components are open, the code word without those.
__device__ __forceinline__ uint32_t code_outside(const float (&v)[4][4], float2 band, double& s1, double& s2,
                                                 uint32_t& wave_cnt, uint64_t (&open)[4][4]) {
  uint64_t keep[4][4];
  double kept[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double av = (double)fabsf(v[j][e]);
      s1 += av;
      keep[j][e] = __ballot(fabsf(v[j][e]) > band.y);
      open[j][e] = __ballot(fabsf(v[j][e]) > band.x) & ~keep[j][e];
      wave_cnt += (uint32_t)__popcll(keep[j][e]);
      add_in_lanes(kept[j], av, keep[j][e]);
    }
  s2 = (kept[0] + kept[1]) + (kept[2] + kept[3]);
  return code_word(v, keep);
}

// Lists the wave's float4 groups j * 256 + thread with open components; their number.  (Groups and not components: a
// third of the instructions.  The settling pass fetches the group, one cache line as for a component alone.)
__device__ __forceinline__ uint32_t list_open(const uint64_t (&open)[4][4], uint16_t* list) {
  uint32_t n = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint64_t some = (open[j][0] | open[j][1]) | (open[j][2] | open[j][3]);
    if (some) {                                          // uniform
      const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((uint32_t)some, n));
      if (((some >> (threadIdx.x % kWave)) & 1ull) && at < kOpenSlots) list[at] = (uint16_t)(j * kThreads + threadIdx.x);
      n += (uint32_t)__popcll(some);
    }
  }
  return n < kOpenMany ? n : kOpenMany;
}

// Looks the open components of groups list[first], list[first + stride], .. (n in all) up: what threshold D keeps of them
// is added to s and c, its codes join the tile's words, where the one pass has left 00.  (Magnitudes inside a bracket
// share their units of the last place: their binary64 sum is exact, in any order.)  live: components of the row from
// the tile's first on, those beyond belong to nobody and are not read.  AHEAD groups are requested together.
template <int AHEAD>
__device__ __forceinline__ void settle_listed(const uint16_t* __restrict__ list, uint32_t first, uint32_t stride,
                                              uint32_t n, const float* __restrict__ g, int64_t live, float2 band, float D,
                                              uint32_t* words, double& s, uint32_t& c) {
  const uint32_t here = live < kTile ? (uint32_t)live : (uint32_t)kTile;
  for (uint32_t i0 = first; i0 < n; i0 += AHEAD * stride) {
    uint32_t group[AHEAD];
    float4 q[AHEAD];
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) group[k] = i0 + k * stride < n ? list[i0 + k * stride] : 0u;
#pragma unroll
    for (int k = 0; k < AHEAD; ++k)
      q[k] = i0 + k * stride < n ? load_group<float4>(g, group[k], here) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int k = 0; k < AHEAD; ++k) {
      const float x[4] = {q[k].x, q[k].y, q[k].z, q[k].w};
      uint32_t byte = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float av = fabsf(x[e]);
        if (av > D && !(av > band.y)) {                  // D >= band.x >= 0
          s += (double)av;
          ++c;
          byte |= ternary_field(x[e], D) << (2 * e);
        }
      }
      if (byte) atomicOr(words + (group[k] >> 2), byte << (8 * (group[k] & 3u)));
    }
  }
}

// Without room for lists the one pass marks open components with the pattern 10, which no message holds.
constexpr int kMarkedList = kSettleTiles * kWaves * (kOpenMany - 1) * 4;   // marked components of eight tiles at most
struct SettleLds {
  uint32_t words[kSettleTiles * kTileWords];
  uint16_t list[kMarkedList];              // word of the eight tiles << 4 | field
  double sum[kSettleTiles];
  uint32_t count[kSettleTiles];
  uint32_t wave_total[kWaves];
};

// w[u]: word t of tile tile0 + u (0 where there is none; such words are not open).  On return w[] holds the settled
// words, lds.sum[u] and lds.count[u] what is kept of tile u's open components.  Contains barriers.  Returns the tiles
// (bit u) whose lists would have been too long: their words stay as they are.  *changed: whether this thread's words did.
__device__ __forceinline__ uint32_t settle_words(const float* __restrict__ g, int64_t tile0, float D,
                                                 uint32_t (&w)[kSettleTiles], SettleLds& lds, bool* changed) {
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  uint32_t open[kSettleTiles], groups_lo = 0, groups_hi = 0;
#pragma unroll
  for (int u = 0; u < kSettleTiles; ++u) {
    open[u] = (w[u] >> 1) & ~w[u] & 0x55555555u;         // low bit of every field 10
    uint32_t o = open[u] | open[u] >> 4;                 // float4 groups with open components: a byte each
    o = (o | o >> 2) & 0x01010101u;
    (u < 4 ? groups_lo : groups_hi) |= (uint32_t)__popc(o) << (8 * (u & 3));
    lds.words[u * kTileWords + t] = w[u];
  }
  // word t holds groups of wave (t / 16) % 4 of the one pass; a row of 16 lanes is a quarter of that wave's (64 groups
  // at most), the other quarters are the same rows of the other waves
  uint32_t* rows = reinterpret_cast<uint32_t*>(lds.list);   // [wave][row][2], before the list is written
  groups_lo += (uint32_t)dpp_i32<kDppQuadXor1>((int)groups_lo);      groups_hi += (uint32_t)dpp_i32<kDppQuadXor1>((int)groups_hi);
  groups_lo += (uint32_t)dpp_i32<kDppQuadXor2>((int)groups_lo);      groups_hi += (uint32_t)dpp_i32<kDppQuadXor2>((int)groups_hi);
  groups_lo += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)groups_lo); groups_hi += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)groups_hi);
  groups_lo += (uint32_t)dpp_i32<kDppRowMirror>((int)groups_lo);     groups_hi += (uint32_t)dpp_i32<kDppRowMirror>((int)groups_hi);
  if (lane % 16 == 0) {
    rows[(wave * 4 + lane / 16) * 2] = groups_lo;
    rows[(wave * 4 + lane / 16) * 2 + 1] = groups_hi;
  }
  if (t < kSettleTiles) { lds.sum[t] = 0.0; lds.count[t] = 0u; }
  __syncthreads();
  uint32_t n_groups = 0;                                 // of tile lane % 8, wave lane / 8 % 4 of the one pass
#pragma unroll
  for (int v = 0; v < kWaves; ++v)
    n_groups += (rows[(v * 4 + lane / 8 % 4) * 2 + (lane % 8) / 4] >> (8 * (lane % 4))) & 0xFFu;
  uint32_t many = (uint32_t)__ballot(n_groups >= kOpenMany);
  many |= many >> 16;
  many = (many | many >> 8) & 0xFFu;
  uint32_t mine = 0;
#pragma unroll
  for (int u = 0; u < kSettleTiles; ++u) {
    if (many >> u & 1u) open[u] = 0u;
    mine += (uint32_t)__popc(open[u]);
  }
  const uint32_t incl = wave_scan_u32(mine);
  if (lane == kWave - 1) lds.wave_total[wave] = incl;
  __syncthreads();                                       // (the rows have been read)
  uint32_t before = incl - mine, total = 0;
#pragma unroll
  for (int v = 0; v < kWaves; ++v) {
    if (v < wave) before += lds.wave_total[v];
    total += lds.wave_total[v];
  }
  *changed = mine != 0;
  if (total == 0) return many;                           // uniform
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
    if (av > D) {
      atomicAdd(&lds.sum[word >> 8], (double)av);        // exact, in any order
      atomicAdd(&lds.count[word >> 8], 1u);
    }
    // the field holds 10; exclusive or with 10 ^ code
    atomicXor(&lds.words[word], (2u ^ ternary_field(x, D)) << (2 * field));
  }
  __syncthreads();
  if (mine) {
#pragma unroll
    for (int u = 0; u < kSettleTiles; ++u) w[u] = lds.words[u * kTileWords + t];
  }
  return many;
}

}  // namespace qa
