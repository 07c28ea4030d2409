// Threshold quantizer + 2-bit encoding (Sections 3.4-3.5 of arXiv 2208.05631) for gfx950.
//
// Tile = 4096 elements of one worker's gradient per 256-thread work-group.  Thread t holds
// four float4 groups f = j*256 + t (j = 0..3), i.e. elements 4f..4f+3 of the tile, so that
// every global load instruction of a wave reads 1 KiB of consecutive memory.
//
//   bucket <= 4096 : one kernel; sums, threshold, scale and codes of a tile's buckets are
//                    formed in registers/LDS; the gradient is read once (4 B/elem + 0.25 B out).
//   up to 65536, and whole vectors (0) that short: the same with a larger work-group per bucket, beyond 45056
//                    components if there are enough of them.
//   otherwise      : tile partial sums -> finalize threshold -> codes and
//                    tile partial (count, sum) -> finalize scale; the gradient is read twice, or,
//                    for long buckets, once: a sample brackets the threshold beforehand.
#include <mutex>
#include <type_traits>

#include "qa_common.h"
#include "qa_settle.h"

namespace qa {

struct QuantArgs {
  const float* g;
  int64_t g_stride;
  int64_t d;
  int64_t W;               // ceil(d/16)
  uint32_t* codes;
  int64_t code_stride;
  float* scales;
  float* thresholds;       // user array, may be null
  int64_t scale_stride;
  int log2b;               // log2(bucket); unused when bucket == 0
  float thr_coef;
  int thresh_given;
  int through;             // code words go through the cache at once: words_go_through()
  // two-pass path
  double* part_sum;        // [M][ntiles]
  uint32_t* part_cnt;      // [M][ntiles]
  float* thr_ws;           // [M][nb]
  int64_t ntiles;
  int64_t tiles_per_bucket;  // ntiles when bucket == 0
  int64_t nb;
  int64_t bucket_len;        // elements per bucket (d when bucket == 0)
  // one-read form of the two-pass path
  double* kept_sum;          // [M][ntiles]; before that the samples' sums
  float2* band;              // [M][nb]
  int64_t samples;           // sampled tiles per bucket (at most)
  int sample_every;          // one tile of so many
  int64_t settle_groups;     // partial sums per bucket that the settling pass leaves
  uint16_t* open;            // [M][ntiles][kWaves][kOpenSlots], null where there is no room for it
};

// Load the thread's 4 float4 groups of tile `tile`; elements at or beyond d read as +0.
__device__ __forceinline__ void load_tile(const float* __restrict__ g, int64_t d, int64_t tile,
                                          float v[4][4]) {
  const int64_t base = tile * kTile;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t i = base + (int64_t)(j * kThreads + (int)threadIdx.x) * 4;
    if (i + 3 < d) {
      const float4 q = *reinterpret_cast<const float4*>(g + i);
      v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = (i + e < d) ? g[i + e] : 0.0f;
    }
  }
}

// The same with streaming (non-temporal) loads for tiles that lie wholly below d: for passes after
// which the element is not needed again soon.
__device__ __forceinline__ void load_tile_stream(const float* __restrict__ g, int64_t d, int64_t tile,
                                                 float v[4][4]) {
  if ((tile + 1) * kTile <= d) {
    typedef float floatx4 __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const floatx4 q = __builtin_nontemporal_load(
          reinterpret_cast<const floatx4*>(g + tile * kTile + (j * kThreads + (int)threadIdx.x) * 4));
      v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    }
  } else {
    load_tile(g, d, tile, v);
  }
}

// The kernels that code a tile per work-group (quantize_tile, quantize_buckets_of_tile, quantize_codes_partial_kernel,
// quantize_bracketed_kernel) store 64 bytes of words side by side.  Through the cache if these are whole: every worker's
// row of words begins on a multiple of 64 bytes; of other rows from 7 * 2^24 components in all (448 MB) on.  There each store
// leaves two partial pieces, which cost more than late evictions as long as the last-level cache takes part.  Other
// gradients in each call, 7 workers, us, stores left in the cache / through it, rows on 64 bytes: quantizer, 4096: 128 MB
// 23.6 / 23.8, 256 45.8 / 44.6, 512 91.2 / 87.2; with the step: 4096, 96 MB 33.2 / 33.9, 256 79.5 / 77.9, 512 152 / 147;
// one scale, 96 MB 55.8 / 56.3, 256 130 / 128, 512 (read once) 182 / 178.  Other rows: quantizer, 4096: 96 MB 18.1 / 19.5,
// 192 34.2 / 35.6, 384 68.6 / 68.3, 512 91.6 / 89.9, 1024 184 / 178; 256: 128 MB 24.0 / 24.9, 256 47.6 / 47.0, 384
// 71.2 / 69.3, 1024 187 / 181; 64, 5 workers, 502 MB 92.5 / 89.9; with the step: 4096, 96 MB 33.4 / 35.1, 256 81.0 / 82.4,
// 416 137 / 139, 512 154 / 155; 256: 256 MB 82.1 / 83.7, 448 150 / 152; one scale, 128 MB 72.9 / 74.6, 320 160 / 161, 512
// 185 / 185.  Kernels whose work-groups hold more tiles or that issue more per word are not slower with such stores at any
// size (buckets of 8192 on, the stochastic rule, the exact one).
constexpr int64_t kThroughFrom = int64_t(7) << 24;
static bool words_go_through(const qa_layout* L, const uint32_t* codes) {
  const int64_t between = L->M > 1 ? 4 * L->code_stride : 0;
  return ((reinterpret_cast<uintptr_t>(codes) | (uintptr_t)between) & 63u) == 0 || L->d > kThroughFrom / L->M;
}

// The word of the tile's thread t (word j*64 + t/4 for j = t & 3).
__device__ __forceinline__ void store_code_word(uint32_t* __restrict__ codes_m, int64_t tile, int64_t W, uint32_t word,
                                                int t, bool through = true) {
  const int64_t widx = tile * kTileWords + (t & 3) * 64 + (t >> 2);
  if (widx >= W) return;
  if (through) store_through(codes_m + widx, word);      // uniform
  else codes_m[widx] = word;
}

// What threshold D keeps of the thread's elements, added to s, and of the wave's, added to wave_cnt; the code word.
__device__ __forceinline__ uint32_t code_tile(const float (&v)[4][4], float D, double& s, uint32_t& wave_cnt) {
  uint64_t keep[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    double sj = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      keep[j][e] = __ballot(fabsf(v[j][e]) > D);
      wave_cnt += (uint32_t)__popcll(keep[j][e]);
      add_in_lanes(sj, (double)fabsf(v[j][e]), keep[j][e]);
    }
    s += sj;
  }
  const float Delta[4] = {D, D, D, D};
  return D < 0.0f ? code_word_compared(v, Delta) : code_word(v, keep);
}

// ---- 64 <= bucket < 4096 : single pass, several buckets per tile --------------------------------
//
// Slice j of the tile (elements j*1024 .. j*1024+1023) is held four elements per thread, so a
// bucket of b <= 1024 elements is SEG = b/4 consecutive threads of one slice, and a bucket of 2048
// is two whole slices.  The four slices are summed together: the first two exchanges (lanes l^1,
// l^2) leave lane l with the part of slice l & 3, the others run on one value instead of four.
// Every exchange adds the same two operands in both lanes, so all lanes of a bucket hold the same
// sum.  Threshold, scale and their divisions are likewise formed once, slice l & 3's in lane l.
__device__ __forceinline__ double lanes_xor4_f64(double v) {
  return dpp_f64<0x1B>(dpp_f64<kDppRowHalfMirror>(v));   // l^7, then l^3
}
__device__ __forceinline__ uint32_t lanes_xor4_u32(uint32_t v) {
  return (uint32_t)dpp_i32<0x1B>(dpp_i32<kDppRowHalfMirror>((int)v));
}
constexpr int kDppRowRor8 = 0x128;                       // l^8 within the row of 16
// v of the even row plus v of the odd row (ROWS = 16), of the lower half plus of the upper (32)
template <int ROWS>
__device__ __forceinline__ void swap_rows(uint32_t v, uint32_t* a, uint32_t* b) {
  const auto r = ROWS == 16 ? __builtin_amdgcn_permlane16_swap(v, v, false, false)
                            : __builtin_amdgcn_permlane32_swap(v, v, false, false);
  *a = r[0]; *b = r[1];
}
template <int ROWS> __device__ __forceinline__ double add_rows_f64(double v) {
  uint32_t al, bl, ah, bh;
  swap_rows<ROWS>((uint32_t)__double2loint(v), &al, &bl);
  swap_rows<ROWS>((uint32_t)__double2hiint(v), &ah, &bh);
  return __hiloint2double((int)ah, (int)al) + __hiloint2double((int)bh, (int)bl);
}
template <int ROWS> __device__ __forceinline__ uint32_t add_rows_u32(uint32_t v) {
  uint32_t a, b;
  swap_rows<ROWS>(v, &a, &b);
  return a + b;
}

// s[j]: this thread's part of slice j -> for slice l & 3, the sum over LANES lanes of the wave
template <int LANES>
__device__ __forceinline__ double slices_sum_f64(const double s[4]) {
  const bool odd = threadIdx.x & 1, high = threadIdx.x & 2;
  const double a = (odd ? s[1] : s[0]) + dpp_f64<kDppQuadXor1>(odd ? s[0] : s[1]);
  const double b = (odd ? s[3] : s[2]) + dpp_f64<kDppQuadXor1>(odd ? s[2] : s[3]);
  double v = (high ? b : a) + dpp_f64<kDppQuadXor2>(high ? a : b);
  v += lanes_xor4_f64(v);
  v += dpp_f64<kDppRowRor8>(v);
  if (LANES >= 32) v = add_rows_f64<16>(v);
  if (LANES >= 64) v = add_rows_f64<32>(v);
  return v;
}
// the same for counts that a quad's lane l holds for slice l & 3 already
template <int LANES>
__device__ __forceinline__ uint32_t quads_sum_u32(uint32_t v) {
  v += lanes_xor4_u32(v);
  v += (uint32_t)dpp_i32<kDppRowRor8>((int)v);
  if (LANES >= 32) v = add_rows_u32<16>(v);
  if (LANES >= 64) v = add_rows_u32<32>(v);
  return v;
}

// The sums over the buckets that hold this thread's part of slice l & 3.  lds_*: 16 entries each that
// nobody else uses; the work-group's threads all take part (barriers for buckets above 256).
template <int LOG2B, bool WITH_COUNT>
__device__ __forceinline__ void bucket_sums(const double s[4], uint32_t quad_count, double* lds_s, uint32_t* lds_c,
                                            double* sum, uint32_t* count) {
  constexpr int SEG = LOG2B >= 10 ? 256 : (1 << LOG2B) / 4;     // threads per bucket within a slice
  constexpr int LANES = SEG < 64 ? SEG : 64;
  *sum = slices_sum_f64<LANES>(s);
  if (WITH_COUNT) *count = quads_sum_u32<LANES>(quad_count);
  if constexpr (SEG > 64) {
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, j = lane & 3;
    __syncthreads();                                     // earlier readers of lds are done
    if (lane < 4) {
      lds_s[j * kWaves + wave] = *sum;
      if (WITH_COUNT) lds_c[j * kWaves + wave] = *count;
    }
    __syncthreads();
    const auto waves_of = [&](int q) {                   // slice q over the waves of the bucket
      const int w0 = SEG == 128 ? wave & ~1 : 0;
      const double pair = lds_s[q * kWaves + w0] + lds_s[q * kWaves + w0 + 1];
      return SEG == 128 ? pair : pair + (lds_s[q * kWaves + 2] + lds_s[q * kWaves + 3]);
    };
    const auto counts_of = [&](int q) {
      const int w0 = SEG == 128 ? wave & ~1 : 0;
      const uint32_t pair = lds_c[q * kWaves + w0] + lds_c[q * kWaves + w0 + 1];
      return SEG == 128 ? pair : pair + lds_c[q * kWaves + 2] + lds_c[q * kWaves + 3];
    };
    if (LOG2B == 11) {                                   // a bucket is two slices
      *sum = waves_of(j & ~1) + waves_of(j | 1);
      if (WITH_COUNT) *count = counts_of(j & ~1) + counts_of(j | 1);
    } else {
      *sum = waves_of(j);
      if (WITH_COUNT) *count = counts_of(j);
    }
  }
}

// Bound by the read of the gradient; where the last-level cache holds that, by vector instructions (about 240 per wave
// and tile: magnitudes stay converted from the first sum to the second, which adds them under a lane mask, and fields
// are shifted in; 398 with selects).  3 000 001 x 8 Gaussian components, buckets of 256 17.3 -> 16.0 us, 1024
// 17.6 -> 16.3.  With the words stored through the cache 2^26 x 4, 512 and 1024 178 -> 171, 256 177 -> 171.
template <int LOG2B, bool GIVEN>                         // a.thresh_given
__device__ __forceinline__ void quantize_buckets_of_tile(const QuantArgs& a, int64_t tile, int m) {
  __shared__ double lds_s[4 * kWaves];
  __shared__ uint32_t lds_c[4 * kWaves];
  constexpr int b = 1 << LOG2B;
  const float* g = a.g + (int64_t)m * a.g_stride;
  const int t = threadIdx.x;
  const bool whole = (tile + 1) * kTile <= a.d;          // the vector does not end inside the tile

  float v[4][4];
  load_tile_stream(g, a.d, tile, v);
  // this lane's bucket among the tile's: the one with its elements of slice l & 3
  const int kb = (((t & 3) * kThreads + t) * 4) >> LOG2B;
  const int64_t k = tile * (kTile >> LOG2B) + kb;
  float mine_delta;                                      // of that bucket
  if constexpr (!GIVEN) {
    double S1[4], sum;
    uint32_t unused;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      S1[j] = (double)fabsf(v[j][0]);
#pragma unroll
      for (int e = 1; e < 4; ++e) S1[j] += (double)fabsf(v[j][e]);
    }
    bucket_sums<LOG2B, false>(S1, 0u, lds_s, lds_c, &sum, &unused);
    // Every bucket of the tile is complete unless the vector ends inside the tile; dividing by
    // the power of two b is then an exact scaling, the same value as the division.
    if (whole) {
      mine_delta = (float)(((double)a.thr_coef * sum) * (1.0 / (double)b));
    } else {
      const int64_t lo = k << LOG2B;
      const int64_t n = (a.d - lo) < (int64_t)b ? (a.d - lo) : (int64_t)b;   // true length
      mine_delta = n > 0 ? threshold_from_sum(sum, a.thr_coef, n) : 0.0f;
    }
  } else {
    mine_delta = k < a.nb ? a.thresholds[(int64_t)m * a.scale_stride + k] : 0.0f;
  }
  float Delta[4];                                        // lane j of every quad has slice j's
  Delta[0] = __int_as_float(dpp_i32<0x00>(__float_as_int(mine_delta)));
  Delta[1] = __int_as_float(dpp_i32<0x55>(__float_as_int(mine_delta)));
  Delta[2] = __int_as_float(dpp_i32<0xAA>(__float_as_int(mine_delta)));
  Delta[3] = __int_as_float(dpp_i32<0xFF>(__float_as_int(mine_delta)));

  // kept sums and 2-bit fields; a negative (given) threshold takes the two plain comparisons
  double S2[4] = {0.0, 0.0, 0.0, 0.0};
  uint64_t keep[4][4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      keep[j][e] = __ballot(fabsf(v[j][e]) > Delta[j]);
      add_in_lanes(S2[j], (double)fabsf(v[j][e]), keep[j][e]);
    }
  const uint32_t mine = GIVEN && __any(mine_delta < 0.0f) ? code_word_compared(v, Delta) : code_word(v, keep);
  // after the ranking kernel, part of the gradient comes from the last-level cache, and stores through the caches cost
  // more than they save (exact threshold, 5e7 x 2, buckets of 64 / 256: 273.8 / 331.3 us, without 272.0 / 329.2)
  store_code_word(a.codes + (int64_t)m * a.code_stride, tile, a.W, mine, threadIdx.x, !GIVEN && a.through);
  double sum;
  uint32_t count;
  // a lane's word holds the quad's components of slice l & 3; what is kept has a field other than 0
  bucket_sums<LOG2B, true>(S2, (uint32_t)__popc(mine & 0x55555555u), lds_s, lds_c, &sum, &count);
  // the quad with the bucket's first element writes (of a bucket of two slices, the first one's lane)
  constexpr int SEG = LOG2B >= 10 ? 256 : b / 4;
  const bool writes = (t & (SEG - 1)) < 4 && (LOG2B < 11 || (t & 1) == 0);
  if (writes && k < a.nb) {
    a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(sum, count);
    if (!GIVEN && a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + k] = mine_delta;
  }
}

template <int LOG2B, bool GIVEN>
__global__ __launch_bounds__(kThreads) void quantize_bucket_kernel(QuantArgs a) {
  quantize_buckets_of_tile<LOG2B, GIVEN>(a, blockIdx.x, blockIdx.y);
}

// ---- bucket == 4096 == the tile : single pass, two work-group reductions ---------------------

// Bound by the read of the gradient; where the last-level cache holds that, by vector instructions (about 220 per
// wave, 323 with selects): 2^20 x 16 components 12.2 -> 11.1 us, 3 000 001 x 8 19.1 -> 17.0.
// With the words stored through the cache 2^28 x 4 721 -> 691 (6.6 TB/s).
template <bool GIVEN>                                    // a.thresh_given
__device__ __forceinline__ void quantize_tile(const QuantArgs& a, int64_t tile, int m) {
  __shared__ double lds_s1[kWaves];
  __shared__ double lds_s2[kWaves];
  __shared__ uint32_t lds_c[kWaves];
  const int t = threadIdx.x;
  const int64_t lo = tile * kTile;
  const float* g = a.g + (int64_t)m * a.g_stride;
  const bool whole = lo + kTile <= a.d;
  float v[4][4];
  if (whole) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // the gradient is read exactly once: nontemporal
      typedef float floatx4 __attribute__((ext_vector_type(4)));
      const floatx4 q = __builtin_nontemporal_load(
          reinterpret_cast<const floatx4*>(g + lo + (j * kThreads + t) * 4));
      v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    }
  } else {
    load_tile(g, a.d, tile, v);
  }

  float Delta;
  if constexpr (!GIVEN) {
    double sj[4];                                        // four independent chains
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      sj[j] = (double)fabsf(v[j][0]);
#pragma unroll
      for (int e = 1; e < 4; ++e) sj[j] += (double)fabsf(v[j][e]);
    }
    const double S1 = block_sum_f64((sj[0] + sj[1]) + (sj[2] + sj[3]), lds_s1);
    // dividing by 4096 is an exact scaling
    Delta = whole ? (float)(((double)a.thr_coef * S1) * (1.0 / (double)kTile))
                  : threshold_from_sum(S1, a.thr_coef, a.d - lo);
  } else {
    Delta = a.thresholds[(int64_t)m * a.scale_stride + tile];
  }
  double s2j[4] = {0.0, 0.0, 0.0, 0.0};
  uint64_t keep[4][4];
  uint32_t wave_cnt = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      keep[j][e] = __ballot(fabsf(v[j][e]) > Delta);
      wave_cnt += (uint32_t)__popcll(keep[j][e]);
      add_in_lanes(s2j[j], (double)fabsf(v[j][e]), keep[j][e]);
    }
  // v > Delta or v < -Delta  <=>  |v| > Delta, unless a caller hands in a threshold below 0 (uniform)
  const float Delta4[4] = {Delta, Delta, Delta, Delta};
  const uint32_t mine = GIVEN && Delta < 0.0f ? code_word_compared(v, Delta4) : code_word(v, keep);
  store_code_word(a.codes + (int64_t)m * a.code_stride, tile, a.W, mine, threadIdx.x, a.through);

  const double s2 = wave_sum_f64((s2j[0] + s2j[1]) + (s2j[2] + s2j[3]));
  if ((t % kWave) == 0) { lds_s2[t / kWave] = s2; lds_c[t / kWave] = wave_cnt; }
  __syncthreads();
  if (t == 0) {
    const double S2 = (lds_s2[0] + lds_s2[1]) + (lds_s2[2] + lds_s2[3]);
    const uint32_t C = lds_c[0] + lds_c[1] + lds_c[2] + lds_c[3];
    a.scales[(int64_t)m * a.scale_stride + tile] = scale_from_sum(S2, C);
    if (!GIVEN && a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + tile] = Delta;
  }
}

template <bool GIVEN>
__global__ __launch_bounds__(kThreads) void quantize_tile_kernel(QuantArgs a) {
  quantize_tile<GIVEN>(a, blockIdx.x, blockIdx.y);
}

// ---- exact optimal threshold by ranking (Section 3.4: the magnitudes are sorted and each one
//      is tried as the threshold) for one 4096-tile ----------------------------------------------
//
// |v| of the tile is sorted in descending order (bitonic network on the bit patterns, which
// order like the non-negative floats), prefix sums are formed in binary64, and the k that
// maximises (sum of the k largest)^2 / k is taken among the k that do not split equal
// magnitudes.  The threshold written is the largest magnitude NOT kept (0 if none), to be
// compared with strictly like the approximate one.
//
// The network runs on 16 keys per thread held in registers.  Position i of the 4096 has 12 bits;
// a thread owns the 16 positions that differ in four of them ("free" bits) and the other eight
// come from its thread index.  Three ownerships cover every stage: free bits 0-3, 4-7 or 8-11.
// A stage that exchanges across bit b is done by the ownership whose free bits hold b, as a
// register min/max; keys move between ownerships through LDS (two buffers, used alternately, so
// one barrier per move is enough: a buffer is rewritten only after the barrier that follows
// every thread's last read of it).  Rows of 16 are padded to 17 words against bank conflicts.
constexpr int kSortPitch = kTile + kTile / 16;

template <int OWN> __device__ __forceinline__ int sort_position(int t, int r) {
  if (OWN == 0) return t * 16 + r;
  if (OWN == 1) return (t & 15) | (r << 4) | ((t >> 4) << 8);
  return t | (r << 8);
}

// The stages of phase P (blocks of 2^P positions, alternately descending and ascending) that
// exchange across the lowest NST free bits of ownership OWN, highest first.  A block that must
// come out ascending is sorted descending on complemented keys.  FLIP: complement here, around
// the stages (phases 1-4, where the block bit is a compile-time bit of r or t & 1); otherwise the
// caller keeps the keys of ascending blocks complemented for the whole phase (an exchange never
// leaves its block, so a key's state stays right for the position it moves to).
template <int OWN, int P, int NST, bool FLIP>
__device__ __forceinline__ void sort_stages(uint32_t (&e)[16], int t) {
  if (FLIP) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      e[r] ^= (uint32_t)(-((sort_position<OWN>(t, r) >> P) & 1));
  }
#pragma unroll
  for (int lb = NST - 1; lb >= 0; --lb)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (!(r & (1 << lb))) {
        const uint32_t x = e[r], y = e[r | (1 << lb)];
        e[r] = x > y ? x : y;
        e[r | (1 << lb)] = x > y ? y : x;
      }
  if (FLIP) {
#pragma unroll
    for (int r = 0; r < 16; ++r)
      e[r] ^= (uint32_t)(-((sort_position<OWN>(t, r) >> P) & 1));
  }
}

template <int FROM, int TO>
__device__ __forceinline__ void sort_move(uint32_t (&e)[16], int t, uint32_t* buf) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = sort_position<FROM>(t, r);
    buf[i + (i >> 4)] = e[r];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int i = sort_position<TO>(t, r);
    e[r] = buf[i + (i >> 4)];
  }
}

// Phase P of the network for P >= 5, entered and left in ownership 0 (positions 16t + r: the
// block bit P is bit P-4 of t, the same for the thread's 16 keys).  On entry the keys carry the
// complement state of phase P-1 (PREV_FLIPPED) or none; they leave in the state of phase P, which
// for the last phase is "none" (FINAL: every block of 2^P comes out descending; for P = 12 that
// is the one block there is).  n counts the moves made so far and picks the buffer.
template <int P, bool PREV_FLIPPED, bool FINAL>
__device__ __forceinline__ void sort_phase(uint32_t (&e)[16], int t, uint32_t (*buf)[kSortPitch],
                                           int& n) {
  {
    const uint32_t now = FINAL ? 0u : (t >> (P - 4)) & 1u, before = PREV_FLIPPED ? (t >> (P - 5)) & 1u : 0u;
    const uint32_t m = (uint32_t)(-(int)(now ^ before));
#pragma unroll
    for (int r = 0; r < 16; ++r) e[r] ^= m;
  }
  if constexpr (P > 8) {
    sort_move<0, 2>(e, t, buf[n++ & 1]);
    sort_stages<2, P, P - 8, false>(e, t);
    sort_move<2, 1>(e, t, buf[n++ & 1]);
    sort_stages<1, P, 4, false>(e, t);
  } else {
    sort_move<0, 1>(e, t, buf[n++ & 1]);
    sort_stages<1, P, P - 4, false>(e, t);
  }
  sort_move<1, 0>(e, t, buf[n++ & 1]);
  sort_stages<0, P, 4, false>(e, t);
}

// LOG2B: log2 of the bucket (6..12): the network stops after phase LOG2B, which leaves every
// bucket of the tile sorted on its own; the prefix sums and the search then run per bucket, over
// the 2^(LOG2B-4) consecutive threads that hold it.
template <int LOG2B>
__device__ __forceinline__ void rank_tile(const QuantArgs& a, int64_t tile, int m) {
  static_assert(LOG2B >= 6 && LOG2B <= 12, "bucket of 64 .. 4096 components");
  constexpr int kSeg = 1 << (LOG2B - 4);                 // threads per bucket
  constexpr int kSegLanes = kSeg < kWave ? kSeg : kWave; // ... of them inside one wave
  constexpr int kSegWaves = kSeg / kSegLanes;            // waves per bucket: 1, 2 or 4
  __shared__ uint32_t buf[2][kSortPitch];
  __shared__ uint32_t lds_first[kThreads];
  __shared__ double lds_tot[kWaves];
  __shared__ double lds_obj[kWaves];
  __shared__ int lds_k[kWaves];
  __shared__ float lds_next[kWaves];
  // opaque: in a loop over tiles the places of the network's moves would otherwise be computed once and
  // kept, 100 registers of them
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  const int lane = t % kWave, wave = t / kWave;
  uint32_t e[16];                 // which 16 of the tile a thread starts with does not matter
  {
    float v[4][4];
    load_tile(a.g + (int64_t)m * a.g_stride, a.d, tile, v);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < 4; ++c) e[j * 4 + c] = __float_as_uint(fabsf(v[j][c]));
  }
  // load_tile hands thread t the float4 groups j*256 + t, i.e. components of up to four buckets
  // when the bucket is smaller than the tile: bring every key to ownership 0 (positions
  // 16t .. 16t+15) first, so that a thread's keys and every later exchange stay inside a bucket
  int n = 0;
  if constexpr (LOG2B < 12) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = ((r >> 2) * kThreads + t) * 4 + (r & 3);
      buf[0][i + (i >> 4)] = e[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int i = 16 * t + r;
      e[r] = buf[0][i + (i >> 4)];
    }
    n = 1;
  }
  sort_stages<0, 1, 1, true>(e, t);
  sort_stages<0, 2, 2, true>(e, t);
  sort_stages<0, 3, 3, true>(e, t);
  sort_stages<0, 4, 4, true>(e, t);
  sort_phase<5, false, false>(e, t, buf, n);
  sort_phase<6, true, LOG2B == 6>(e, t, buf, n);
  if constexpr (LOG2B >= 7) sort_phase<7, true, LOG2B == 7>(e, t, buf, n);
  if constexpr (LOG2B >= 8) sort_phase<8, true, LOG2B == 8>(e, t, buf, n);
  if constexpr (LOG2B >= 9) sort_phase<9, true, LOG2B == 9>(e, t, buf, n);
  if constexpr (LOG2B >= 10) sort_phase<10, true, LOG2B == 10>(e, t, buf, n);
  if constexpr (LOG2B >= 11) sort_phase<11, true, LOG2B == 11>(e, t, buf, n);
  if constexpr (LOG2B >= 12) sort_phase<12, true, true>(e, t, buf, n);
  // the thread now holds positions 16t .. 16t+15 of the tile, each bucket in descending order
  const int ts = t & (kSeg - 1);                         // this thread's place among its bucket's threads
  lds_first[t] = e[0];
  __syncthreads();
  float av[17];
#pragma unroll
  for (int j = 0; j < 16; ++j) av[j] = __uint_as_float(e[j]);
  av[16] = ts < kSeg - 1 ? __uint_as_float(lds_first[t + 1]) : 0.0f;
  double run[16];
  run[0] = (double)av[0];
#pragma unroll
  for (int j = 1; j < 16; ++j) run[j] = run[j - 1] + (double)av[j];
  double incl = run[15];
#pragma unroll
  for (int off = 1; off < kSegLanes; off <<= 1) {
    const double o = __shfl_up(incl, off, kWave);
    if ((lane & (kSegLanes - 1)) >= off) incl += o;
  }
  // by the neighbour and not incl - run[15], which is not a number where this thread holds an infinity
  const double left = __shfl_up(incl, 1, kWave);
  double before = (lane & (kSegLanes - 1)) ? left : 0.0;
  if constexpr (kSegWaves > 1) {
    if (lane == kWave - 1) lds_tot[wave] = incl;
    __syncthreads();
    for (int w = wave & ~(kSegWaves - 1); w < wave; ++w) before += lds_tot[w];
  }
  // best candidate of this thread (smallest k among equal objectives); k = 0: none
  double best = -1.0;
  int best_k = 0;
  float best_next = 0.0f;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int k = 16 * ts + j + 1;
    if (av[j] > 0.0f && av[j] > av[j + 1]) {
      const double r = before + run[j];
      const double obj = r * r / (double)k;
      if (obj > best) { best = obj; best_k = k; best_next = av[j + 1]; }
    }
  }
#pragma unroll
  for (int off = 1; off < kSegLanes; off <<= 1) {
    const double o = __shfl_xor(best, off, kWave);
    const int ok = __shfl_xor(best_k, off, kWave);
    const float on = __shfl_xor(best_next, off, kWave);
    if (o > best || (o == best && ok < best_k)) { best = o; best_k = ok; best_next = on; }
  }
  if constexpr (kSegWaves > 1) {
    if (lane == 0) { lds_obj[wave] = best; lds_k[wave] = best_k; lds_next[wave] = best_next; }
    __syncthreads();
    if (ts == 0)
      for (int w = wave + 1; w < wave + kSegWaves; ++w) {
        const double o = lds_obj[w];
        const int ok = lds_k[w];
        if (o > best || (o == best && ok < best_k)) { best = o; best_k = ok; best_next = lds_next[w]; }
      }
  }
  if (ts == 0) {
    const int64_t k = tile * (kTile >> LOG2B) + (t >> (LOG2B - 4));   // bucket index
    if (k < a.nb) a.thresholds[(int64_t)m * a.scale_stride + k] = best_k > 0 ? best_next : 0.0f;
  }
}

template <int LOG2B>
__global__ __launch_bounds__(kThreads) void exact_threshold_kernel(QuantArgs a) {
  rank_tile<LOG2B>(a, blockIdx.x, blockIdx.y);
}

// ---- the same optimum without ranking everything: buckets of 512 .. 4096 ------------------------
//
// With s_k the mean of the k largest magnitudes, the objective k s_k^2 does not grow when the next
// magnitude a is added iff a <= s_k (sqrt(k^2 + k) - k) < s_k / 2, and does not grow when the last
// one is taken away iff that one is >= s_k / 2.  So the optimum keeps nothing below half the mean,
// and only a few positions around the best one have to be looked at:
//
//   1. magnitudes in [mean/2, max] are counted in a histogram whose bins are equal ranges of the bit
//      pattern; a bin holds its count and the sum of its members' offsets from the bin's lower end in
//      units of the last place, so the bin's sum is exact;
//   2. every lane sums its run of bins; per run the objective at its lower edge, and a bound for every
//      cut inside it: the j largest of c members with sum o + c L in [L, H] sum to at most
//      min(j H, o + j L), largest objective where the two meet, at j = o / (H - L); towards the
//      run's ends the bound falls to the edges' values because (A + B j)^2 / (K + j) is convex in j;
//   3. the same bin by bin (a lane per bin) within the runs that reach the best edge;
//   4. the members of the bins that still reach it, and of the next one below -- some 20 magnitudes of
//      a smooth distribution -- are collected, ranked by counting and evaluated in binary64 exactly
//      like the ranking network does.  More than 64 of them: if every one of these bins holds a single
//      value (ties), the cuts between the bins are all there are, and they are compared in binary64.
//
// One wave per bucket, 64 to 8 components per lane: no work-group barrier.  A bucket where more than 64
// different magnitudes survive (objectives flat over a long stretch, all magnitudes within a bin), with
// non-finite members, with subnormal ones above mean/2 or with more than 64 binades between mean/2 and
// max gets the mark -1 for a threshold and is left to the ranking network (exact_rank_marked_kernel,
// launched behind this one).  Such buckets pay for both: 2^24 x 4 components with |v| ~ u^(-1/2), u uniform,
// buckets of 512 275 us by ranking all, 430 now (4096: 343, 240); ties cost less than by ranking (three
// values, one of them 0: 512 254 -> 214, 4096 321 -> 176), but for one single value in buckets of 512 (238 -> 286).
//
// Bound by vector instructions (some 1900 per wave and bucket of 4096; the network took 78 stages for the same
// and left the codes to a second pass over the gradient).  2^26 x 4 Gaussian components, thresholds and
// codes, ranking + quantizing -> this: buckets of 4096 1366 -> 235 us, 2048 1300 -> 273,
// 1024 1189 -> 347, 512 1094 -> 587.  (2^28 x 4, 4096: 992 -> 940 with one comparison and one bit field per component for
// the histogram, where it was a mask, a difference, a comparison and a shift, and with fields shifted in; 2^26 x 8 485 -> 473
// without a jump round the addition of each component: 100003 x 4, 10 %-dense Student-t, 13.8 -> 12.7, but where one
// component in 1000 is not 0, 5e7 x 2, 92 -> 97.)  Steps 2 to 4 cost the same for every bucket size, so halving
// the bucket nearly doubles the time: at 256 the network (889 us) stays ahead.
constexpr float kRankMark = -1.0f;
constexpr int kExactList = 64;            // survivors that one wave ranks by counting
constexpr float kBelowBest = 1.0f - 2e-6f;   // objectives in binary32 are good to a few 2^-24

__device__ __forceinline__ float wave_sum_f32(float v) {
  v += __int_as_float(dpp_i32<kDppQuadXor1>(__float_as_int(v)));
  v += __int_as_float(dpp_i32<kDppQuadXor2>(__float_as_int(v)));
  v += __int_as_float(dpp_i32<kDppRowHalfMirror>(__float_as_int(v)));
  v += __int_as_float(dpp_i32<kDppRowMirror>(__float_as_int(v)));
  const int i = __float_as_int(v);
  return (__int_as_float(__builtin_amdgcn_readlane(i, 0)) + __int_as_float(__builtin_amdgcn_readlane(i, 16))) +
         (__int_as_float(__builtin_amdgcn_readlane(i, 32)) + __int_as_float(__builtin_amdgcn_readlane(i, 48)));
}
// maximum of non-negative floats, by their bit patterns
__device__ __forceinline__ float wave_max_positive(float v) {
  return __int_as_float(wave_reduce_i32(__float_as_int(v), [](int p, int q) { return p > q ? p : q; }));
}
// LDS of one wave only: order between its own accesses, no barrier
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// Bits of |x|, formed anew at every use: kept from one pass over the registers to the next, the 64
// masked copies would not fit beside the components (the empty statement makes x opaque).
__device__ __forceinline__ uint32_t magnitude_bits(float& x) {
  asm volatile("" : "+v"(x));
  return __float_as_uint(x) & 0x7fffffffu;
}
// A run of c magnitudes with sum `sum` = c * low + excess in [low, high) below k0 others with sum s0:
// the objective with all of them kept, or the bound for keeping some if that is larger (0 without any).
__device__ __forceinline__ float run_score(float s0, float k0, float sum, float c, float excess, float low,
                                           float high, float* edge) {
  const float s1 = s0 + sum, j = excess * __builtin_amdgcn_rcpf(high - low);
  const float s_in = fmaf(j, high, s0);
  *edge = c > 0.0f ? s1 * s1 * __builtin_amdgcn_rcpf(k0 + c) : 0.0f;
  const float inside = c > 1.0f ? s_in * s_in * __builtin_amdgcn_rcpf(k0 + j) : 0.0f;
  return inside > *edge ? inside : *edge;
}

template <int LOG2B>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4)))
void exact_histogram_kernel(QuantArgs a) {
  static_assert(LOG2B >= 9 && LOG2B <= 12, "64 lanes x 8 .. 64 components");
  constexpr int b = 1 << LOG2B;
  constexpr int kGroups = b / (4 * kWave);               // float4 groups per lane
  constexpr int kLogBins = LOG2B - 2, kBins = 1 << kLogBins;
  constexpr int kLogPer = kLogBins - 6, kPer = 1 << kLogPer;       // bins per lane
  // a bin lies within a binade, and its members' offsets sum to less than 2^32
  constexpr int kMaxShift = 32 - LOG2B;
  __shared__ uint64_t hist_of[kWaves][kBins];
  __shared__ uint32_t list_of[kWaves][kExactList];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t k = (int64_t)blockIdx.x * kWaves + wave;           // bucket
  const int m = blockIdx.y;
  if (k >= a.nb) return;                                 // the whole wave
  uint64_t* hist = hist_of[wave];
  uint32_t* list = list_of[wave];
  const float* g = a.g + (int64_t)m * a.g_stride;
  const int64_t lo = k << LOG2B;

  float v[kGroups][4];                                   // group j * 64 + lane of the bucket
  if (lo + b <= a.d) {
#pragma unroll
    for (int j = 0; j < kGroups; ++j) {
      typedef float floatx4 __attribute__((ext_vector_type(4)));
      const floatx4 q = __builtin_nontemporal_load(
          reinterpret_cast<const floatx4*>(g + lo + (j * kWave + lane) * 4));
      v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < kGroups; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int64_t i = lo + (j * kWave + lane) * 4 + e;
        v[j][e] = i < a.d ? g[i] : 0.0f;
      }
  }
#pragma unroll
  for (int r = 0; r < kPer; ++r) hist[r * kWave + lane] = 0;

  // the largest magnitude by whole numbers: among negative values the largest pattern, among the others the largest
  // signed one, three at a time (a NaN shows in the total)
  float s32[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  uint32_t neg = 0;
  int pos = 0;
#pragma unroll
  for (int j = 0; j < kGroups; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s32[e] += fabsf(v[j][e]);
      const uint32_t bits = __float_as_uint(v[j][e]);
      neg = bits > neg ? bits : neg;
      pos = (int)bits > pos ? (int)bits : pos;
    }
  neg = neg & 0x80000000u ? neg & 0x7fffffffu : 0u;
  const uint32_t top = (uint32_t)wave_reduce_i32((uint32_t)pos > neg ? pos : (int)neg, [](int p, int q) { return p > q ? p : q; });
  const float total = wave_sum_f32((s32[0] + s32[1]) + (s32[2] + s32[3]));       // NaN if any member is

  float* thr_out = a.thresholds + (int64_t)m * a.scale_stride + k;
  float delta = 0.0f, scale = 0.0f;
  if (top != 0 || !(total == total)) {
    // half the mean, less more than the binary32 sum's error
    const uint32_t low = __float_as_uint(total * (0.499f / (float)b));
    int shift = 32 - __clz((int)((top - low) | 1u)) - kLogBins;
    shift = shift < 0 ? 0 : shift;
    uint32_t base = low & ~((1u << shift) - 1u);
    if (((top - base) >> shift) >= (uint32_t)kBins) { ++shift; base = low & ~((1u << shift) - 1u); }
    // (a total that overflowed makes low larger than top, a NaN larger than anything)
    bool leave = top >= 0x7f800000u || low >= top || low < 0x00800000u || (top >> 23) - (base >> 23) > 64u ||
                 shift > kMaxShift;
    bool ties = false, look_below = false;
    uint32_t count = 0, k_above = 0;
    double s_above = 0.0;
    float env_lo = 0.0f;
    // sums are formed on magnitudes scaled by a power of two that puts max into [1, 2)
    const uint32_t rescale = ((top >> 23) - 127u) << 23;
    // the scale in the magnitudes' own units: the power of two comes back exactly
    const double back = __hiloint2double((int)((top >> 23) - 127u + 1023u) << 20, 0);
    if (!leave) {
      // no member lies above the last bin, so one comparison tells which are counted; `base` is a multiple of a bin
      const uint32_t mask = (1u << shift) - 1u, limit = (uint32_t)kBins << shift;
      const uint32_t bin_base = base >> shift;
      const float first_counted = __uint_as_float(base);
      wave_lds_fence();
#pragma unroll
      for (int j = 0; j < kGroups; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (__builtin_expect(fabsf(v[j][e]) >= first_counted, 1)) {   // no branch round it
            const uint32_t bits = __float_as_uint(v[j][e]);
            const uint32_t bin = __builtin_amdgcn_ubfe(bits, (uint32_t)shift, 31u - (uint32_t)shift) - bin_base;
            atomicAdd(reinterpret_cast<unsigned long long*>(hist + bin),
                      (1ull << 32) | (unsigned long long)(bits & mask));
          }
      wave_lds_fence();
      // sum of a bin's members in binary64: count * lower end + offsets in units of the last place
      const auto scaled_end = [&](uint32_t bin) { return base + (bin << shift) - rescale; };
      const auto bin_sum = [&](uint64_t h, uint32_t bits) {
        const double ulp = __hiloint2double((int)(((bits >> 23) + (1023 - 150)) << 20), 0);
        return fma((double)(uint32_t)h, ulp, (double)(uint32_t)(h >> 32) * (double)__uint_as_float(bits));
      };
      // lane 0 holds the run of the kPer topmost bins, lane 63 the lowest; a lane starts reading at a
      // place of its own in its run so that the lanes' reads fall into different LDS banks
      const uint32_t bin0 = (uint32_t)((kWave - 1 - lane) << kLogPer);
      double lane_sum = 0.0;
      uint32_t lane_cnt = 0;
#pragma unroll 4
      for (int r = 0; r < kPer; ++r) {
        const uint32_t bin = bin0 + (uint32_t)((r + lane) & (kPer - 1));
        const uint64_t h = hist[bin];
        lane_sum += bin_sum(h, scaled_end(bin));
        lane_cnt += (uint32_t)(h >> 32);
      }
      const double run_before = wave_scan_f64(lane_sum) - lane_sum;
      const uint32_t run_cnt_before = wave_scan_u32(lane_cnt) - lane_cnt;
      float edge;
      const float run_low = __uint_as_float(scaled_end(bin0));
      const float excess = (float)fma(-(double)lane_cnt, (double)run_low, lane_sum);
      const float score = run_score((float)run_before, (float)run_cnt_before, (float)lane_sum, (float)lane_cnt,
                                    excess, run_low, __uint_as_float(scaled_end(bin0 + kPer)), &edge);
      const float bar = wave_max_positive(edge) * kBelowBest;
      const uint64_t runs = __ballot(lane_cnt != 0u && score >= bar), filled_runs = __ballot(lane_cnt != 0u);
      const int first = __ffsll((unsigned long long)runs) - 1;
      int last = 63 - __clzll((long long)runs);
      const uint64_t after = last < kWave - 1 ? filled_runs >> (last + 1) : 0ull;
      if (after) last += __ffsll((unsigned long long)after);        // the next magnitude below lies there
      // the bins of runs first .. last from the top, a row of 64 at a time
      const uint32_t bin_top = (uint32_t)(((kWave - first) << kLogPer) - 1);
      const int n_bins = (last - first + 1) << kLogPer;
      const double row_sum0 = readlane_f64(run_before, first);
      const uint32_t row_cnt0 = (uint32_t)__builtin_amdgcn_readlane((int)run_cnt_before, first);
      float best = 0.0f;
      double row_sum = row_sum0;
      uint32_t row_cnt = row_cnt0;
      uint32_t c = 0;
      double before = 0.0, row_total = 0.0;              // of this lane's bin: what lies above it, its sum
      uint32_t cnt_before = 0;
      const auto next_row = [&](int i0) {                // this lane's bin i0 + lane from the top
        const bool live = i0 + lane < n_bins;
        const uint32_t bin = live ? bin_top - (uint32_t)(i0 + lane) : 0u;
        const uint64_t h = live ? hist[bin] : 0ull;
        const uint32_t bits = scaled_end(bin);
        const double sum = bin_sum(h, bits);
        c = (uint32_t)(h >> 32);
        const double incl = wave_scan_f64(sum);
        const uint32_t cnt_incl = wave_scan_u32(c);
        before = row_sum + (incl - sum);
        row_total = sum;
        cnt_before = row_cnt + (cnt_incl - c);
        row_sum += readlane_f64(incl, kWave - 1);
        row_cnt += (uint32_t)__builtin_amdgcn_readlane((int)cnt_incl, kWave - 1);
        const float ulp = __uint_as_float((bits & 0x7f800000u) - (23u << 23));
        return run_score((float)before, (float)cnt_before, (float)sum, (float)c, (float)(uint32_t)h * ulp,
                         __uint_as_float(bits), __uint_as_float(bits + mask + 1u), &edge);
      };
#pragma unroll 1
      for (int i0 = 0; i0 < n_bins; i0 += kWave) {
        next_row(i0);
        best = edge > best ? edge : best;
      }
      const float bin_bar = wave_max_positive(best) * kBelowBest;
      // envelope: from the topmost surviving bin down to the next filled bin below the lowest one
      uint32_t bin_t = 0, bin_b = 0;
      bool found = false, open = false;
      row_sum = row_sum0;
      row_cnt = row_cnt0;
#pragma unroll 1
      for (int i0 = 0; i0 < n_bins; i0 += kWave) {
        const float bin_score = next_row(i0);
        const uint64_t with = __ballot(c != 0u && bin_score >= bin_bar), any = __ballot(c != 0u);
        const uint32_t row_top = bin_top - (uint32_t)i0;
        if (with) {
          const int lt = __ffsll((unsigned long long)with) - 1, lb = 63 - __clzll((long long)with);
          if (!found) {
            bin_t = row_top - (uint32_t)lt;
            s_above = readlane_f64(before, lt);
            k_above = (uint32_t)__builtin_amdgcn_readlane((int)cnt_before, lt);
            found = true;
          }
          const uint64_t lower = lb < kWave - 1 ? any >> (lb + 1) : 0ull;
          open = lower == 0ull;
          bin_b = row_top - (uint32_t)(open ? lb : lb + __ffsll((unsigned long long)lower));
        } else if (open && any) {
          open = false;
          bin_b = row_top - (uint32_t)(__ffsll((unsigned long long)any) - 1);
        }
      }
      const uint32_t lo_bits = base + (bin_b << shift);
      env_lo = __uint_as_float(lo_bits);
      const float env_hi = __uint_as_float(base + ((bin_t + 1u) << shift));
#pragma unroll
      for (int j = 0; j < kGroups; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint64_t who = __ballot(fabsf(v[j][e]) >= env_lo) & __ballot(fabsf(v[j][e]) < env_hi);
          if (who) {
            const uint32_t at = count + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                            __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u));
            if (((who >> lane) & 1ull) && at < (uint32_t)kExactList) list[at] = __float_as_uint(fabsf(v[j][e]));
            count += (uint32_t)__popcll(who);
          }
        }
      leave = count > (uint32_t)kExactList;
      if (leave) {                                         // does every bin of the envelope hold a single value?
        bool several = false;
#pragma unroll
        for (int j = 0; j < kGroups; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const uint32_t rel = magnitude_bits(v[j][e]) - base, bin = rel >> shift;
            if (rel < limit && bin >= bin_b && bin <= bin_t) {
              const uint64_t h = hist[bin];
              several |= (rel & mask) * (uint32_t)(h >> 32) != (uint32_t)h;        // offset != the mean offset
            }
          }
        ties = !__any(several);
      }
      if (ties) {                                          // the cuts between the bins are all there are
        leave = false;
        double best_obj = -1.0, best_sum = 0.0;
        uint32_t best_cnt = 0, best_at = 0;
        row_sum = row_sum0;
        row_cnt = row_cnt0;
#pragma unroll 1
        for (int i0 = 0; i0 < n_bins; i0 += kWave) {
          next_row(i0);
          const double kept_sum = before + row_total, kept = (double)(cnt_before + c);
          const double obj = c ? kept_sum * kept_sum / kept : -1.0;
          if (obj > best_obj) { best_obj = obj; best_sum = kept_sum; best_cnt = cnt_before + c; best_at = (uint32_t)(i0 + lane); }
        }
        double top_obj = best_obj;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
          const double o = shfl_xor_f64(top_obj, off);
          top_obj = o > top_obj ? o : top_obj;
        }
        // smallest k: the topmost of the bins that reach it
        const int at = wave_reduce_i32(best_obj == top_obj ? (int)best_at : 0x7fffffff, [](int p, int q) { return p < q ? p : q; });
        const int w = __ffsll((unsigned long long)__ballot(best_obj == top_obj && (int)best_at == at)) - 1;
        scale = scale_from_sum(readlane_f64(best_sum, w) * back, (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)best_cnt, w));
        // the next filled bin's value
        look_below = true;
#pragma unroll 1
        for (int i0 = at + 1; i0 < n_bins && look_below; i0 += kWave) {
          const uint64_t h = i0 + lane < n_bins ? hist[bin_top - (uint32_t)(i0 + lane)] : 0ull;
          const uint64_t any = __ballot(h != 0ull);
          if (any) {
            const int l = __ffsll((unsigned long long)any) - 1;
            const uint32_t cnt = (uint32_t)__builtin_amdgcn_readlane((int)(h >> 32), l);
            const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)h, l);
            delta = __uint_as_float(base + ((bin_top - (uint32_t)(i0 + l)) << shift) + sum / cnt);
            look_below = false;
          }
        }
      }
    }
    if (leave) {                                           // the ranking network takes this bucket
      if (lane == 0) *thr_out = kRankMark;
      return;
    }
    if (!ties) {
      wave_lds_fence();
      uint32_t key = lane < (int)count ? list[lane] : 0u;
      uint32_t rank = 0;
      for (int j = 0; j < (int)count; ++j) {
        const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)key, j);
        rank += (o > key || (o == key && j < lane)) ? 1u : 0u;
      }
      wave_lds_fence();
      if (lane < (int)count) list[rank] = key;
      wave_lds_fence();
      key = lane < (int)count ? list[lane] : 0u;
      const uint32_t next = lane + 1 < (int)count ? list[lane + 1] : 0u;
      const double value = lane < (int)count ? (double)__uint_as_float(key - rescale) : 0.0;
      const double sum = s_above + wave_scan_f64(value);
      const double kept = (double)(k_above + (uint32_t)lane + 1u);
      const double obj = lane < (int)count && key > next ? sum * sum / kept : -1.0;
      double top_obj = obj;
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const double o = shfl_xor_f64(top_obj, off);
        top_obj = o > top_obj ? o : top_obj;
      }
      const int w = __ffsll((unsigned long long)__ballot(obj == top_obj)) - 1;       // smallest k
      scale = scale_from_sum(readlane_f64(sum, w) * back, (uint64_t)(k_above + (uint32_t)w + 1u));
      look_below = w + 1 >= (int)count;                    // everything collected is kept
      if (!look_below) delta = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)key, w + 1));
    }
    if (look_below) {
      float below = 0.0f;
#pragma unroll
      for (int j = 0; j < kGroups; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = fabsf(v[j][e]);
          below = x < env_lo && x > below ? x : below;
        }
      delta = wave_max_positive(below);
    }
  }
  if (lane == 0) {
    *thr_out = delta;
    a.scales[(int64_t)m * a.scale_stride + k] = scale;
  }
  // group j * 64 + lane gives byte lane & 3 of code word j * 16 + lane / 4; four groups at a time,
  // lane l of a quad stores group l & 3's word
  uint32_t* codes = a.codes + (int64_t)m * a.code_stride;
  const int64_t w0 = lo / 16;
#pragma unroll
  for (int j4 = 0; j4 < kGroups; j4 += 4) {
    constexpr int kQuads = kGroups < 4 ? kGroups : 4;
    float x[4][4] = {};
    uint64_t kept[4][4] = {};
#pragma unroll
    for (int j = 0; j < kQuads; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        x[j][e] = v[j4 + j][e];
        kept[j][e] = __ballot(fabsf(x[j][e]) > delta);
      }
    const uint32_t mine = code_word(x, kept);
    const int64_t widx = w0 + (j4 + (lane & 3)) * 16 + (lane >> 2);
    if ((lane & 3) < kQuads && widx < a.W) store_through(codes + widx, mine);
  }
}

// The buckets that exact_histogram_kernel marked: ranked by the network, then quantized with the
// thresholds it found.  A work-group looks at kRankSpan tiles; a tile without a mark costs it one load.
constexpr int kRankSpan = 8;
template <int LOG2B>
__global__ __launch_bounds__(kThreads) void exact_rank_marked_kernel(QuantArgs a) {
  constexpr int kPerTile = kTile >> LOG2B;
  const int m = blockIdx.y;
  const int64_t tile0 = (int64_t)blockIdx.x * kRankSpan;
  const float* thr = a.thresholds + (int64_t)m * a.scale_stride;
  const int64_t mine = tile0 * kPerTile + threadIdx.x;
  const bool marked = threadIdx.x < kRankSpan * kPerTile && mine < a.nb && thr[mine] == kRankMark;
  __shared__ uint64_t lds_marks;
  if (threadIdx.x < kWave) {
    const uint64_t w = __ballot(marked);
    if (threadIdx.x == 0) lds_marks = w;
  }
  __syncthreads();
  uint64_t marks = lds_marks;
  while (marks) {
    const int64_t tile = tile0 + (__ffsll((unsigned long long)marks) - 1) / kPerTile;
    marks &= ~(((1ull << kPerTile) - 1ull) << ((tile - tile0) * kPerTile));
    rank_tile<LOG2B>(a, tile, m);
    __syncthreads();                                     // its thresholds are read next
    if constexpr (LOG2B == 12) quantize_tile<true>(a, tile, m);
    else quantize_buckets_of_tile<LOG2B, true>(a, tile, m);
    __syncthreads();                                     // LDS is free for the next tile
  }
}

// ---- bucket > 4096 or whole vector : two passes -----------------------------------------------

// pass 1: part_sum[m][tile] = sum |v| over the tile
__global__ __launch_bounds__(kThreads) void quantize_abs_partial_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  float v[4][4];
  // streaming: the second pass over the gradient comes after all of it has gone by
  load_tile_stream(a.g + (int64_t)m * a.g_stride, a.d, tile, v);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) s += (double)fabsf(v[j][e]);
  s = block_sum_f64(s, lds_d);
  if (threadIdx.x == 0) a.part_sum[(int64_t)m * a.ntiles + tile] = s;
}

// finalize 1: one work-group per (bucket, worker): threshold from the tile partials
__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void quantize_threshold_finalize_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t t0 = k * a.tiles_per_bucket;
  const int64_t t1 = (t0 + a.tiles_per_bucket) < a.ntiles ? (t0 + a.tiles_per_bucket) : a.ntiles;
  double s = strided_partial_sum(a.part_sum + (int64_t)m * a.ntiles, t0, t1);
  s = segment_sum(s, kThreads, lds_d);
  if (threadIdx.x == 0) {
    const int64_t lo = k * a.bucket_len;
    const int64_t n = (a.d - lo) < a.bucket_len ? (a.d - lo) : a.bucket_len;
    const float Delta = threshold_from_sum(s, a.thr_coef, n);
    a.thr_ws[(int64_t)m * a.nb + k] = Delta;
    if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + k] = Delta;
  }
}

// pass 2: codes of the tile and its partial (count, sum) of kept magnitudes
__global__ __launch_bounds__(kThreads) void quantize_codes_partial_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ uint32_t lds_u[kWaves];
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t k = tile / a.tiles_per_bucket;
  const float D = a.thresh_given ? a.thresholds[(int64_t)m * a.scale_stride + k]
                                 : a.thr_ws[(int64_t)m * a.nb + k];
  float v[4][4];
  load_tile_stream(a.g + (int64_t)m * a.g_stride, a.d, tile, v);
  double s = 0.0;
  uint32_t c = 0;
  store_code_word(a.codes + (int64_t)m * a.code_stride, tile, a.W, code_tile(v, D, s, c), threadIdx.x, a.through);
  s = wave_sum_f64(s);
  if ((threadIdx.x % kWave) == 0) { lds_d[threadIdx.x / kWave] = s; lds_u[threadIdx.x / kWave] = c; }
  __syncthreads();
  if (threadIdx.x == 0) {
    a.part_sum[(int64_t)m * a.ntiles + tile] = (lds_d[0] + lds_d[1]) + (lds_d[2] + lds_d[3]);
    a.part_cnt[(int64_t)m * a.ntiles + tile] = lds_u[0] + lds_u[1] + lds_u[2] + lds_u[3];
  }
}

// finalize 2: scale of each (bucket, worker)
__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void quantize_scale_finalize_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ double lds_c[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t t0 = k * a.tiles_per_bucket;
  const int64_t t1 = (t0 + a.tiles_per_bucket) < a.ntiles ? (t0 + a.tiles_per_bucket) : a.ntiles;
  // counts are integers < 2^53: exact in binary64
  double s, c;
  strided_partial_sums(a.part_sum + (int64_t)m * a.ntiles, a.part_cnt + (int64_t)m * a.ntiles, t0, t1, &s, &c);
  s = segment_sum(s, kThreads, lds_d);
  c = segment_sum(c, kThreads, lds_c);
  if (threadIdx.x == 0)
    a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(s, (uint64_t)c);
}

// ---- buckets of 2 .. 16 tiles held in registers ---------------------------------------------------
//
// A work-group holds its bucket between the threshold and the codes, so the gradient is read once and one launch does
// what the two passes and their finalize kernels take four for.  256 threads per tile up to four tiles, beyond
// that 1024 threads with two or four tiles each.  The sums are added as the two passes add them, so thresholds,
// codes and scales are the same numbers.  Bound by HBM up to 8 tiles; of 16 tiles the registers of a compute unit hold
// one bucket only, and nothing is read while it is coded.  Two passes -> held, us, at 2^26 x 4 components: buckets of
// 8192 495 -> 178, 16384 415 -> 186, 32768 372 -> 169, 65536 351 -> 229; 3 000 001 x 8: 48 -> 18, 40 -> 19, 37 -> 19,
// 35 -> 27; one scale for 5000 .. 40 000 components, 1 or 16 workers: 9 .. 10 -> 3 .. 9.5 (captured).
// A work-group takes its time for a long bucket, and two passes have one per tile.  Captured calls with other gradients in
// each, two passes -> held, us: 8 tiles, 1 work-group 8.9 -> 6.7, 24 10.2 -> 8.4; 11 tiles 1 9.1 -> 8.8, 3 9.5 -> 9.5, 24
// 10.8 -> 10.0; 12 tiles 4 9.3 -> 10.3, 24 11.0 -> 10.9; 14 tiles 32 0.96 times as fast, 48 1.06; 16 tiles 1 9.1 -> 9.6, 4 9.4 ->
// 12.8, 48 13.4 -> 14.2, 64 14.7 -> 14.8, 96 17.2 -> 15.1.
static bool bucket_is_held(int64_t tiles, int64_t groups) {
  return tiles <= 11 || (tiles <= 16 && groups >= 12 * (tiles - 10));
}
template <int TILES> constexpr int kHeldSide = TILES < 4 ? TILES : 4;   // tiles side by side
// Element e of float4 group j of thread t of tile tile0 + u * side by side + side; beyond d +0.
template <int TILES>
__device__ __forceinline__ void load_held(const float* __restrict__ g, int64_t d, int64_t tile0, int side, int t,
                                          float (&v)[TILES / kHeldSide<TILES>][4][4]) {
  constexpr int kSide = kHeldSide<TILES>, kEach = TILES / kSide;
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  if ((tile0 + TILES) * kTile <= d) {                  // uniform
#pragma unroll
    for (int u = 0; u < kEach; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const floatx4 q = __builtin_nontemporal_load(
            reinterpret_cast<const floatx4*>(g + (tile0 + u * kSide + side) * kTile + 4 * (int64_t)(j * kThreads + t)));
        v[u][j][0] = q.x; v[u][j][1] = q.y; v[u][j][2] = q.z; v[u][j][3] = q.w;
      }
  } else {
#pragma unroll
    for (int u = 0; u < kEach; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t i = (tile0 + u * kSide + side) * kTile + 4 * (int64_t)(j * kThreads + t);
        if (i + 3 < d) {
          const floatx4 q = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(g + i));
          v[u][j][0] = q.x; v[u][j][1] = q.y; v[u][j][2] = q.z; v[u][j][3] = q.w;
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[u][j][e] = i + e < d ? g[i + e] : 0.0f;
        }
      }
  }
}

template <int TILES>
__global__ __launch_bounds__(kHeldSide<TILES> * kThreads, TILES < 16 ? 8 : 4) void quantize_held_kernel(QuantArgs a) {
  constexpr int kSide = kHeldSide<TILES>, kEach = TILES / kSide;
  __shared__ double lds_s1[TILES][kWaves], lds_s2[TILES][kWaves];
  __shared__ uint32_t lds_c[TILES][kWaves];
  const int t = threadIdx.x % kThreads, lane = threadIdx.x % kWave;
  const int side = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads);
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int64_t k = blockIdx.x, tile0 = k * a.tiles_per_bucket;
  const int m = blockIdx.y;
  const float* __restrict__ g = a.g + (int64_t)m * a.g_stride;
  const int64_t left = a.ntiles - tile0;
  const int tiles = (int)(left < a.tiles_per_bucket ? left : a.tiles_per_bucket);   // TILES at most
  float v[kEach][4][4];
  load_held<TILES>(g, a.d, tile0, side, t, v);
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s += (double)fabsf(v[u][j][e]);
    s = wave_sum_f64(s);
    if (lane == 0) lds_s1[u * kSide + side][wave] = s;
  }
  __syncthreads();
  // as the finalize kernels add the tiles' sums: a tree over the lanes, the others' zeros left out
  const auto over_tiles = [lane](const double (&part)[TILES][kWaves]) {
    const int i = lane % 16;
    double s = i < TILES ? (part[i % TILES][0] + part[i % TILES][1]) + (part[i % TILES][2] + part[i % TILES][3]) : 0.0;
    s += dpp_f64<kDppQuadXor1>(s);
    s += dpp_f64<kDppQuadXor2>(s);
    s += dpp_f64<kDppRowHalfMirror>(s);
    return s + dpp_f64<kDppRowMirror>(s);
  };
  const int64_t lo = k * a.bucket_len, n = a.d - lo < a.bucket_len ? a.d - lo : a.bucket_len;
  const float Delta = __uint_as_float(
      (uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(threshold_from_sum(over_tiles(lds_s1), a.thr_coef, n))));
  uint32_t* codes = a.codes + (int64_t)m * a.code_stride;
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    double s = 0.0;
    uint32_t c = 0;
    const int of = u * kSide + side;
    if (of < tiles) {                                    // uniform in the wave
      store_code_word(codes, tile0 + of, a.W, code_tile(v[u], Delta, s, c), t);
      s = wave_sum_f64(s);
    }
    if (lane == 0) { lds_s2[of][wave] = s; lds_c[of][wave] = c; }
  }
  __syncthreads();
  if (threadIdx.x >= kWave) return;
  const double S2 = over_tiles(lds_s2);
  uint32_t C = 0;
  for (int i = 0; i < TILES; ++i) C += lds_c[i][0] + lds_c[i][1] + lds_c[i][2] + lds_c[i][3];
  if (lane == 0) {
    a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(S2, C);
    if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + k] = Delta;
  }
}

// ---- long buckets in one read -------------------------------------------------------------------
//
// The threshold of a long bucket is known only after all of it has been read, but a sample of its tiles
// brackets it closely: [lo, hi] from the mean of every 64th tile (every 32nd of buckets below 16384 tiles) and the
// spread between neighbouring samples, four standard errors to either side (0.25 % for 10^8 Gaussian components; one
// bracket in 15000 misses).  The one pass over the gradient then sums |v| and writes final codes for every component
// outside the bracket; of the few inside (some 9 per 4096) it lists the float4 groups.  When the threshold is known
// the settling pass looks those up in the gradient and joins their codes to the words.  Exactly the same threshold and
// codes as the two-read passes; the kept magnitudes are added in another order.  A caller whose workspace
// has no room for the lists gets the pattern 10, which no message holds, for an open component, and a settling pass that
// reads the codes: the same sums in the same order.
//
// Where the sample says nothing (few tiles, a spread above 8 %, non-finite values) or the threshold falls
// outside its bracket, the settling pass does the second read for that bucket after all.  That costs two
// launches and the sample on top of the two-read passes.
//
// Bound by the read of the gradient (6.4 TB/s in the one pass).  What an open component costs is a cache line read and,
// if it is kept, one changed: hence the four standard errors (five: 2^24 x 4 Gaussian components 97 us for 78, with lists
// that overflow here and there) and the denser sample where the bucket gives few (78 for 86; 10^8 x 8 Student-t with
// it 605 for 595).
// Below 2^25 components the two further launches cost more than the second read (2^24 x 1 27.4 -> 31), and buckets
// of fewer than 4096 tiles give too few samples (2^22: 343 -> 376 at 2^26 x 4 sparse components).
constexpr int64_t kManyTiles = 16384;
constexpr int64_t kSpreadBelow = 512;                    // work-groups, see quantize_settle_listed_kernel
constexpr float kWidestBand = 0.08f;

// Full tiles of bucket k.
__device__ __forceinline__ int64_t whole_tiles(const QuantArgs& a, int64_t k) {
  const int64_t t0 = k * a.tiles_per_bucket, all = a.d / kTile - t0;
  return all < a.tiles_per_bucket ? (all > 0 ? all : 0) : a.tiles_per_bucket;
}

__global__ __launch_bounds__(kThreads) void quantize_sample_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t k = blockIdx.x / a.samples, i = blockIdx.x % a.samples;
  const int m = blockIdx.y;
  if (i >= whole_tiles(a, k) / a.sample_every) return;
  // one tile of every 64 or 32, not always the same one of them
  const int64_t tile = k * a.tiles_per_bucket + i * a.sample_every + (i * 29) % a.sample_every;
  float v[4][4];
  load_tile(a.g + (int64_t)m * a.g_stride, a.d, tile, v);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) s += (double)fabsf(v[j][e]);
  s = block_sum_f64(s, lds_d);
  if (threadIdx.x == 0) a.kept_sum[((int64_t)m * a.nb + k) * a.samples + i] = s;
}

__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void quantize_band_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const double* part = a.kept_sum + ((int64_t)m * a.nb + k) * a.samples;
  const int64_t n = whole_tiles(a, k) / a.sample_every;
  double sum = 0.0, diff = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += kThreads) {
    const double v = part[i], w = i + 1 < n ? part[i + 1] : v;
    sum += v;
    diff += (w - v) * (w - v);
  }
  sum = segment_sum(sum, kThreads, lds_d);
  diff = segment_sum(diff, kThreads, lds_d);
  if (threadIdx.x == 0) {
    float2 band = make_float2(-1.0f, -1.0f);               // no bracket
    if (n >= 16) {
      // neighbouring samples differ by two independent deviations; trends along the vector drop out
      const double mean = sum / (double)n, rel = 4.0 * sqrt(diff / (2.0 * (double)(n - 1)) / (double)n) / mean + 1e-6;
      const double mid = (double)a.thr_coef * mean / (double)kTile;
      if (mean > 0.0 && rel < (double)kWidestBand && mid < 1e38)
        band = make_float2((float)(mid * (1.0 - rel)), (float)(mid * (1.0 + rel)));
    }
    a.band[(int64_t)m * a.nb + k] = band;
  }
}

// The one pass: tile sums of |v|; with a bracket also codes, sums and counts of what is certainly kept, and the open
// components, LISTED or marked.
template <bool LISTED>
__global__ __launch_bounds__(kThreads) void quantize_bracketed_kernel(QuantArgs a) {
  __shared__ double lds_s1[kWaves];
  __shared__ double lds_s2[kWaves];
  __shared__ uint32_t lds_c[kWaves];
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  const int t = threadIdx.x;
  const int64_t at = (int64_t)m * a.ntiles + tile;
  const float2 band = a.band[(int64_t)m * a.nb + tile / a.tiles_per_bucket];
  float v[4][4];
  load_tile_stream(a.g + (int64_t)m * a.g_stride, a.d, tile, v);
  double s1 = 0.0, s2 = 0.0;
  if (!(band.x >= 0.0f)) {                               // uniform; the settling pass codes the tile
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s1 += (double)fabsf(v[j][e]);
    const double S1 = block_sum_f64(s1, lds_s1);
    if (t == 0) a.part_sum[at] = S1;
    return;
  }
  uint32_t wave_cnt = 0;
  uint64_t open[4][4];
  uint32_t word = code_outside(v, band, s1, s2, wave_cnt, open);
  if (!LISTED) {
    uint32_t marks = 0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float av = fabsf(v[i / 4][i % 4]);
      marks |= av > band.x && !(av > band.y) ? 2u << (2 * i) : 0u;
    }
    word |= quad_transpose(marks);
  }
  store_code_word(a.codes + (int64_t)m * a.code_stride, tile, a.W, word, threadIdx.x, a.through);
  if (LISTED) wave_cnt |= list_open(open, a.open + (at * kWaves + t / kWave) * kOpenSlots) << 16;
  const double S1 = wave_sum_f64(s1), S2 = wave_sum_f64(s2);
  if (t % kWave == 0) { lds_s1[t / kWave] = S1; lds_s2[t / kWave] = S2; lds_c[t / kWave] = wave_cnt; }
  __syncthreads();
  if (t == 0) {
    a.part_sum[at] = (lds_s1[0] + lds_s1[1]) + (lds_s1[2] + lds_s1[3]);
    a.kept_sum[at] = (lds_s2[0] + lds_s2[1]) + (lds_s2[2] + lds_s2[3]);
    a.part_cnt[at] = tile_counts(lds_c);
  }
}

// A tile read again: its codes for threshold D, and what they keep per wave.
__device__ __forceinline__ void code_again(const QuantArgs& a, int m, int64_t tile, float D, double* wave_sum,
                                           uint32_t* wave_cnt) {
  float v[4][4];
  load_tile_stream(a.g + (int64_t)m * a.g_stride, a.d, tile, v);
  double s = 0.0;
  uint32_t c = 0;
  store_code_word(a.codes + (int64_t)m * a.code_stride, tile, a.W, code_tile(v, D, s, c), threadIdx.x);
  s = wave_sum_f64(s);
  if (threadIdx.x % kWave == 0) { wave_sum[threadIdx.x / kWave] = s; wave_cnt[threadIdx.x / kWave] = c; }
}
// The settling pass leaves a sum and a count of all that eight tiles keep, in the place of the tile sums of |v|, which
// the threshold has been made of: [M][nb * settle_groups] sums, then as many counts.  Called by the first wave, lane l with
// tile l of the group's eights and its four waves' sums and counts, or all of it in the first ones' place; `live`: it has such an eight.
struct TileKept {
  double sum[kWaves];
  uint32_t cnt[kWaves];
};
__device__ __forceinline__ void settled_parts(const QuantArgs& a, int m, int64_t part, bool live, bool again, const TileKept& k) {
  double s = again ? (k.sum[0] + k.sum[1]) + (k.sum[2] + k.sum[3]) : k.sum[0];
  uint32_t c = again ? k.cnt[0] + k.cnt[1] + k.cnt[2] + k.cnt[3] : k.cnt[0];
  s += dpp_f64<kDppQuadXor1>(s);        c += (uint32_t)dpp_i32<kDppQuadXor1>((int)c);
  s += dpp_f64<kDppQuadXor2>(s);        c += (uint32_t)dpp_i32<kDppQuadXor2>((int)c);
  s += dpp_f64<kDppRowHalfMirror>(s);   c += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)c);
  if (live && threadIdx.x % 8 == 0) {
    const int64_t groups = a.nb * a.settle_groups, at = (int64_t)m * groups + part;
    a.part_sum[at] = s;
    reinterpret_cast<uint32_t*>(a.part_sum + gridDim.y * groups)[at] = c;
  }
}

// With lists: a wave per eight tiles, eight lanes per tile, no look at the codes.  Tiles that have to be coded again are
// left to the whole work-group.  Bound by latency where few components are open (10^8 x 8 10 %-dense Student-t 76 us
// with marks, 26 with lists), by the lines that they touch where many are.
// A bucket without a bracket (or whose threshold lies outside) is coded again as a whole, and 32 tiles one after the other
// leave the chip idle where there are few groups: then the grid has four layers (kSpreadBelow), each of which codes one of
// the four eights of such a bucket, and the first one alone settles the others (2^24 x 2 components, one in 1000 not 0, the
// whole call 74 -> 58 us; 512 groups, 2^24 x 4, keep the chip busy: 108 with eights as groups and with four of them).
__global__ __launch_bounds__(kThreads) void quantize_settle_listed_kernel(QuantArgs a) {
  __shared__ TileKept kept[kWaves * kSettleTiles];
  __shared__ uint32_t lds_again[kWaves];
  const int t = threadIdx.x, lane = t % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(t / kWave);
  const int64_t per_bucket = (a.settle_groups + kWaves - 1) / kWaves;
  const int64_t k = blockIdx.x / per_bucket, part0 = (blockIdx.x % per_bucket) * kWaves;
  const int m = blockIdx.y;
  const int64_t tile0 = k * a.tiles_per_bucket + part0 * kSettleTiles;
  const int64_t bucket1 = (k + 1) * a.tiles_per_bucket < a.ntiles ? (k + 1) * a.tiles_per_bucket : a.ntiles;
  const int own = wave * kSettleTiles + lane / 8;        // of the 32 tiles
  const int64_t tile = tile0 + own, at = (int64_t)m * a.ntiles + tile;
  const float D = a.thr_ws[(int64_t)m * a.nb + k];
  const float2 band = a.band[(int64_t)m * a.nb + k];
  const bool all = gridDim.z == 1 || bracket_held(band, D);
  const int eight = (int)blockIdx.z;
  if (all && eight != 0) return;                         // uniform
  const bool live = tile < bucket1 && (all || wave == eight);
  const uint32_t counts = live ? a.part_cnt[at] : 0u;
  const double certain = live ? a.kept_sum[at] : 0.0;
  const bool again = live && (!bracket_held(band, D) || too_many_open(counts));
  double s = 0.0;
  uint32_t c = 0;
  if (live && !again) {
    const uint32_t list = (lane & 7) >> 1, n = (counts >> (16 + 4 * list)) & 15u;
    settle_listed<4>(a.open + (at * kWaves + list) * kOpenSlots, (uint32_t)lane & 1u, 2u, n,
                     a.g + (int64_t)m * a.g_stride + tile * kTile, a.d - tile * kTile, band, D,
                     a.codes + (int64_t)m * a.code_stride + tile * kTileWords, s, c);
  }
  s += dpp_f64<kDppQuadXor1>(s);        c += (uint32_t)dpp_i32<kDppQuadXor1>((int)c);
  s += dpp_f64<kDppQuadXor2>(s);        c += (uint32_t)dpp_i32<kDppQuadXor2>((int)c);
  s += dpp_f64<kDppRowHalfMirror>(s);   c += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)c);
  const uint64_t again_lanes = __ballot(again);          // eight equal bits per tile
  if ((lane & 7) == 0 && !again) {
    kept[own].sum[0] = live ? certain + s : 0.0;
    kept[own].cnt[0] = live ? c + (counts & 0xFFFFu) : 0u;
  }
  if (lane == 0) {
    uint32_t tiles = 0;
#pragma unroll
    for (int u = 0; u < kSettleTiles; ++u) tiles |= (uint32_t)(again_lanes >> (8 * u) & 1ull) << u;
    lds_again[wave] = tiles << (wave * kSettleTiles);
  }
  __syncthreads();
  const uint32_t repeat = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_again[0] | lds_again[1] | lds_again[2] | lds_again[3]));
  for (uint32_t left = repeat; left; left &= left - 1u) {  // uniform
    const int u = __ffs((int)left) - 1;
    code_again(a, m, tile0 + u, D, kept[u].sum, kept[u].cnt);
  }
  if (repeat) __syncthreads();
  if (wave == 0)
    settled_parts(a, m, k * a.settle_groups + part0 + lane / 8,
                  lane < kWaves * kSettleTiles && part0 + lane / 8 < a.settle_groups && (all || lane / 8 == eight),
                  lane < kWaves * kSettleTiles && (repeat >> (lane & 31) & 1u), kept[lane & 31]);
}

// With marks: eight tiles per work-group, thread t holds word t of each.  The same sums in the same order.
__global__ __launch_bounds__(kThreads) void quantize_settle_marked_kernel(QuantArgs a) {
  __shared__ SettleLds lds;
  __shared__ TileKept kept[kSettleTiles];
  const int64_t k = blockIdx.x / a.settle_groups, part = blockIdx.x % a.settle_groups;
  const int m = blockIdx.y;
  const int t = threadIdx.x;
  const int64_t tile0 = k * a.tiles_per_bucket + part * kSettleTiles;
  const int64_t bucket_end = (k + 1) * a.tiles_per_bucket < a.ntiles ? (k + 1) * a.tiles_per_bucket : a.ntiles;
  const int64_t tile1 = tile0 + kSettleTiles < bucket_end ? tile0 + kSettleTiles : bucket_end;
  const uint32_t here = tile1 > tile0 ? (1u << (tile1 - tile0)) - 1u : 0u;   // (the last bucket may be shorter)
  const float D = a.thr_ws[(int64_t)m * a.nb + k];
  uint32_t* codes = a.codes + (int64_t)m * a.code_stride;
  uint32_t repeat = here;
  if (bracket_held(a.band[(int64_t)m * a.nb + k], D)) {
    uint32_t w[kSettleTiles];
#pragma unroll
    for (int u = 0; u < kSettleTiles; ++u) {
      const int64_t widx = (tile0 + u) * kTileWords + t;
      w[u] = tile0 + u < tile1 && widx < a.W ? codes[widx] : 0u;
    }
    bool changed;
    repeat = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)settle_words(a.g + (int64_t)m * a.g_stride, tile0, D, w, lds, &changed));
    if (changed) {
#pragma unroll
      for (int u = 0; u < kSettleTiles; ++u) {
        const int64_t widx = (tile0 + u) * kTileWords + t;
        if (tile0 + u < tile1 && widx < a.W) codes[widx] = w[u];
      }
    }
    if (t < kSettleTiles && !(repeat >> t & 1u)) {
      const bool live = tile0 + t < tile1;
      const int64_t at = (int64_t)m * a.ntiles + tile0 + t;
      kept[t].sum[0] = live ? a.kept_sum[at] + lds.sum[t] : 0.0;
      kept[t].cnt[0] = live ? (a.part_cnt[at] & 0xFFFFu) + lds.count[t] : 0u;
    }
  } else if (t < kSettleTiles && !(here >> t & 1u)) {
    kept[t].sum[0] = 0.0;
    kept[t].cnt[0] = 0u;
  }
  if (repeat) __syncthreads();                           // (a word of a tile that is coded again may have been rewritten)
  for (uint32_t left = repeat; left; left &= left - 1u) {
    const int u = __ffs((int)left) - 1;
    code_again(a, m, tile0 + u, D, kept[u].sum, kept[u].cnt);
  }
  __syncthreads();
  if (t < kWave) settled_parts(a, m, blockIdx.x, t < kSettleTiles, repeat >> (t & 7) & 1u, kept[t & 7]);
}

__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void quantize_settled_scale_kernel(QuantArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ double lds_c[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t t0 = k * a.tiles_per_bucket;
  const int64_t t1 = (t0 + a.tiles_per_bucket) < a.ntiles ? (t0 + a.tiles_per_bucket) : a.ntiles;
  const int64_t groups = a.nb * a.settle_groups, g0 = k * a.settle_groups;
  const int64_t g1 = g0 + (t1 - t0 + kSettleTiles - 1) / kSettleTiles;
  const uint32_t* settled_cnt = reinterpret_cast<const uint32_t*>(a.part_sum + gridDim.y * groups);
  double s, c;
  strided_partial_sums(a.part_sum + (int64_t)m * groups, settled_cnt + (int64_t)m * groups, g0, g1, &s, &c);
  s = segment_sum(s, kThreads, lds_d);
  c = segment_sum(c, kThreads, lds_c);
  if (threadIdx.x == 0)
    a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(s, (uint64_t)c);
}

// ---- stochastic ternary quantizer (TernGrad: max-norm scale, keep probability |v|/s) ----------
//
// Uniform numbers: Philox4x32-10 keyed by the 64-bit seed, counter (j low, j high, worker, step)
// with j the index of the float4 group, so one generator call serves the four components of a
// group (component i takes output word i % 4).  u = (r >> 8) * 2^-24; keep iff u < |v| / s with
// the division in binary32.  The max is exact, so its reduction order is free.

struct StochArgs {
  QuantArgs q;
  uint32_t seed_lo, seed_hi, step;
  int span;                 // tiles per work-group of the pass that finds the maxima
};

__device__ __forceinline__ void philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                              uint32_t k0, uint32_t k1, uint32_t out[4]) {
#pragma unroll
  for (int round = 0; round < 10; ++round) {
    if (round > 0) { k0 += 0x9E3779B9u; k1 += 0xBB67AE85u; }
    const uint64_t p0 = (uint64_t)0xD2511F53u * c0;      // one 32x32->64 multiply each
    const uint64_t p1 = (uint64_t)0xCD9E8D57u * c2;
    // 0x96: exclusive or of three, one instruction
    const uint32_t n0 = __builtin_amdgcn_bitop3_b32((uint32_t)(p1 >> 32), c1, k0, 0x96);
    const uint32_t n2 = __builtin_amdgcn_bitop3_b32((uint32_t)(p0 >> 32), c3, k1, 0x96);
    c0 = n0; c1 = (uint32_t)p1; c2 = n2; c3 = (uint32_t)p0;
  }
  out[0] = c0; out[1] = c1; out[2] = c2; out[3] = c3;
}

// The largest magnitude among the thread's values, NaNs left out.  As whole numbers the negative values' patterns grow
// with the magnitude above all others, the others' below: two three-way maxima for two values.
__device__ __forceinline__ float abs_max(const float* v, int n) {
  uint32_t neg = 0;
  int pos = 0;
  for (int i = 0; i < n; ++i) {
    const uint32_t b = __float_as_uint(v[i]);
    neg = b > neg ? b : neg;
    pos = (int)b > pos ? (int)b : pos;
  }
  uint32_t top = neg & 0x80000000u ? neg & 0x7fffffffu : 0u;
  top = (uint32_t)pos > top ? (uint32_t)pos : top;
  if (__any(top > 0x7f800000u)) {                        // rare: a NaN among the wave's values
    top = 0;
    for (int i = 0; i < n; ++i) {
      const uint32_t b = __float_as_uint(v[i]) & 0x7fffffffu;
      top = b <= 0x7f800000u && b > top ? b : top;
    }
  }
  return __uint_as_float(top);
}
__device__ __forceinline__ float tile_abs_max(const float v[4][4]) { return abs_max(v[0], 16); }

__device__ __forceinline__ float wave_max_f32(float s) {
  float o;
  o = __int_as_float(dpp_i32<kDppQuadXor1>(__float_as_int(s))); s = o > s ? o : s;
  o = __int_as_float(dpp_i32<kDppQuadXor2>(__float_as_int(s))); s = o > s ? o : s;
  o = __int_as_float(dpp_i32<kDppRowHalfMirror>(__float_as_int(s))); s = o > s ? o : s;
  o = __int_as_float(dpp_i32<kDppRowMirror>(__float_as_int(s))); s = o > s ? o : s;
  float r = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), 0));
#pragma unroll
  for (int l = 16; l < 64; l += 16) {
    o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), l));
    r = o > r ? o : r;
  }
  return r;
}

// Hardware conversion: 0 for NaN and below 0, the largest number above the range.
__device__ __forceinline__ uint32_t to_u32_saturated(float x) {
  uint32_t r;
  asm("v_cvt_u32_f32 %0, %1" : "=v"(r) : "v"(x));
  return r;
}

// codes of the tile, float4 group j of every thread with scale sj[j]; element (j, e) of thread t
// is vector index base + 4*(j*256+t)+e
//
// Keep iff u < fl(|v| / s), u = (r >> 8) * 2^-24.  Compared as whole numbers: the reciprocal's product (good to 2.5e-7)
// less a part in 10^6, in units of 2^-32, lies below the quotient, and 8192 units further on above it (5810 would do: of
// the largest quotient, 1, the 1.013e-6 that 0.999999f leaves off, the product's 2.5e-7 and the quotient's own rounding, 3e-8,
// 1.3e-6 in all; one unit; the 255 that r is above u).  Only when r lies between the two
// (probability 2e-6) is the correctly rounded quotient needed, and where the scale leaves the range in which none of the factors
// overflows or loses bits.
// Bound by instruction issue, half of it Philox's, and memory.  2^28 x 4 components, bucket 4096, with margins in binary32
// and fields from selects 800 us, now 713; 2^20 x 16 14.6 -> 12.7, buckets of 256, 2^26 x 4 285 -> 264.
__device__ __forceinline__ void stochastic_codes(const StochArgs& a, const float v[4][4],
                                                 const float sj[4], int64_t tile, int m, int t) {
  float vv[4][4];
  uint64_t kept[4][4];
  const uint64_t grp0 = (uint64_t)tile * (kTile / 4);      // a multiple of 1024: no carry from the thread's part
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float s = sj[j];
    const float below = __builtin_amdgcn_rcpf(s) * (0.999999f * 0x1p32f);
    uint32_t r[4];
    philox4x32_10((uint32_t)grp0 | (uint32_t)(j * kThreads + t), (uint32_t)(grp0 >> 32), (uint32_t)m, a.step, a.seed_lo,
                  a.seed_hi, r);
    // 2^-90 .. 2^125
    bool unsure = __float_as_uint(s) - 0x12800000u > 0x7e000000u - 0x12800000u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      vv[j][e] = v[j][e];
      const uint32_t low = to_u32_saturated(fabsf(v[j][e]) * below);
      uint32_t above;                                    // r - low; the borrow says r < low
      asm("v_sub_co_u32_e64 %0, %1, %2, %3" : "=v"(above), "=s"(kept[j][e]) : "v"(r[e]), "v"(low));
      unsure |= above < 8192u;
    }
    if (__any(unsure)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) kept[j][e] = __ballot((float)(r[e] >> 8) * 0x1p-24f < fabsf(v[j][e]) / s);
    }
  }
  store_code_word(a.q.codes + (int64_t)m * a.q.code_stride, tile, a.q.W, code_word(vv, kept), t);
}

// bucket == tile (4096, or one scale per vector with d <= 4096): one pass
__global__ __launch_bounds__(kThreads) void quantize_stochastic_tile_kernel(StochArgs a) {
  __shared__ float lds_m[kWaves];
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  float v[4][4];
  load_tile_stream(a.q.g + (int64_t)m * a.q.g_stride, a.q.d, tile, v);
  float s = wave_max_f32(tile_abs_max(v));
  if ((threadIdx.x % kWave) == 0) lds_m[threadIdx.x / kWave] = s;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWaves; ++w) s = lds_m[w] > s ? lds_m[w] : s;
  if (threadIdx.x == 0) a.q.scales[(int64_t)m * a.q.scale_stride + tile] = s;
  const float sj[4] = {s, s, s, s};
  stochastic_codes(a, v, sj, tile, m, threadIdx.x);
}

// Maximum over aligned segments of `seg` consecutive threads (a power of two, 16 <= seg <= 256);
// every thread receives its segment's maximum.  Barriers when seg > 64: all threads must call.
__device__ __forceinline__ float segment_max_f32(float v, int seg, float* lds) {
  const int lim = seg < kWave ? seg : kWave;
  for (int off = 1; off < lim; off <<= 1) {
    const float o = __shfl_xor(v, off, kWave);
    v = o > v ? o : v;
  }
  if (seg > kWave) {
    const int wave = threadIdx.x / kWave;
    __syncthreads();
    if ((threadIdx.x % kWave) == 0) lds[wave] = v;
    __syncthreads();
    const int wps = seg / kWave, w0 = wave & ~(wps - 1);
    float r = lds[w0];
    for (int k = 1; k < wps; ++k) r = lds[w0 + k] > r ? lds[w0 + k] : r;
    v = r;
  }
  return v;
}

// buckets of 64 .. 2048 elements: float4 group f = j*256 + t of the tile lies in the tile's bucket
// f / (bucket/4), so a bucket is a segment of bucket/4 consecutive threads of one j (two j's for
// 2048).  Not tuned: one segmented maximum per j.
__global__ __launch_bounds__(kThreads) void quantize_stochastic_bucket_kernel(StochArgs a) {
  __shared__ float lds_m[kWaves];
  const int t = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  float v[4][4];
  load_tile_stream(a.q.g + (int64_t)m * a.q.g_stride, a.q.d, tile, v);
  const int groups = (int)(a.q.bucket_len / 4);          // float4 groups per bucket: 16 .. 512
  const int seg = groups < kThreads ? groups : kThreads;
  float sj[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    sj[j] = segment_max_f32(abs_max(v[j], 4), seg, lds_m);
  }
  if (groups > kThreads) {                               // 2048: j = 0,1 and j = 2,3 share a bucket
    const float lo = sj[0] > sj[1] ? sj[0] : sj[1], hi = sj[2] > sj[3] ? sj[2] : sj[3];
    sj[0] = sj[1] = lo; sj[2] = sj[3] = hi;
  }
  if ((t & (seg - 1)) == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int f = j * kThreads + t;
      if (f % groups == 0) {
        const int64_t kb = tile * (kTile / a.q.bucket_len) + f / groups;
        if (kb < a.q.nb) a.q.scales[(int64_t)m * a.q.scale_stride + kb] = sj[j];
      }
    }
  }
  stochastic_codes(a, v, sj, tile, m, threadIdx.x);
}

// buckets of 2 .. 16 tiles: held as by quantize_held_kernel, the scale is the largest magnitude.  Three launches and two
// reads -> one, us, at 2^26 x 4 components: buckets of 8192 328 -> 196, 16384 329 -> 221, 32768 331 -> 198, 65536 331 -> 247
// (one work-group's bucket fills the registers of a compute unit); 3 000 001 x 8: 34 -> 20, 34 -> 24, 36 -> 24, 36 -> 32;
// one scale for 5000 .. 24 000 components 7 -> 3.5 .. 6.5 (captured).  A work-group takes its time here too: three launches ->
// held, captured, us: 6 tiles 1 work-group 6.9 -> 6.3, 8 7.5 -> 7.9, 48 9.4 -> 8.4; 7 tiles 4 7.2 -> 7.7, 32 8.4 -> 8.7, 48 9.8 ->
// 9.0; 8 tiles 1 6.9 -> 7.8, 4 7.1 -> 9.0, 48 9.7 -> 10.1, 64 10.4 -> 10.3; 16 tiles 1 6.8 -> 11.8, 16 9.9 -> 15.6, 64 15.1 ->
// 16.8, 96 17.4 -> 17.3.
static bool bucket_is_held_stochastic(int64_t tiles, int64_t groups) {
  return tiles <= 6 || (tiles <= 16 && groups >= 6 * tiles);
}
template <int TILES>
__global__ __launch_bounds__(kHeldSide<TILES> * kThreads, TILES < 16 ? 8 : 4) void quantize_stochastic_held_kernel(StochArgs a) {
  constexpr int kSide = kHeldSide<TILES>, kEach = TILES / kSide;
  __shared__ float lds_m[kSide * kWaves];
  const int t = threadIdx.x % kThreads;
  const int side = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kThreads);
  const int64_t k = blockIdx.x, tile0 = k * a.q.tiles_per_bucket;
  const int m = blockIdx.y;
  float v[kEach][4][4];
  load_held<TILES>(a.q.g + (int64_t)m * a.q.g_stride, a.q.d, tile0, side, t, v);
  float s = wave_max_f32(abs_max(v[0][0], kEach * 16));
  if (threadIdx.x % kWave == 0) lds_m[threadIdx.x / kWave] = s;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kSide * kWaves; ++w) s = lds_m[w] > s ? lds_m[w] : s;
  s = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(s)));
  if (threadIdx.x == 0) a.q.scales[(int64_t)m * a.q.scale_stride + k] = s;
  const float sj[4] = {s, s, s, s};
#pragma unroll
  for (int u = 0; u < kEach; ++u) {
    const int of = u * kSide + side;
    if (of < a.q.tiles_per_bucket && tile0 + of < a.q.ntiles) stochastic_codes(a, v[u], sj, tile0 + of, m, t);
  }
}

// longer buckets or one scale per large vector: the maxima fold into scales[] (which an earlier launch zeroed) with
// integer atomic max on the bit pattern of the non-negative float; then the codes, with the finished scale.
// A work-group takes `span` consecutive tiles of a bucket and its maximum goes to the scale once: additions to one address
// follow each other at 42 ns, which was nearly all of the time with one per wave and tile (one scale per vector,
// 2^26 x 4 components 3166 us, now 350; 3 000 001 x 8 288 -> 43).
__global__ __launch_bounds__(kThreads) void quantize_stochastic_max_kernel(StochArgs a) {
  __shared__ float lds_m[kWaves];
  const int64_t per_bucket = (a.q.tiles_per_bucket + a.span - 1) / a.span;
  const int64_t k = blockIdx.x / per_bucket;
  const int64_t tile0 = k * a.q.tiles_per_bucket + (blockIdx.x % per_bucket) * a.span;
  const int64_t bucket1 = (k + 1) * a.q.tiles_per_bucket < a.q.ntiles ? (k + 1) * a.q.tiles_per_bucket : a.q.ntiles;
  const int64_t tile1 = tile0 + a.span < bucket1 ? tile0 + a.span : bucket1;
  const int m = blockIdx.y;
  float s = 0.0f;
#pragma unroll 2
  for (int64_t tile = tile0; tile < tile1; ++tile) {
    float v[4][4];
    load_tile_stream(a.q.g + (int64_t)m * a.q.g_stride, a.q.d, tile, v);
    const float o = tile_abs_max(v);
    s = o > s ? o : s;
  }
  s = wave_max_f32(s);
  if ((threadIdx.x % kWave) == 0) lds_m[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w = 1; w < kWaves; ++w) s = lds_m[w] > s ? lds_m[w] : s;
    if (s > 0.0f)
      atomicMax(reinterpret_cast<unsigned int*>(a.q.scales + (int64_t)m * a.q.scale_stride + k), __float_as_uint(s));
  }
}
__global__ __launch_bounds__(kThreads) void quantize_stochastic_codes_kernel(StochArgs a) {
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  float v[4][4];
  load_tile_stream(a.q.g + (int64_t)m * a.q.g_stride, a.q.d, tile, v);
  const float s = a.q.scales[(int64_t)m * a.q.scale_stride + tile / a.q.tiles_per_bucket];
  const float sj[4] = {s, s, s, s};
  stochastic_codes(a, v, sj, tile, m, threadIdx.x);
}

__global__ __launch_bounds__(kThreads) void zero_scales_kernel(float* scales, int64_t stride, int64_t nb) {
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (k < nb) scales[(int64_t)blockIdx.y * stride + k] = 0.0f;
}

// ---- host side -------------------------------------------------------------------------------

static inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

size_t exact_wide_workspace_bytes(const qa_layout* L);
int exact_thresholds_wide(const qa_layout* L, const float* g, int64_t g_stride, uint32_t* codes, float* scales,
                          float* thresholds, double* part_sum, uint32_t* part_cnt, void* ws, size_t ws_bytes,
                          bool* coded, hipStream_t stream);
void quantize_workspace_parts(const qa_layout* L, void* ws, double** part_sum, uint32_t** part_cnt, float** thr);

size_t quantize_workspace_bytes(const qa_layout* L) {
  if (L->bucket != 0 && L->bucket <= kTile) return 0;
  if (L->bucket == 0 && tiles_of(L->d) == 1) return 0;   // one tile: one pass
  const int64_t nt = tiles_of(L->d), nb = buckets_of(L->d, L->bucket);
  return align256((size_t)L->M * nt * sizeof(double)) + align256((size_t)L->M * nt * sizeof(uint32_t)) +
         align256((size_t)L->M * nb * sizeof(float));
}

// What the one-read form needs on top of it, 0 where it is not taken: buckets of fewer than 4096 tiles
// (128 samples), or less than 2^25 components in all.
constexpr int64_t kOneReadBucketTiles = 4096, kOneReadTiles = 8192;
static size_t one_read_sums_bytes(const qa_layout* L) {
  const int64_t nt = tiles_of(L->d), nb = buckets_of(L->d, L->bucket);
  const int64_t per = L->bucket ? L->bucket / kTile : nt;
  if (per < kOneReadBucketTiles || nt < kOneReadBucketTiles || nt * L->M < kOneReadTiles) return 0;
  return align256((size_t)L->M * nt * sizeof(double)) + align256((size_t)L->M * nb * sizeof(float2));
}
static size_t open_lists_bytes(const qa_layout* L) {
  return (size_t)L->M * tiles_of(L->d) * kWaves * kOpenSlots * sizeof(uint16_t);
}
size_t one_read_bytes(const qa_layout* L) {
  const size_t sums = one_read_sums_bytes(L);
  return sums ? sums + open_lists_bytes(L) : 0;
}

// Where the multi-pass quantizer keeps its per-tile sums, counts and per-bucket thresholds inside
// its workspace (all worker-major).
void quantize_workspace_parts(const qa_layout* L, void* ws, double** part_sum, uint32_t** part_cnt,
                              float** thr) {
  char* p = static_cast<char*>(ws);
  const int64_t nt = tiles_of(L->d);
  *part_sum = reinterpret_cast<double*>(p);
  p += align256((size_t)L->M * nt * sizeof(double));
  *part_cnt = reinterpret_cast<uint32_t*>(p);
  p += align256((size_t)L->M * nt * sizeof(uint32_t));
  *thr = reinterpret_cast<float*>(p);
}

int quantize_launch(const qa_layout* L, const float* g, int64_t g_stride, uint32_t* codes,
                    float* scales, float* thresholds, uint32_t flags, void* ws, size_t ws_bytes,
                    hipStream_t stream) {
  QuantArgs a{};
  a.g = g; a.g_stride = g_stride; a.d = L->d; a.W = words_of(L->d);
  a.codes = codes; a.code_stride = L->code_stride;
  a.scales = scales; a.thresholds = thresholds; a.scale_stride = L->scale_stride;
  a.thr_coef = L->thr_coef;
  a.thresh_given = (flags & QA_THRESH_GIVEN) ? 1 : 0;
  a.through = words_go_through(L, codes) ? 1 : 0;
  a.ntiles = tiles_of(L->d);
  a.nb = buckets_of(L->d, L->bucket);
  const dim3 block(kThreads);
  if (a.ntiles > 0x7fffffffLL) return QA_ERR_INVALID_ARG;
  const dim3 grid_tiles((unsigned)a.ntiles, (unsigned)L->M);
  const bool one_pass = (L->bucket != 0 && L->bucket <= kTile) || (L->bucket == 0 && a.ntiles == 1);
  if ((flags & QA_THRESH_EXACT) && !one_pass) {
    // buckets that span tiles: device-wide search, in the part of the workspace that follows
    // the multi-pass quantizer's own
    const size_t own = quantize_workspace_bytes(L), more = exact_wide_workspace_bytes(L);
    if (!ws || ws_bytes < own + more) return QA_ERR_WORKSPACE;
    if (!aligned(ws, 256)) return QA_ERR_ALIGNMENT;
    bool coded = false;
    quantize_workspace_parts(L, ws, &a.part_sum, &a.part_cnt, &a.thr_ws);
    const int rc = exact_thresholds_wide(L, g, g_stride, codes, scales, thresholds, a.part_sum, a.part_cnt,
                                         static_cast<char*>(ws) + own, ws_bytes - own, &coded, stream);
    if (rc != QA_OK || coded) return rc;
    a.thresh_given = 1;                                  // the passes below read what it wrote
  } else if (flags & QA_THRESH_EXACT) {
    const int log2b = L->bucket ? ilog2(L->bucket) : 12;
    if (log2b >= 9) {                                    // threshold, scale and codes in one pass
      QuantArgs q = a;
      q.thresh_given = 1;                                // for the buckets that are ranked behind it
      q.bucket_len = 1 << log2b;
      q.log2b = log2b;
      const dim3 grid_waves((unsigned)((a.nb + kWaves - 1) / kWaves), (unsigned)L->M);
      const dim3 grid_spans((unsigned)((a.ntiles + kRankSpan - 1) / kRankSpan), (unsigned)L->M);
      if (log2b == 9) {
        hipLaunchKernelGGL(exact_histogram_kernel<9>, grid_waves, block, 0, stream, q);
        hipLaunchKernelGGL(exact_rank_marked_kernel<9>, grid_spans, block, 0, stream, q);
      } else if (log2b == 10) {
        hipLaunchKernelGGL(exact_histogram_kernel<10>, grid_waves, block, 0, stream, q);
        hipLaunchKernelGGL(exact_rank_marked_kernel<10>, grid_spans, block, 0, stream, q);
      } else if (log2b == 11) {
        hipLaunchKernelGGL(exact_histogram_kernel<11>, grid_waves, block, 0, stream, q);
        hipLaunchKernelGGL(exact_rank_marked_kernel<11>, grid_spans, block, 0, stream, q);
      } else {
        hipLaunchKernelGGL(exact_histogram_kernel<12>, grid_waves, block, 0, stream, q);
        hipLaunchKernelGGL(exact_rank_marked_kernel<12>, grid_spans, block, 0, stream, q);
      }
      return launch_status();
    }
    // one ranking network per tile for the smaller buckets
    switch (log2b) {
      case 6: hipLaunchKernelGGL(exact_threshold_kernel<6>, grid_tiles, block, 0, stream, a); break;
      case 7: hipLaunchKernelGGL(exact_threshold_kernel<7>, grid_tiles, block, 0, stream, a); break;
      default: hipLaunchKernelGGL(exact_threshold_kernel<8>, grid_tiles, block, 0, stream, a); break;
    }
    a.thresh_given = 1;                                  // the passes below read what it wrote
  }

  const auto launch_buckets = [&](auto log2b) {
    if (a.thresh_given) hipLaunchKernelGGL((quantize_bucket_kernel<log2b(), true>), grid_tiles, block, 0, stream, a);
    else hipLaunchKernelGGL((quantize_bucket_kernel<log2b(), false>), grid_tiles, block, 0, stream, a);
  };
  const auto launch_tile = [&] {
    if (a.thresh_given) hipLaunchKernelGGL(quantize_tile_kernel<true>, grid_tiles, block, 0, stream, a);
    else hipLaunchKernelGGL(quantize_tile_kernel<false>, grid_tiles, block, 0, stream, a);
  };
  if (L->bucket != 0 && L->bucket <= kTile) {
    a.log2b = ilog2(L->bucket);
    a.bucket_len = L->bucket;
    switch (a.log2b) {
      case 6: launch_buckets(std::integral_constant<int, 6>()); break;
      case 7: launch_buckets(std::integral_constant<int, 7>()); break;
      case 8: launch_buckets(std::integral_constant<int, 8>()); break;
      case 9: launch_buckets(std::integral_constant<int, 9>()); break;
      case 10: launch_buckets(std::integral_constant<int, 10>()); break;
      case 11: launch_buckets(std::integral_constant<int, 11>()); break;
      default: launch_tile(); break;
    }
    return launch_status();
  }
  if (L->bucket == 0 && a.ntiles == 1) {                 // the whole vector is one tile: one pass
    a.log2b = ilog2(kTile);
    a.bucket_len = kTile;
    launch_tile();
    return launch_status();
  }

  const size_t need = quantize_workspace_bytes(L);
  if (!ws || ws_bytes < need) return QA_ERR_WORKSPACE;
  if (!aligned(ws, 256)) return QA_ERR_ALIGNMENT;
  quantize_workspace_parts(L, ws, &a.part_sum, &a.part_cnt, &a.thr_ws);
  a.bucket_len = L->bucket ? L->bucket : L->d;
  a.tiles_per_bucket = L->bucket ? L->bucket / kTile : a.ntiles;
  a.log2b = L->bucket ? ilog2(L->bucket) : 0;
  const dim3 grid_buckets((unsigned)a.nb, (unsigned)L->M);

  const int64_t held = a.tiles_per_bucket < a.ntiles ? a.tiles_per_bucket : a.ntiles;
  if (!a.thresh_given && !(flags & kQuantAbsPartialsGiven) && bucket_is_held(held, a.nb * L->M)) {
    const dim3 block_of_4(4 * kThreads);
    if (held <= 2) hipLaunchKernelGGL(quantize_held_kernel<2>, grid_buckets, dim3(2 * kThreads), 0, stream, a);
    else if (held <= 4) hipLaunchKernelGGL(quantize_held_kernel<4>, grid_buckets, block_of_4, 0, stream, a);
    else if (held <= 8) hipLaunchKernelGGL(quantize_held_kernel<8>, grid_buckets, block_of_4, 0, stream, a);
    else hipLaunchKernelGGL(quantize_held_kernel<16>, grid_buckets, block_of_4, 0, stream, a);
    return launch_status();
  }

  const size_t one_read_sums = one_read_sums_bytes(L);
  if (!a.thresh_given && !(flags & kQuantAbsPartialsGiven) && one_read_sums != 0 && ws_bytes >= need + one_read_sums) {
    char* p = static_cast<char*>(ws) + need;
    a.kept_sum = reinterpret_cast<double*>(p);
    a.band = reinterpret_cast<float2*>(p + align256((size_t)L->M * a.ntiles * sizeof(double)));
    if (ws_bytes >= need + one_read_sums + open_lists_bytes(L)) a.open = reinterpret_cast<uint16_t*>(p + one_read_sums);
    // the tiles that the vector has: a bucket may be nominally far longer, and the settling pass leaves its
    // sums and counts in the place of the tile sums
    if (a.tiles_per_bucket > a.ntiles) a.tiles_per_bucket = a.ntiles;
    a.sample_every = a.tiles_per_bucket >= kManyTiles ? 64 : 32;
    a.samples = a.tiles_per_bucket / a.sample_every;
    a.settle_groups = (a.tiles_per_bucket + kSettleTiles - 1) / kSettleTiles;
    if (a.nb * a.samples <= 0x7fffffffLL && a.nb * a.settle_groups <= 0x7fffffffLL) {
      const dim3 grid_samples((unsigned)(a.nb * a.samples), (unsigned)L->M);
      const int64_t settle = a.nb * (a.open ? (a.settle_groups + kWaves - 1) / kWaves : a.settle_groups);
      const dim3 grid_settle((unsigned)settle, (unsigned)L->M, a.open && settle * L->M < kSpreadBelow ? kWaves : 1);
      hipLaunchKernelGGL(quantize_sample_kernel, grid_samples, block, 0, stream, a);
      hipLaunchKernelGGL(quantize_band_kernel, grid_buckets, block, 0, stream, a);
      if (a.open) hipLaunchKernelGGL(quantize_bracketed_kernel<true>, grid_tiles, block, 0, stream, a);
      else hipLaunchKernelGGL(quantize_bracketed_kernel<false>, grid_tiles, block, 0, stream, a);
      hipLaunchKernelGGL(quantize_threshold_finalize_kernel, grid_buckets, block, 0, stream, a);
      if (a.open) hipLaunchKernelGGL(quantize_settle_listed_kernel, grid_settle, block, 0, stream, a);
      else hipLaunchKernelGGL(quantize_settle_marked_kernel, grid_settle, block, 0, stream, a);
      hipLaunchKernelGGL(quantize_settled_scale_kernel, grid_buckets, block, 0, stream, a);
      return launch_status();
    }
  }
  if (!a.thresh_given) {
    if (!(flags & kQuantAbsPartialsGiven))
      hipLaunchKernelGGL(quantize_abs_partial_kernel, grid_tiles, block, 0, stream, a);
    hipLaunchKernelGGL(quantize_threshold_finalize_kernel, grid_buckets, block, 0, stream, a);
  }
  hipLaunchKernelGGL(quantize_codes_partial_kernel, grid_tiles, block, 0, stream, a);
  hipLaunchKernelGGL(quantize_scale_finalize_kernel, grid_buckets, block, 0, stream, a);
  return launch_status();
}

// The multi-pass quantizer's finalize kernels alone, for a producer that leaves the partial sums in
// the quantizer's workspace itself and never materialises the quantizer's input (the steps that
// form Q(SynQ) from the messages).  which = 0: thresholds from the partial sums of |v| (also
// written to thresholds[] if given); which = 1: scales from the partial sums and counts of the
// kept |v|.  n_partials = 0: one partial per 4096-tile, as the quantizer's own passes leave them;
// otherwise the layout must have a single bucket, whose n_partials partials (each over some whole
// tiles, in order) are at the start of the arrays.
int quantize_finalize_launch(const qa_layout* L, int which, int64_t n_partials, float* scales,
                             float* thresholds, void* ws, size_t ws_bytes, hipStream_t stream) {
  const size_t need = quantize_workspace_bytes(L);
  if (need == 0 || !ws || ws_bytes < need) return QA_ERR_WORKSPACE;   // (need == 0: a one-pass layout)
  if (!aligned(ws, 256)) return QA_ERR_ALIGNMENT;
  QuantArgs a{};
  a.d = L->d; a.W = words_of(L->d);
  a.scales = scales; a.thresholds = thresholds; a.scale_stride = L->scale_stride;
  a.thr_coef = L->thr_coef;
  a.ntiles = tiles_of(L->d);
  a.nb = buckets_of(L->d, L->bucket);
  quantize_workspace_parts(L, ws, &a.part_sum, &a.part_cnt, &a.thr_ws);
  a.bucket_len = L->bucket ? L->bucket : L->d;
  a.tiles_per_bucket = L->bucket ? L->bucket / kTile : a.ntiles;
  if (n_partials != 0) {
    if (a.nb != 1 || n_partials < 1 || n_partials > a.ntiles || L->M != 1) return QA_ERR_INVALID_ARG;
    a.ntiles = n_partials; a.tiles_per_bucket = n_partials;
  }
  const dim3 grid_buckets((unsigned)a.nb, (unsigned)L->M), block(kThreads);
  if (which == 0) hipLaunchKernelGGL(quantize_threshold_finalize_kernel, grid_buckets, block, 0, stream, a);
  else hipLaunchKernelGGL(quantize_scale_finalize_kernel, grid_buckets, block, 0, stream, a);
  return launch_status();
}

// ---- scratch that the library owns, for callers that cannot hand over a workspace -------------
//
// The multi-pass quantizer keeps per-tile partial sums, counts and the thresholds between its
// launches.  qa_quantize_pack_static keeps them in this array instead of a caller's workspace.
// Every GPU the library runs on holds its own copy until the process ends; its device address
// is looked up once per device and that address (never the symbol itself) is what host code
// hands to the kernels.  A call is accepted by the size of its partial sums (12 bytes per worker and
// tile); the rest is for the one-read form, which adds 8 bytes to those 12 and 8 per worker and bucket of at
// least 4096 tiles: the static call takes it wherever qa_quantize_pack with its full workspace does, so
// that their sums are added in the same order.  Up to some 49 600 tiles of all workers (2 * 10^8 components) the array
// has room for the lists of open groups as well, another 128 bytes each; beyond, what is open is marked in the
// code words, with the same result.
constexpr size_t kScratchSums = QA_STATIC_SCRATCH_BYTES, kScratchBytes = size_t(7) << 20;
static_assert(kScratchBytes >= kScratchSums + kScratchSums / 12 * 8 + kScratchSums / 12 / kOneReadBucketTiles * 16 + 512,
              "room for the one-read form of every accepted layout");
static __device__ __align__(256) __attribute__((used)) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex scratch_mutex;
static void* scratch_ptr[kMaxDevices];    // device address of `scratch` on each GPU, 0 = not yet asked

// Address of the current device's copy of `scratch`.
static int scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return QA_ERR_LAUNCH;
  }
  std::lock_guard<std::mutex> lock(scratch_mutex);
  if (!scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return QA_ERR_LAUNCH;
    }
    scratch_ptr[dev] = p;
  }
  *out = scratch_ptr[dev];
  return QA_OK;
}

}  // namespace qa

extern "C" int qa_quantize_pack_static(const qa_layout* layout, const float* g, int64_t g_stride,
                                       uint32_t* codes, float* scales, float* thresholds,
                                       uint32_t flags, void* stream) {
  using namespace qa;
  int rc = check_layout(layout);
  if (rc != QA_OK) return rc;
  if (!g || !codes || !scales) return QA_ERR_INVALID_ARG;
  if (flags & ~(QA_THRESH_GIVEN | QA_THRESH_EXACT)) return QA_ERR_INVALID_ARG;
  if ((flags & QA_THRESH_GIVEN) && (flags & QA_THRESH_EXACT)) return QA_ERR_INVALID_ARG;
  if ((flags & (QA_THRESH_GIVEN | QA_THRESH_EXACT)) && !thresholds) return QA_ERR_INVALID_ARG;
  if (g_stride < layout->d || (g_stride % 4) != 0) return QA_ERR_INVALID_ARG;
  if (!aligned(g, 16) || !aligned(codes, 4) || !aligned(scales, 4) || !aligned(thresholds, 4))
    return QA_ERR_ALIGNMENT;
  const size_t need = quantize_workspace_bytes(layout);
  if (need > kScratchSums) return QA_ERR_TOO_LARGE;
  // the device-wide search has a sort's worth of scratch in reserve: not from this array
  if ((flags & QA_THRESH_EXACT) && exact_wide_workspace_bytes(layout) != 0) return QA_ERR_TOO_LARGE;
  void* ws = nullptr;
  if (need) {
    rc = scratch_address(&ws);
    if (rc != QA_OK) return rc;
  }
  // every partial that a later launch reads is written by an earlier launch of the same call:
  // nothing in the array has to start at zero
  return quantize_launch(layout, g, g_stride, codes, scales, thresholds, flags, ws,
                         need ? kScratchBytes : 0, static_cast<hipStream_t>(stream));
}

extern "C" int qa_quantize_pack(const qa_layout* layout, const float* g, int64_t g_stride,
                                uint32_t* codes, float* scales, float* thresholds, uint32_t flags,
                                void* ws, size_t ws_bytes, void* stream) {
  using namespace qa;
  int rc = check_layout(layout);
  if (rc != QA_OK) return rc;
  if (!g || !codes || !scales) return QA_ERR_INVALID_ARG;
  if (flags & ~(QA_THRESH_GIVEN | QA_THRESH_EXACT)) return QA_ERR_INVALID_ARG;
  if ((flags & QA_THRESH_GIVEN) && (flags & QA_THRESH_EXACT)) return QA_ERR_INVALID_ARG;
  if ((flags & (QA_THRESH_GIVEN | QA_THRESH_EXACT)) && !thresholds) return QA_ERR_INVALID_ARG;
  if (g_stride < layout->d || (g_stride % 4) != 0) return QA_ERR_INVALID_ARG;
  if (!aligned(g, 16) || !aligned(codes, 4) || !aligned(scales, 4) || !aligned(thresholds, 4))
    return QA_ERR_ALIGNMENT;
  return quantize_launch(layout, g, g_stride, codes, scales, thresholds, flags, ws, ws_bytes,
                         static_cast<hipStream_t>(stream));
}

extern "C" int qa_quantize_pack_stochastic(const qa_layout* layout, const float* g, int64_t g_stride,
                                           uint32_t* codes, float* scales, uint64_t seed,
                                           uint32_t step, void* stream_) {
  using namespace qa;
  int rc = check_layout(layout);
  if (rc != QA_OK) return rc;
  if (!g || !codes || !scales) return QA_ERR_INVALID_ARG;
  if (g_stride < layout->d || (g_stride % 4) != 0) return QA_ERR_INVALID_ARG;
  if (!aligned(g, 16) || !aligned(codes, 4) || !aligned(scales, 4)) return QA_ERR_ALIGNMENT;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  StochArgs a{};
  a.q.g = g; a.q.g_stride = g_stride; a.q.d = layout->d; a.q.W = words_of(layout->d);
  a.q.codes = codes; a.q.code_stride = layout->code_stride;
  a.q.scales = scales; a.q.scale_stride = layout->scale_stride;
  a.q.ntiles = tiles_of(layout->d);
  a.q.nb = buckets_of(layout->d, layout->bucket);
  a.seed_lo = (uint32_t)seed; a.seed_hi = (uint32_t)(seed >> 32); a.step = step;
  if (a.q.ntiles > 0x7fffffffLL) return QA_ERR_INVALID_ARG;
  const dim3 block(kThreads), grid((unsigned)a.q.ntiles, (unsigned)layout->M);
  if (layout->bucket != 0 && layout->bucket < kTile) {
    a.q.bucket_len = layout->bucket;
    hipLaunchKernelGGL(quantize_stochastic_bucket_kernel, grid, block, 0, stream, a);
    return launch_status();
  }
  if (layout->bucket == kTile || a.q.ntiles == 1) {
    hipLaunchKernelGGL(quantize_stochastic_tile_kernel, grid, block, 0, stream, a);
    return launch_status();
  }
  a.q.tiles_per_bucket = layout->bucket ? layout->bucket / kTile : a.q.ntiles;
  if (a.q.tiles_per_bucket > a.q.ntiles) a.q.tiles_per_bucket = a.q.ntiles;
  if (bucket_is_held_stochastic(a.q.tiles_per_bucket, a.q.nb * layout->M)) {
    const dim3 buckets((unsigned)a.q.nb, (unsigned)layout->M), block_of_4(4 * kThreads);
    if (a.q.tiles_per_bucket <= 2) hipLaunchKernelGGL(quantize_stochastic_held_kernel<2>, buckets, dim3(2 * kThreads), 0, stream, a);
    else if (a.q.tiles_per_bucket <= 4) hipLaunchKernelGGL(quantize_stochastic_held_kernel<4>, buckets, block_of_4, 0, stream, a);
    else if (a.q.tiles_per_bucket <= 8) hipLaunchKernelGGL(quantize_stochastic_held_kernel<8>, buckets, block_of_4, 0, stream, a);
    else hipLaunchKernelGGL(quantize_stochastic_held_kernel<16>, buckets, block_of_4, 0, stream, a);
    return launch_status();
  }
  hipLaunchKernelGGL(zero_scales_kernel, dim3((unsigned)((a.q.nb + kThreads - 1) / kThreads),
                                              (unsigned)layout->M), block, 0, stream, scales,
                     layout->scale_stride, a.q.nb);
  constexpr int64_t kMaxGroups = 1024;                   // some work-groups per compute unit, up to 16 tiles each
  const int64_t tiles = a.q.ntiles * layout->M;
  a.span = (int)(tiles / kMaxGroups < 1 ? 1 : (tiles / kMaxGroups < 16 ? tiles / kMaxGroups : 16));
  const int64_t groups = a.q.nb * ((a.q.tiles_per_bucket + a.span - 1) / a.span);
  hipLaunchKernelGGL(quantize_stochastic_max_kernel, dim3((unsigned)groups, (unsigned)layout->M), block, 0, stream, a);
  hipLaunchKernelGGL(quantize_stochastic_codes_kernel, grid, block, 0, stream, a);
  return launch_status();
}
