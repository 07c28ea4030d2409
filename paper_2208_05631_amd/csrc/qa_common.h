// Internal helpers of libqadagrad (gfx950 only).  Not part of the public interface.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qadagrad.h"

namespace qa {

constexpr int kThreads = 256;          // work-group size of every tile kernel: 4 wave64
constexpr int kWave = 64;
constexpr int kWaves = kThreads / kWave;
constexpr int kTile = 4096;            // coordinates per work-group tile = 256 code words
constexpr int kTileWords = kTile / 16;

// ---- host-side argument checks ---------------------------------------------------------

inline bool is_pow2(int64_t v) { return v > 0 && (v & (v - 1)) == 0; }
inline int ilog2(int64_t v) { int l = 0; while ((int64_t(1) << l) < v) ++l; return l; }
inline bool aligned(const void* p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

inline int64_t words_of(int64_t d) { return (d + 15) / 16; }
inline int64_t tiles_of(int64_t d) { return (d + kTile - 1) / kTile; }
inline int64_t buckets_of(int64_t d, int64_t bucket) {
  return bucket > 0 ? (d + bucket - 1) / bucket : 1;
}

// Layout rules shared by every entry point that takes a qa_layout.
inline int check_layout(const qa_layout* L) {
  if (!L) return QA_ERR_INVALID_ARG;
  if (L->d < 1 || L->d >= (int64_t(1) << 40)) return QA_ERR_INVALID_ARG;
  if (L->M < 1 || L->M > 4096) return QA_ERR_INVALID_ARG;
  if (L->bucket != 0 && (L->bucket < 64 || !is_pow2(L->bucket))) return QA_ERR_INVALID_ARG;
  if (!(L->thr_coef > 0.0f) || !(L->thr_coef < 1e30f)) return QA_ERR_INVALID_ARG;
  if (L->code_stride < words_of(L->d)) return QA_ERR_INVALID_ARG;
  if (L->scale_stride < buckets_of(L->d, L->bucket)) return QA_ERR_INVALID_ARG;
  return QA_OK;
}

// Internal flag of quantize_launch (never accepted from the C ABI): the tile sums of |v| are
// already in the workspace, whose first M*ntiles doubles hold them (worker-major), so the first
// pass over the input is skipped.  Used when the producer of the input computed them on the way.
constexpr uint32_t kQuantAbsPartialsGiven = 0x80000000u;
inline int launch_status() { return hipGetLastError() == hipSuccess ? QA_OK : QA_ERR_LAUNCH; }

// ---- device-side reductions (binary64, fixed order: run-to-run deterministic) -----------

#if defined(__HIPCC__)

__device__ __forceinline__ double shfl_xor_f64(double v, int mask) {
  return __shfl_xor(v, mask, kWave);
}

// ---- wave64 sums with DPP (no LDS traffic): every lane receives the sum of all 64 lanes ----
template <int CTRL>
__device__ __forceinline__ int dpp_i32(int v) {
  // every lane has a source; no former value of the target, which would be copied there first and would keep the
  // move from being folded into the instruction that uses it
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, true);
}
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const int lo = dpp_i32<CTRL>(__double2loint(v)), hi = dpp_i32<CTRL>(__double2hiint(v));
  return __hiloint2double(hi, lo);
}
constexpr int kDppQuadXor1 = 0xB1;      // quad_perm:[1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;      // quad_perm:[2,3,0,1]
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowMirror = 0x140;

__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double wave_sum_f64(double v) {
  v += dpp_f64<kDppQuadXor1>(v);
  v += dpp_f64<kDppQuadXor2>(v);
  v += dpp_f64<kDppRowHalfMirror>(v);
  v += dpp_f64<kDppRowMirror>(v);        // every lane: sum of its row of 16
  return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  v += (uint32_t)dpp_i32<kDppQuadXor1>((int)v);
  v += (uint32_t)dpp_i32<kDppQuadXor2>((int)v);
  v += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)v);
  v += (uint32_t)dpp_i32<kDppRowMirror>((int)v);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 0) + (uint32_t)__builtin_amdgcn_readlane((int)v, 16) +
         (uint32_t)__builtin_amdgcn_readlane((int)v, 32) + (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
}

// The same pattern for any associative, commutative operation on 32-bit integers.
template <typename F>
__device__ __forceinline__ int wave_reduce_i32(int v, F f) {
  v = f(v, dpp_i32<kDppQuadXor1>(v));
  v = f(v, dpp_i32<kDppQuadXor2>(v));
  v = f(v, dpp_i32<kDppRowHalfMirror>(v));
  v = f(v, dpp_i32<kDppRowMirror>(v));
  return f(f(__builtin_amdgcn_readlane(v, 0), __builtin_amdgcn_readlane(v, 16)),
           f(__builtin_amdgcn_readlane(v, 32), __builtin_amdgcn_readlane(v, 48)));
}

// Inclusive prefix sums over the 64 lanes with DPP: shifts within each row of 16 lanes, then the last lane of a row
// is broadcast into the following rows.  A lane without a source adds 0.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t lanes_or_zero_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double lanes_or_zero_f64(double v) {
  return __hiloint2double((int)lanes_or_zero_u32<CTRL, ROW_MASK>((uint32_t)__double2hiint(v)),
                          (int)lanes_or_zero_u32<CTRL, ROW_MASK>((uint32_t)__double2loint(v)));
}
__device__ __forceinline__ double wave_scan_f64(double v) {
  v += lanes_or_zero_f64<0x111, 0xF>(v);      // row_shr:1
  v += lanes_or_zero_f64<0x112, 0xF>(v);      // row_shr:2
  v += lanes_or_zero_f64<0x114, 0xF>(v);      // row_shr:4
  v += lanes_or_zero_f64<0x118, 0xF>(v);      // row_shr:8
  v += lanes_or_zero_f64<0x142, 0xA>(v);      // row_bcast:15 into rows 1 and 3
  v += lanes_or_zero_f64<0x143, 0xC>(v);      // row_bcast:31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t v) {
  v += lanes_or_zero_u32<0x111, 0xF>(v);
  v += lanes_or_zero_u32<0x112, 0xF>(v);
  v += lanes_or_zero_u32<0x114, 0xF>(v);
  v += lanes_or_zero_u32<0x118, 0xF>(v);
  v += lanes_or_zero_u32<0x142, 0xA>(v);
  v += lanes_or_zero_u32<0x143, 0xC>(v);
  return v;
}

// Sum over the whole 256-thread work-group, returned to every thread.  One barrier; `lds`
// (kWaves doubles) must not be reused by another call before a later barrier.
__device__ __forceinline__ double block_sum_f64(double v, double* lds) {
  v = wave_sum_f64(v);
  if ((threadIdx.x % kWave) == 0) lds[threadIdx.x / kWave] = v;
  __syncthreads();
  return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

// Sum of `v` over aligned segments of `seg` consecutive threads (seg a power of two,
// 1 <= seg <= 256); every thread receives the sum of its own segment.  `lds` points to at
// least kWaves doubles of shared memory that no one else uses across the call.
// Contains barriers when seg > 64: every thread of the work-group must call it.
__device__ __forceinline__ double segment_sum(double v, int seg, double* lds) {
  const int lim = seg < kWave ? seg : kWave;
  for (int off = 1; off < lim; off <<= 1) v += shfl_xor_f64(v, off);
  if (seg > kWave) {
    const int wave = threadIdx.x / kWave;
    __syncthreads();
    if ((threadIdx.x % kWave) == 0) lds[wave] = v;
    __syncthreads();
    const int wps = seg / kWave;              // waves per segment: 2 or 4
    const int w0 = wave & ~(wps - 1);
    double t = lds[w0];
    for (int k = 1; k < wps; ++k) t += lds[w0 + k];
    v = t;
  }
  return v;
}

__device__ __forceinline__ uint32_t segment_sum_u32(uint32_t v, int seg, uint32_t* lds) {
  const int lim = seg < kWave ? seg : kWave;
  for (int off = 1; off < lim; off <<= 1) v += __shfl_xor(v, off, kWave);
  if (seg > kWave) {
    const int wave = threadIdx.x / kWave;
    __syncthreads();
    if ((threadIdx.x % kWave) == 0) lds[wave] = v;
    __syncthreads();
    const int wps = seg / kWave;
    const int w0 = wave & ~(wps - 1);
    uint32_t t = lds[w0];
    for (int k = 1; k < wps; ++k) t += lds[w0 + k];
    v = t;
  }
  return v;
}

// This thread's share of part[i0 .. i1): elements i0 + threadIdx.x + k*256, sixteen loads in
// flight at a time (a fixed order: the result does not depend on scheduling).  These sums run
// in a single work-group per bucket, so the number of dependent rounds of loads is their time.
constexpr int kPartialLoads = 16;
// For the kernels that call them: one or two waves per SIMD is all they ever run at, and saying so
// keeps the compiler from serialising the loads to save registers (it did: one load, one wait).
#define QA_FEW_WAVES __attribute__((amdgpu_waves_per_eu(1, 2)))
__device__ __forceinline__ double fold_partials(const double (&acc)[kPartialLoads]) {
  double r[kPartialLoads / 2];
#pragma unroll
  for (int u = 0; u < kPartialLoads / 2; ++u) r[u] = acc[2 * u] + acc[2 * u + 1];
#pragma unroll
  for (int w = kPartialLoads / 4; w >= 1; w /= 2)
#pragma unroll
    for (int u = 0; u < w; ++u) r[u] = r[2 * u] + r[2 * u + 1];
  return r[0];
}
template <typename T>
__device__ __forceinline__ double strided_partial_sum(const T* __restrict__ part, int64_t i0,
                                                      int64_t i1) {
  double acc[kPartialLoads];
#pragma unroll
  for (int u = 0; u < kPartialLoads; ++u) acc[u] = 0.0;
  int64_t i = i0 + threadIdx.x;
  for (; i + (kPartialLoads - 1) * kThreads < i1; i += kPartialLoads * kThreads) {
    T v[kPartialLoads];
#pragma unroll
    for (int u = 0; u < kPartialLoads; ++u) v[u] = part[i + u * kThreads];
#pragma unroll
    for (int u = 0; u < kPartialLoads; ++u) acc[u] += (double)v[u];
  }
  for (; i < i1; i += kThreads) acc[0] += (double)part[i];
  return fold_partials(acc);
}
// The same for a pair of arrays (sums and counts of the same tiles), their loads interleaved.
template <typename T, typename U>
__device__ __forceinline__ void strided_partial_sums(const T* __restrict__ pa, const U* __restrict__ pb,
                                                     int64_t i0, int64_t i1, double* sa, double* sb) {
  double acc[kPartialLoads], bcc[kPartialLoads];
#pragma unroll
  for (int u = 0; u < kPartialLoads; ++u) { acc[u] = 0.0; bcc[u] = 0.0; }
  int64_t i = i0 + threadIdx.x;
  for (; i + (kPartialLoads - 1) * kThreads < i1; i += kPartialLoads * kThreads) {
    T v[kPartialLoads];
    U w[kPartialLoads];
#pragma unroll
    for (int u = 0; u < kPartialLoads; ++u) { v[u] = pa[i + u * kThreads]; w[u] = pb[i + u * kThreads]; }
#pragma unroll
    for (int u = 0; u < kPartialLoads; ++u) { acc[u] += (double)v[u]; bcc[u] += (double)w[u]; }
  }
  for (; i < i1; i += kThreads) { acc[0] += (double)pa[i]; bcc[0] += (double)pb[i]; }
  *sa = fold_partials(acc);
  *sb = fold_partials(bcc);
}

// Threshold and scale from the binary64 sums, rounded once (Sections 3.4-3.5).
__device__ __forceinline__ float threshold_from_sum(double S1, float thr_coef, int64_t n) {
  return (float)(((double)thr_coef * S1) / (double)n);
}
__device__ __forceinline__ float scale_from_sum(double S2, uint64_t cnt) {
  return cnt ? (float)(S2 / (double)cnt) : 0.0f;
}

// ---- code words from compare masks ----------------------------------------------------------------
//
// The kernels that write codes are bound by vector instructions as much as by memory.  A field costs two: its bits
// are shifted into the word from below, the last component first, the sign by v_alignbit and the kept bit as the
// carry of word + word + carry.  Built from selects it was four.

// word << 8 | the fields of four components, sign and kept bit; the signs of what is not kept go with clear_signs().
// A mask that a vector compare has just written may be read as a carry two wait states later at the earliest, and
// what the compiler puts in front of the statement is not known: hence the s_nop.
__device__ __forceinline__ uint32_t push_codes(uint32_t word, const float (&v)[4], const uint64_t (&kept)[4]) {
  uint64_t carry_out;
  asm("s_nop 1\n\t"
      "v_alignbit_b32 %0, %0, %5, 31\n\tv_addc_co_u32_e64 %0, %1, %0, %0, %9\n\t"
      "v_alignbit_b32 %0, %0, %4, 31\n\tv_addc_co_u32_e64 %0, %1, %0, %0, %8\n\t"
      "v_alignbit_b32 %0, %0, %3, 31\n\tv_addc_co_u32_e64 %0, %1, %0, %0, %7\n\t"
      "v_alignbit_b32 %0, %0, %2, 31\n\tv_addc_co_u32_e64 %0, %1, %0, %0, %6"
      : "+&v"(word), "=&s"(carry_out)
      : "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "s"(kept[0]), "s"(kept[1]), "s"(kept[2]), "s"(kept[3]));
  return word;
}
__device__ __forceinline__ uint32_t clear_signs(uint32_t word) {
  const uint32_t kept = word & 0x55555555u;
  return word & (kept | kept << 1);
}
// Byte j of lane i's word (i, j in 0 .. 3 within each quad) to byte i of lane j's.
__device__ __forceinline__ uint32_t quad_transpose(uint32_t word) {
  const uint32_t t = threadIdx.x;
  const uint32_t beside = (uint32_t)dpp_i32<kDppQuadXor1>((int)word);
  const uint32_t pairs = __builtin_amdgcn_perm(beside, word, t & 1u ? 0x03070105u : 0x06020400u);
  const uint32_t across = (uint32_t)dpp_i32<kDppQuadXor2>((int)pairs);
  return __builtin_amdgcn_perm(across, pairs, t & 2u ? 0x03020706u : 0x05040100u);
}
// Code word j * 64 + thread / 4 of a tile in lane j of each quad, from v[j][e], component e of the thread's float4
// group j * 256 + thread, and the lanes that keep it.
__device__ __forceinline__ uint32_t code_word(const float (&v)[4][4], const uint64_t (&kept)[4][4]) {
  uint32_t word = 0;
#pragma unroll
  for (int j = 3; j >= 0; --j) word = push_codes(word, v[j], kept[j]);
  return quad_transpose(clear_signs(word));
}
// A store that goes through the second-level cache at once instead of leaving its line there until it is evicted.
// For words written beside a stream of reads many times as long, which late evictions disturb (2^30 components read
// and 1/16 of that written by a kernel that does nothing else: 713 us, with this 677, without any writes 597).  Not
// where a barrier follows in a loop (it waits for memory then), and not for read-modify-write streams, which
// write as much as they read (the fused step's accesses 813 -> 838 us at 2^28 coordinates, 8 workers).  The indicator's
// words lose by it too (8 x 10^8: 823 -> 847 us), the exact threshold's one pass does not change.
__device__ __forceinline__ void store_through(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// s += x in the lanes of `lanes` alone: one vector instruction where a selected addend takes two more.
__device__ __forceinline__ void add_in_lanes(double& s, double x, uint64_t lanes) {
  uint64_t all;
  asm("s_and_saveexec_b64 %1, %3\n\tv_add_f64 %0, %0, %2\n\ts_mov_b64 exec, %1"
      : "+v"(s), "=&s"(all) : "v"(x), "s"(lanes) : "scc");
}

// Ternary code as the 2-bit field 00 / 01 / 11; NaN compares false on both sides -> 00.
__device__ __forceinline__ uint32_t ternary_field(float v, float Delta) {
  return v > Delta ? 1u : (v < -Delta ? 3u : 0u);
}
// code_word() by the two comparisons as they are defined, which differ from |v| > Delta for thresholds below 0.
__device__ __forceinline__ uint32_t code_word_compared(const float (&v)[4][4], const float (&Delta)[4]) {
  uint32_t word = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) word |= ternary_field(v[i / 4][i % 4], Delta[i / 4]) << (2 * i);
  return quad_transpose(word);
}

#endif  // __HIPCC__

}  // namespace qa
