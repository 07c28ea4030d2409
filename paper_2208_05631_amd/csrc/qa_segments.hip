// Tensor-list quantizer: the threshold quantizer of Sections 3.4-3.5 applied to each tensor of a
// flat vector on its own, all tensors and all workers in one launch per pass.
//
// Work-group = one piece (tile x tensor intersection) of one worker.  Four passes, as for a
// bucket larger than a tile: piece sums of |v| -> threshold per tensor -> codes and piece
// (sum, count) of the kept magnitudes -> scale per tensor.  Partial results are combined in a
// fixed order in binary64, so the result does not depend on scheduling.  Large lists read the long
// tensors' gradients once (see the passes around seg_bracketed_kernel).
#include <vector>

#include "qa_segments.h"
#include "qa_settle.h"

namespace qa {

struct SegQuantArgs {
  const float* g;
  int64_t g_stride;
  int64_t d;
  uint32_t* codes;
  int64_t code_stride;
  float* scales;
  float* thresholds;        // user array, may be null
  int64_t scale_stride;
  float thr_coef;
  double* part_sum;         // [M][n_pieces]
  uint32_t* part_cnt;       // [M][n_pieces]
  float* thr_ws;            // [M][n_seg]
  SegTable seg;
  // one-read form, null without it
  double* kept_sum;         // [M][n_pieces]; before that the samples
  float2* band;             // [M][n_seg]
  uint16_t* open;           // [M][n_pieces][kWaves][kOpenSlots]
};

// The thread's 4 float4 groups f = j*256 + t of the piece's tile; elements outside [lo, hi)
// read as +0 (lo is a multiple of 16, so a group never straddles it).
__device__ __forceinline__ void load_piece_values(const float* __restrict__ g, const Piece& pc,
                                                  float v[4][4]) {
  const int64_t base = pc.tile * kTile;
  // streaming: the passes over the gradients read an element once each, a whole pass apart
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  if (pc.hi - pc.lo == kTile) {                          // uniform: nothing to test per lane
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const floatx4 q = __builtin_nontemporal_load(
          reinterpret_cast<const floatx4*>(g + base + (int64_t)(j * kThreads + (int)threadIdx.x) * 4));
      v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t i = base + (int64_t)(j * kThreads + (int)threadIdx.x) * 4;
    if (i >= pc.lo && i + 3 < pc.hi) {
      const floatx4 q = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(g + i));
      v[j][0] = q.x; v[j][1] = q.y; v[j][2] = q.z; v[j][3] = q.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[j][e] = (i + e >= pc.lo && i + e < pc.hi) ? g[i + e] : 0.0f;
    }
  }
}

__global__ __launch_bounds__(kThreads) void seg_abs_partial_kernel(SegQuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t p = blockIdx.x;
  const int m = blockIdx.y;
  const Piece pc = load_piece(a.seg, p, a.d);
  float v[4][4];
  load_piece_values(a.g + (int64_t)m * a.g_stride, pc, v);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) s += (double)fabsf(v[j][e]);
  s = block_sum_f64(s, lds_d);
  if (threadIdx.x == 0) a.part_sum[(int64_t)m * a.seg.n_pieces + p] = s;
}

// Pieces of tensor s, clamped to the table.
__device__ __forceinline__ void piece_range(const SegTable& T, int64_t s, int64_t* p0, int64_t* p1) {
  int64_t a = T.piece_first[s], b = T.piece_first[s + 1];
  a = a < 0 ? 0 : (a > T.n_pieces ? T.n_pieces : a);
  b = b < a ? a : (b > T.n_pieces ? T.n_pieces : b);
  *p0 = a; *p1 = b;
}

__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void seg_threshold_finalize_kernel(SegQuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t s = blockIdx.x;
  const int m = blockIdx.y;
  int64_t p0, p1;
  piece_range(a.seg, s, &p0, &p1);
  double sum = strided_partial_sum(a.part_sum + (int64_t)m * a.seg.n_pieces, p0, p1);
  sum = segment_sum(sum, kThreads, lds_d);
  if (threadIdx.x == 0) {
    const int64_t n = a.seg.length[s];
    const float Delta = n > 0 ? threshold_from_sum(sum, a.thr_coef, n) : 0.0f;
    a.thr_ws[(int64_t)m * a.seg.n_seg + s] = Delta;
    if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + s] = Delta;
  }
}

// Codes of piece p of worker m for threshold D, and what they keep to the piece's slots.
__device__ __forceinline__ void code_piece(const SegQuantArgs& a, const Piece& pc, int64_t p, int m, float D,
                                           double* lds_d, uint32_t* lds_u) {
  const int t = threadIdx.x;
  float v[4][4];
  load_piece_values(a.g + (int64_t)m * a.g_stride, pc, v);
  double s = 0.0;
  uint32_t c = 0;
  uint32_t mine = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint32_t b = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float av = fabsf(v[j][e]);
      if (av > D) { s += (double)av; ++c; }
      b |= ternary_field(v[j][e], D) << (2 * e);
    }
    // the four lanes of a quad hold the four bytes of code word j*64 + t/4 of the tile
    uint32_t w = b << (8 * (t & 3));
    w |= (uint32_t)dpp_i32<kDppQuadXor1>((int)w);
    w |= (uint32_t)dpp_i32<kDppQuadXor2>((int)w);
    if ((t & 3) == j) mine = w;
  }
  s = wave_sum_f64(s);
  c = wave_sum_u32(c);
  if ((t % kWave) == 0) { lds_d[t / kWave] = s; lds_u[t / kWave] = c; }
  __syncthreads();
  // words of the tile that hold coordinates of this piece
  const int64_t base = pc.tile * kTile;
  const int wlo = (int)((pc.lo - base) >> 4), whi = (int)((pc.hi - base + 15) >> 4);
  const int wl = (t & 3) * 64 + (t >> 2);
  if (wl >= wlo && wl < whi)
    a.codes[(int64_t)m * a.code_stride + pc.tile * kTileWords + wl] = mine;
  if (t == 0) {
    a.part_sum[(int64_t)m * a.seg.n_pieces + p] = (lds_d[0] + lds_d[1]) + (lds_d[2] + lds_d[3]);
    a.part_cnt[(int64_t)m * a.seg.n_pieces + p] = lds_u[0] + lds_u[1] + lds_u[2] + lds_u[3];
  }
}

__global__ __launch_bounds__(kThreads) void seg_codes_partial_kernel(SegQuantArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ uint32_t lds_u[kWaves];
  const Piece pc = load_piece(a.seg, blockIdx.x, a.d);
  code_piece(a, pc, blockIdx.x, blockIdx.y, a.thr_ws[(int64_t)blockIdx.y * a.seg.n_seg + pc.seg], lds_d, lds_u);
}

__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void seg_scale_finalize_kernel(SegQuantArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ double lds_c[kWaves];
  const int64_t s = blockIdx.x;
  const int m = blockIdx.y;
  int64_t p0, p1;
  piece_range(a.seg, s, &p0, &p1);
  // counts are integers < 2^53: exact in binary64
  double sum, cnt;
  strided_partial_sums(a.part_sum + (int64_t)m * a.seg.n_pieces, a.part_cnt + (int64_t)m * a.seg.n_pieces, p0, p1,
                       &sum, &cnt);
  sum = segment_sum(sum, kThreads, lds_d);
  cnt = segment_sum(cnt, kThreads, lds_c);
  if (threadIdx.x == 0)
    a.scales[(int64_t)m * a.scale_stride + s] = scale_from_sum(sum, (uint64_t)cnt);
}

// ---- long tensors in one read -------------------------------------------------------------------
//
// As for long buckets of a plain vector: 32 samples or more of a tensor of at least 128 pieces give a
// bracket around the tensor's threshold (four standard errors, at most 8 % to either side),
// the one pass writes final codes outside the bracket and the piece sums of |v| and lists the open float4 groups,
// and the settling pass looks these up once the threshold is known.  Of tensors
// without a bracket, or whose threshold falls outside it, it reads the gradient again.  32 samples hold the bracket of a
// Gaussian tensor to 0.8 %, of whose components the lists have room for all but a few in a hundred pieces; with 16 a
// fifth of the pieces would be read again, so shorter tensors keep both reads.
constexpr int kSegSampleEvery = 32;
constexpr int64_t kSegShortest = 128;
constexpr int64_t kSegLong = 1024;
constexpr double kSegWidestBand = 0.08;

// Every how many pieces (a power of two) a tensor of n pieces is sampled: 32 samples, of a long tensor more; 0: none.
__device__ __forceinline__ int64_t seg_sample_stride(int64_t n) {
  return n >= kSegLong ? 32 : n >= 512 ? 16 : n >= 256 ? 8 : n >= kSegShortest ? 4 : 0;
}

// A work-group looks through 32 pieces, a wave reads a sampled one; sample k of a tensor goes to slot k of the tensor's
// slots, as -1 if the piece is not a whole tile.
__global__ __launch_bounds__(kThreads) void seg_sample_kernel(SegQuantArgs a) {
  const int m = blockIdx.y, lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int64_t own = (int64_t)blockIdx.x * kSegSampleEvery + lane % kSegSampleEvery;
  bool sampled = false;
  int64_t slot = 0, tile = 0;
  if (own < a.seg.n_pieces) {
    const Piece pc = load_piece(a.seg, own, a.d);
    int64_t p0, p1;
    piece_range(a.seg, pc.seg, &p0, &p1);
    const int64_t stride = seg_sample_stride(p1 - p0);
    if (stride != 0 && own >= p0) {
      const int64_t k = (own - p0) / stride;
      sampled = (own - p0) % stride == k * 29 % stride && (k + 1) * stride <= p1 - p0;
      slot = (int64_t)m * a.seg.n_pieces + p0 + k;
      tile = pc.hi - pc.lo == kTile ? pc.tile : -1;
    }
  }
  int rank = 0;
  for (uint32_t left = (uint32_t)__ballot(sampled); left; left &= left - 1u, ++rank) {   // the same in every wave
    if (rank % kWaves != wave) continue;
    const int u = __ffs((int)left) - 1;
    const int64_t whole = __shfl(tile, u, kWave);
    double s = -1.0;
    if (whole >= 0) {
      typedef float floatx4 __attribute__((ext_vector_type(4)));
      const floatx4* g = reinterpret_cast<const floatx4*>(a.g + (int64_t)m * a.g_stride + whole * kTile) + lane;
      floatx4 q[kTile / 4 / kWave];
#pragma unroll
      for (int i = 0; i < kTile / 4 / kWave; ++i) q[i] = __builtin_nontemporal_load(g + i * kWave);
      s = 0.0;
#pragma unroll
      for (int i = 0; i < kTile / 4 / kWave; ++i)
        s += ((double)fabsf(q[i].x) + (double)fabsf(q[i].y)) + ((double)fabsf(q[i].z) + (double)fabsf(q[i].w));
      s = wave_sum_f64(s);
    }
    if (lane == u) a.kept_sum[slot] = s;
  }
}

__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void seg_band_kernel(SegQuantArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t s = blockIdx.x;
  const int m = blockIdx.y;
  int64_t p0, p1;
  piece_range(a.seg, s, &p0, &p1);
  const int64_t stride = seg_sample_stride(p1 - p0), samples = stride != 0 ? (p1 - p0) / stride : 0;
  const double* part = a.kept_sum + (int64_t)m * a.seg.n_pieces + p0;
  double sum = 0.0, diff = 0.0, n = 0.0, nd = 0.0;
  for (int64_t i = threadIdx.x; i < samples; i += kThreads) {
    const double v = part[i], w = i + 1 < samples ? part[i + 1] : -1.0;
    if (v >= 0.0 || v != v) { sum += v; n += 1.0; }
    if (v >= 0.0 && w >= 0.0) { diff += (w - v) * (w - v); nd += 1.0; }
  }
  sum = segment_sum(sum, kThreads, lds_d);
  diff = segment_sum(diff, kThreads, lds_d);
  n = segment_sum(n, kThreads, lds_d);
  nd = segment_sum(nd, kThreads, lds_d);
  if (threadIdx.x == 0) {
    float2 band = make_float2(-1.0f, -1.0f);
    if (n >= 12.0 && nd >= 8.0) {
      const double mean = sum / n, rel = 4.0 * sqrt(diff / (2.0 * nd) / n) / mean + 1e-6;
      const double mid = (double)a.thr_coef * mean / (double)kTile;
      if (mean > 0.0 && rel < kSegWidestBand && mid < 1e38)
        band = make_float2((float)(mid * (1.0 - rel)), (float)(mid * (1.0 + rel)));
    }
    a.band[(int64_t)m * a.seg.n_seg + s] = band;
  }
}

__global__ __launch_bounds__(kThreads) void seg_bracketed_kernel(SegQuantArgs a) {
  __shared__ double lds_s1[kWaves];
  __shared__ double lds_s2[kWaves];
  __shared__ uint32_t lds_c[kWaves];
  const int t = threadIdx.x;
  const int64_t p = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t at = (int64_t)m * a.seg.n_pieces + p;
  const Piece pc = load_piece(a.seg, p, a.d);
  const float2 band = a.band[(int64_t)m * a.seg.n_seg + pc.seg];
  float v[4][4];
  load_piece_values(a.g + (int64_t)m * a.g_stride, pc, v);
  double s1 = 0.0, s2 = 0.0;
  if (!(band.x >= 0.0f)) {                               // uniform; the settling pass codes the piece
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) s1 += (double)fabsf(v[j][e]);
    const double S1 = block_sum_f64(s1, lds_s1);
    if (t == 0) a.part_sum[at] = S1;
    return;
  }
  // in the order of seg_abs_partial_kernel: the threshold is the same number in both forms
  uint32_t wave_cnt = 0;
  uint64_t open[4][4];
  const uint32_t word = code_outside(v, band, s1, s2, wave_cnt, open);
  const int64_t base = pc.tile * kTile;
  const int wlo = (int)((pc.lo - base) >> 4), whi = (int)((pc.hi - base + 15) >> 4);
  const int wl = (t & 3) * 64 + (t >> 2);
  if (wl >= wlo && wl < whi) store_through(a.codes + (int64_t)m * a.code_stride + pc.tile * kTileWords + wl, word);
  wave_cnt |= list_open(open, a.open + (at * kWaves + t / kWave) * kOpenSlots) << 16;
  const double S1 = wave_sum_f64(s1), S2 = wave_sum_f64(s2);
  if (t % kWave == 0) { lds_s1[t / kWave] = S1; lds_s2[t / kWave] = S2; lds_c[t / kWave] = wave_cnt; }
  __syncthreads();
  if (t == 0) {
    a.part_sum[at] = (lds_s1[0] + lds_s1[1]) + (lds_s1[2] + lds_s1[3]);
    a.kept_sum[at] = (lds_s2[0] + lds_s2[1]) + (lds_s2[2] + lds_s2[3]);
    a.part_cnt[at] = tile_counts(lds_c);
  }
}

// Eight consecutive pieces per work-group, 32 lanes per listed piece; the others are coded one by one.  What a piece
// keeps goes to its slots of part_sum / part_cnt.
__global__ __launch_bounds__(kThreads) void seg_settle_kernel(SegQuantArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ uint32_t lds_u[kWaves];
  __shared__ uint32_t lds_again[kSettleTiles];
  const int t = threadIdx.x, lane = t & 31;
  const int m = blockIdx.y;
  const int64_t piece0 = (int64_t)blockIdx.x * kSettleTiles;
  const int64_t p = piece0 + t / 32, row = (int64_t)m * a.seg.n_pieces, at = row + p;
  bool again = false, listed = false;
  double s = 0.0, kept = 0.0;
  uint32_t c = 0;
  if (p < a.seg.n_pieces) {
    const Piece pc = load_piece(a.seg, p, a.d);
    const float D = a.thr_ws[(int64_t)m * a.seg.n_seg + pc.seg];
    const float2 band = a.band[(int64_t)m * a.seg.n_seg + pc.seg];
    const uint32_t counts = a.part_cnt[at];
    kept = a.kept_sum[at];
    again = !bracket_held(band, D) || too_many_open(counts);   // (without a bracket the piece has no counts)
    listed = !again;
    if (listed) {
      const uint32_t list = lane >> 3, n = (counts >> (16 + 4 * list)) & 15u;
      settle_listed<2>(a.open + (at * kWaves + list) * kOpenSlots, (uint32_t)lane & 7u, 8u, n,
                       a.g + (int64_t)m * a.g_stride + pc.tile * kTile, pc.hi - pc.tile * kTile, band, D,
                       a.codes + (int64_t)m * a.code_stride + pc.tile * kTileWords, s, c);
      if (lane == 0) c += counts & 0xFFFFu;
    }
  }
  s += dpp_f64<kDppQuadXor1>(s);          c += (uint32_t)dpp_i32<kDppQuadXor1>((int)c);
  s += dpp_f64<kDppQuadXor2>(s);          c += (uint32_t)dpp_i32<kDppQuadXor2>((int)c);
  s += dpp_f64<kDppRowHalfMirror>(s);     c += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)c);
  s += dpp_f64<kDppRowMirror>(s);         c += (uint32_t)dpp_i32<kDppRowMirror>((int)c);
  s += __shfl_xor(s, 16, kWave);          c += (uint32_t)__shfl_xor((int)c, 16, kWave);
  if (lane == 0) {
    lds_again[t / 32] = again ? 1u : 0u;
    if (listed) { a.part_sum[at] = s + kept; a.part_cnt[at] = c; }
  }
  __syncthreads();
  for (int u = 0; u < kSettleTiles; ++u) {
    if (lds_again[u] == 0u) continue;                    // uniform
    const Piece pc = load_piece(a.seg, piece0 + u, a.d);
    code_piece(a, pc, piece0 + u, m, a.thr_ws[(int64_t)m * a.seg.n_seg + pc.seg], lds_d, lds_u);
    __syncthreads();                                     // LDS is free again
  }
}

static inline size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

size_t quantize_segments_workspace_bytes(const qa_segment_plan* P, int M) {
  const size_t np = (size_t)(P->n_pieces > 0 ? P->n_pieces : 1);
  return align256((size_t)M * np * sizeof(double)) + align256((size_t)M * np * sizeof(uint32_t)) +
         align256((size_t)M * (size_t)P->n_seg * sizeof(float));
}

// What the one-read form needs on top of it, 0 where it is not taken.  The length of the longest tensor is
// known on the device only, so the form has to pay where there are long tensors and cost little where
// there are none: from 2^27 components on and with 128 pieces per tensor on average.  At that limit
// (32768 pieces in all workers together), two reads -> one, us: 1 worker x 8 tensors of 4096 pieces 193 -> 143,
// 8 x 4 of 1024 193 -> 152; 32 tensors, 58.4 M parameters, most of them in two tensors, 3 workers 250 -> 191,
// 8 workers 641 -> 420.  With the step, one read for tensors of 1024 pieces on -> of 128 on: 2 x 64 of 500 832 -> 690,
// 1 x 64 of 1000 1279 -> 1128, 8 x 60 of 130 510 -> 398, 4 x 100 of 300 1145 -> 928; where no bracket holds (one component
// in 1000 not 0, Cauchy components) the samples are read for nothing: 820 -> 850, 1255 -> 1275, 500 -> 550, 1135 -> 1195.
// Below the average, where the bracket's work-group per tensor counts (quantizer): 8 x 64 of 64 190 -> 203, 4 x 2000 of 5
// 271 -> 311, 40000 of one or two 551 -> 755.
constexpr int64_t kSegOneReadPieces = 32768, kSegOneReadMean = 128;
size_t segments_one_read_bytes(const qa_segment_plan* P, int M) {
  if (P->n_pieces < kSegLong || P->n_pieces * M < kSegOneReadPieces || P->n_pieces < kSegOneReadMean * P->n_seg) return 0;
  return align256((size_t)M * (size_t)P->n_pieces * sizeof(double)) + align256((size_t)M * (size_t)P->n_seg * sizeof(float2)) +
         (size_t)M * (size_t)P->n_pieces * kWaves * kOpenSlots * sizeof(uint16_t);
}

static SegQuantArgs seg_args(const qa_layout* L, const qa_segment_plan* P, float* scales, float* thresholds, void* ws) {
  SegQuantArgs a{};
  a.d = L->d;
  a.scales = scales; a.thresholds = thresholds; a.scale_stride = L->scale_stride;
  a.thr_coef = L->thr_coef;
  a.seg = seg_table_of(P);
  const size_t np = (size_t)(P->n_pieces > 0 ? P->n_pieces : 1);
  char* p = static_cast<char*>(ws);
  a.part_sum = reinterpret_cast<double*>(p);    p += align256((size_t)L->M * np * sizeof(double));
  a.part_cnt = reinterpret_cast<uint32_t*>(p);  p += align256((size_t)L->M * np * sizeof(uint32_t));
  a.thr_ws = reinterpret_cast<float*>(p);
  return a;
}

// For a producer that forms the quantizer's input piece by piece and leaves its sums itself: where they
// go, and the finalize kernels alone (which = 0: thresholds, 1: scales).
void segments_workspace_parts(const qa_layout* L, const qa_segment_plan* P, void* ws, double** part_sum,
                              uint32_t** part_cnt, float** thr) {
  const SegQuantArgs a = seg_args(L, P, nullptr, nullptr, ws);
  *part_sum = a.part_sum; *part_cnt = a.part_cnt; *thr = a.thr_ws;
}
void segments_finalize_launch(const qa_layout* L, const qa_segment_plan* P, int which, float* scales, void* ws,
                              hipStream_t stream) {
  const SegQuantArgs a = seg_args(L, P, scales, nullptr, ws);
  const dim3 block(kThreads), grid_s((unsigned)P->n_seg, (unsigned)L->M);
  if (which == 0) hipLaunchKernelGGL(seg_threshold_finalize_kernel, grid_s, block, 0, stream, a);
  else hipLaunchKernelGGL(seg_scale_finalize_kernel, grid_s, block, 0, stream, a);
}

int quantize_segments_launch(const qa_layout* L, const qa_segment_plan* P, const float* g,
                             int64_t g_stride, uint32_t* codes, float* scales, float* thresholds,
                             void* ws, size_t ws_bytes, hipStream_t stream) {
  if (!ws || ws_bytes < quantize_segments_workspace_bytes(P, L->M)) return QA_ERR_WORKSPACE;
  if (!aligned(ws, 256)) return QA_ERR_ALIGNMENT;
  SegQuantArgs a = seg_args(L, P, scales, thresholds, ws);
  a.g = g; a.g_stride = g_stride;
  a.codes = codes; a.code_stride = L->code_stride;
  const dim3 block(kThreads);
  const dim3 grid_p((unsigned)P->n_pieces, (unsigned)L->M), grid_s((unsigned)P->n_seg, (unsigned)L->M);
  const size_t base = quantize_segments_workspace_bytes(P, L->M), more = segments_one_read_bytes(P, L->M);
  if (more != 0 && ws_bytes >= base + more) {
    char* p = static_cast<char*>(ws) + base;
    a.kept_sum = reinterpret_cast<double*>(p);
    p += align256((size_t)L->M * (size_t)P->n_pieces * sizeof(double));
    a.band = reinterpret_cast<float2*>(p);
    a.open = reinterpret_cast<uint16_t*>(p + align256((size_t)L->M * (size_t)P->n_seg * sizeof(float2)));
    const dim3 samples((unsigned)((P->n_pieces + kSegSampleEvery - 1) / kSegSampleEvery), (unsigned)L->M);
    const dim3 settle((unsigned)((P->n_pieces + kSettleTiles - 1) / kSettleTiles), (unsigned)L->M);
    hipLaunchKernelGGL(seg_sample_kernel, samples, block, 0, stream, a);
    hipLaunchKernelGGL(seg_band_kernel, grid_s, block, 0, stream, a);
    hipLaunchKernelGGL(seg_bracketed_kernel, grid_p, block, 0, stream, a);
    hipLaunchKernelGGL(seg_threshold_finalize_kernel, grid_s, block, 0, stream, a);
    hipLaunchKernelGGL(seg_settle_kernel, settle, block, 0, stream, a);
    hipLaunchKernelGGL(seg_scale_finalize_kernel, grid_s, block, 0, stream, a);
    return launch_status();
  }
  if (P->n_pieces > 0) hipLaunchKernelGGL(seg_abs_partial_kernel, grid_p, block, 0, stream, a);
  hipLaunchKernelGGL(seg_threshold_finalize_kernel, grid_s, block, 0, stream, a);
  if (P->n_pieces > 0) hipLaunchKernelGGL(seg_codes_partial_kernel, grid_p, block, 0, stream, a);
  hipLaunchKernelGGL(seg_scale_finalize_kernel, grid_s, block, 0, stream, a);
  return launch_status();
}

}  // namespace qa

extern "C" size_t qa_segment_plan_bytes(int64_t d, int64_t n_seg) {
  using namespace qa;
  if (d < 1 || d >= (int64_t(1) << 40) || n_seg < 1 || n_seg > 0x7fffffffLL) return 0;
  const int64_t np_max = tiles_of(d) + n_seg;
  return (size_t)(kSegHeader + 2 * n_seg + (n_seg + 1) + 2 * np_max) * sizeof(int64_t);
}

// Validates the tensor list and writes the table (layout in qa_segments.h) into host memory.
static int build_table(int64_t d, int64_t n_seg, const int64_t* begin, const int64_t* length,
                       std::vector<int64_t>& h, int64_t* n_pieces_out) {
  using namespace qa;
  if (!begin || !length) return QA_ERR_INVALID_ARG;
  if (qa_segment_plan_bytes(d, n_seg) == 0) return QA_ERR_INVALID_ARG;
  int64_t end_prev = 0, n_pieces = 0;
  for (int64_t s = 0; s < n_seg; ++s) {
    if (begin[s] < end_prev || (begin[s] & 15) != 0 || length[s] < 0) return QA_ERR_INVALID_ARG;
    if (begin[s] > d || length[s] > d - begin[s]) return QA_ERR_INVALID_ARG;
    end_prev = begin[s] + length[s];
    if (length[s] > 0) n_pieces += (end_prev - 1) / kTile - begin[s] / kTile + 1;
  }
  if (n_pieces > 0x7fffffffLL) return QA_ERR_INVALID_ARG;
  h.assign((size_t)(kSegHeader + 2 * n_seg + (n_seg + 1) + 2 * n_pieces), 0);
  h[0] = kSegMagic; h[1] = d; h[2] = n_seg; h[3] = n_pieces;
  int64_t* hb = h.data() + kSegHeader;
  int64_t* hl = hb + n_seg;
  int64_t* hf = hl + n_seg;
  int64_t* ht = hf + n_seg + 1;
  int64_t* hs = ht + n_pieces;
  int64_t p = 0;
  for (int64_t s = 0; s < n_seg; ++s) {
    hb[s] = begin[s]; hl[s] = length[s]; hf[s] = p;
    if (length[s] > 0)
      for (int64_t T = begin[s] / kTile; T <= (begin[s] + length[s] - 1) / kTile; ++T) { ht[p] = T; hs[p] = s; ++p; }
  }
  hf[n_seg] = p;
  *n_pieces_out = n_pieces;
  return QA_OK;
}

extern "C" int qa_segment_plan_host(int64_t d, int64_t n_seg, const int64_t* begin,
                                    const int64_t* length, int64_t* table_host, size_t table_bytes,
                                    int64_t* n_pieces_out) {
  if (!n_pieces_out) return QA_ERR_INVALID_ARG;
  std::vector<int64_t> h;
  int rc = build_table(d, n_seg, begin, length, h, n_pieces_out);
  if (rc != QA_OK) return rc;
  if (table_host) {
    if (table_bytes < h.size() * sizeof(int64_t)) return QA_ERR_WORKSPACE;
    for (size_t i = 0; i < h.size(); ++i) table_host[i] = h[i];
  }
  return QA_OK;
}

extern "C" int qa_segment_plan_init(int64_t d, int64_t n_seg, const int64_t* begin,
                                    const int64_t* length, void* table, size_t table_bytes,
                                    qa_segment_plan* plan_out, void* stream) {
  using namespace qa;
  if (!begin || !length || !table || !plan_out) return QA_ERR_INVALID_ARG;
  if (qa_segment_plan_bytes(d, n_seg) == 0) return QA_ERR_INVALID_ARG;
  if (!aligned(table, 8)) return QA_ERR_ALIGNMENT;
  std::vector<int64_t> h;
  int64_t n_pieces = 0;
  int rc = build_table(d, n_seg, begin, length, h, &n_pieces);
  if (rc != QA_OK) return rc;
  if (table_bytes < h.size() * sizeof(int64_t)) return QA_ERR_WORKSPACE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (hipMemcpyAsync(table, h.data(), h.size() * sizeof(int64_t), hipMemcpyHostToDevice, st) != hipSuccess)
    return QA_ERR_LAUNCH;
  if (hipStreamSynchronize(st) != hipSuccess) return QA_ERR_LAUNCH;
  plan_out->d = d; plan_out->n_seg = n_seg; plan_out->n_pieces = n_pieces; plan_out->table = table;
  return QA_OK;
}

extern "C" int qa_quantize_pack_segments(const qa_layout* layout, const qa_segment_plan* plan,
                                         const float* g, int64_t g_stride, uint32_t* codes,
                                         float* scales, float* thresholds, void* ws,
                                         size_t ws_bytes, void* stream) {
  using namespace qa;
  int rc = check_layout(layout);
  if (rc != QA_OK) return rc;
  rc = check_plan(plan, layout);
  if (rc != QA_OK) return rc;
  if (!g || !codes || !scales) return QA_ERR_INVALID_ARG;
  if (g_stride < layout->d || (g_stride & 3) != 0) return QA_ERR_INVALID_ARG;
  if (!aligned(g, 16) || !aligned(codes, 4) || !aligned(scales, 4) || !aligned(thresholds, 4))
    return QA_ERR_ALIGNMENT;
  return quantize_segments_launch(layout, plan, g, g_stride, codes, scales, thresholds, ws, ws_bytes,
                                  static_cast<hipStream_t>(stream));
}
