// Minibatch gradient of the logistic loss for one worker (stochastic gradient of Section 3.1
// for the L1-regularised logistic regression of Section 5.1, arXiv 2208.05631), dense rows or
// CSR rows, for gfx950.
//
//   margins  : p_b = a_{r_b}.x in binary64 (work-group per row for dense, wave per row for CSR),
//              then coef_b = -y/(1+exp(y p_b))/B and the row's loss, in binary64.
//   gradient : dense -- one thread per 4 columns walks the batch (or a quarter of it), binary64
//                       accumulators;
//              CSR   -- the batch's entries are sorted into ranges of columns while the margins are
//                       formed, and a work-group per range adds them up in LDS and writes its part
//                       of g; vectors of more than 2^22 columns, and batches of too many rows for
//                       the workspace, take hardware binary64 atomic adds into a d-long accumulator
//                       that is cleared only at the batch's columns, then rounded into the
//                       zero-filled g.
//   Every product coef*a is exact in binary64, so only the order of the binary64 additions can
//   differ from a sequential evaluation.
#include "qa_common.h"

namespace qa {

constexpr int kMaxBatch = 65536;

// Dense rows: up to this many columns a wave takes a row, beyond it a work-group (4 workers x 64 rows of
// 1000 columns, both kernels: 6.9 us with a work-group per row, 7.7 with a wave; 16 x 384 rows of
// 64 columns: 19.3 and 10.8).
constexpr int kShortRow = 512;
// Column sums take the 16-way split of the batch below this many work-groups of the 4-way split (the chip has
// 256 compute units) if the batch has rows for all sixteen parts: 8 x 256 rows of 4000 columns (128
// work-groups) 16.6 us against 19.0; 2 x 256 rows of 30000 (236) 27.3 against 25.9.
constexpr int kFewGroups = 192;

static constexpr size_t align256(size_t v) { return (v + 255) & ~size_t(255); }
static constexpr size_t workspace_of(int64_t d, bool csr) {
  return align256((size_t)kMaxBatch * sizeof(float)) + align256((size_t)kMaxBatch * sizeof(double)) +
         (csr ? align256((size_t)d * sizeof(double)) : 0);
}

struct GradArgs {
  const float* A;            // dense matrix or CSR values
  const int64_t* indptr;
  const int32_t* indices;
  int64_t n_rows, d;
  const float* y;
  const int32_t* rows;
  int B;
  const float* x;
  float* g;
  float* loss_out;
  float* coef;               // [B]   workspace
  double* loss_part;         // [B]   workspace
  double* acc;               // [d]   workspace (CSR)
  // batched calls: worker m = blockIdx.y uses rows + m*B, g + m*g_stride, loss_out + m and the
  // m-th slice of each workspace array
  int64_t g_stride;
  int64_t ws_stride_bytes;
};

// View of the arguments for the worker selected by blockIdx.y.
__device__ __forceinline__ GradArgs for_worker(GradArgs a) {
  const int64_t m = blockIdx.y;
  a.rows += m * a.B;
  a.g += m * a.g_stride;
  if (a.loss_out) a.loss_out += m;
  a.coef = reinterpret_cast<float*>(reinterpret_cast<char*>(a.coef) + m * a.ws_stride_bytes);
  a.loss_part = reinterpret_cast<double*>(reinterpret_cast<char*>(a.loss_part) + m * a.ws_stride_bytes);
  a.acc = reinterpret_cast<double*>(reinterpret_cast<char*>(a.acc) + m * a.ws_stride_bytes);
  return a;
}

// Four consecutive floats at any address that is a multiple of 4: the memory system takes a 16-byte
// load on a 4-byte boundary (rows of an odd length start on those).
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef floatx4 floatx4_any __attribute__((aligned(4)));
__device__ __forceinline__ floatx4 load4(const float* p) { return *reinterpret_cast<const floatx4_any*>(p); }
// The same of a batch's rows.  The column sums read the margins' rows again and a later batch draws some of them again, so
// rows are streamed only where the cache would not hold them anyway: batches of more than 2^27 components (512 MB, twice
// the last-level cache).  Plain / streamed, us, other rows in each call and the same ones: 8 x 128 rows of 100003 columns 156
// and 152 / 155 153, 8 x 256 of 30001 94 82 / 93 92, 4 x 8 of 2^20 217 156 / 224 224, 4 x 32 of 2^20 (the line) 292 288 / 285 288,
// 4 x 64 of 2^20 427 421 / 403 402, 4 x 256 of 2^20 1525 1529 / 1445 1456, 8 x 256 of 300001 877 876 / 885 885.
constexpr int64_t kStreamedBatch = int64_t(1) << 27;
template <bool STREAM>
__device__ __forceinline__ floatx4 row_load4(const float* p) {
  return STREAM ? __builtin_nontemporal_load(reinterpret_cast<const floatx4_any*>(p)) : load4(p);
}

// coef and loss of one sample from its binary32 margin term p = a.x
__device__ __forceinline__ void logistic_terms(float p, float y, int B, float* coef, double* loss) {
  const double m = (double)y * (double)p;
  const double e = exp(-fabs(m));
  *loss = log1p(e) + (m < 0.0 ? -m : 0.0);
  const double sig = m >= 0.0 ? e / (1.0 + e) : 1.0 / (1.0 + e);
  *coef = (float)((-(double)y * sig) / (double)B);
}

// sum of the losses of a worker's batch rows -> loss_out, by one work-group
__device__ __forceinline__ void reduce_loss(const GradArgs& a, double* lds_d) {
  double s = 0.0;
  for (int b = threadIdx.x; b < a.B; b += kThreads) s += a.loss_part[b];
  s = segment_sum(s, kThreads, lds_d);
  if (threadIdx.x == 0) *a.loss_out = (float)(s / (double)a.B);
}

// LANES threads per batch row (the work-group, or a wave for short rows), which is read as 16-byte
// pieces with four loads in flight per thread.
template <int LANES, bool STREAM>
__global__ __launch_bounds__(kThreads) void dense_margin_kernel(GradArgs a_all) {
  static_assert(LANES == kThreads || LANES == kWave, "a work-group or a wave per row");
  const GradArgs a = for_worker(a_all);
  __shared__ double lds_d[kWaves];
  const int b = LANES == kWave ? (int)(blockIdx.x * kWaves + threadIdx.x / kWave) : (int)blockIdx.x;
  if (LANES == kWave && b >= a.B) return;
  const int lane = threadIdx.x % LANES;
  const int64_t r = a.rows[b];
  const bool ok = r >= 0 && r < a.n_rows;
  double s = 0.0;
  if (ok) {
    const float* row = a.A + r * a.d;
    const int64_t whole = a.d & ~int64_t(3);
    double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
    int64_t j = 4 * lane;
    for (; j + 4 * 3 * LANES < whole; j += 4 * 4 * LANES) {
      floatx4 v[4], w[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = row_load4<STREAM>(row + j + u * 4 * LANES);
#pragma unroll
      for (int u = 0; u < 4; ++u) w[u] = load4(a.x + j + u * 4 * LANES);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        s0 = fma((double)v[u].x, (double)w[u].x, s0);
        s1 = fma((double)v[u].y, (double)w[u].y, s1);
        s2 = fma((double)v[u].z, (double)w[u].z, s2);
        s3 = fma((double)v[u].w, (double)w[u].w, s3);
      }
    }
    for (; j < whole; j += 4 * LANES) {
      const floatx4 v = row_load4<STREAM>(row + j), w = load4(a.x + j);
      s0 = fma((double)v.x, (double)w.x, s0);
      s1 = fma((double)v.y, (double)w.y, s1);
      s2 = fma((double)v.z, (double)w.z, s2);
      s3 = fma((double)v.w, (double)w.w, s3);
    }
    if (whole + lane < a.d)
      s0 = fma((double)row[whole + lane], (double)a.x[whole + lane], s0);
    s = (s0 + s1) + (s2 + s3);
  }
  s = LANES == kWave ? wave_sum_f64(s) : segment_sum(s, kThreads, lds_d);
  if (lane == 0) {
    float c = 0.0f; double l = 0.0;
    if (ok) logistic_terms((float)s, a.y[r], a.B, &c, &l);
    a.coef[b] = c; a.loss_part[b] = l;
  }
}

// g_j = sum over the batch of coef_b * A[r_b][j]: thread per 4 columns, sixteen rows' loads in
// flight.  The batch's row ids and coefficients pass through LDS, 1024 at a time, so that the matrix
// loads of a thread depend on nothing but an LDS read (read one by one from memory they made a
// chain of dependent scalar loads).
// SPLIT parts of the work-group share out the rows, sixteen at a time, for 256 / SPLIT threads' columns:
// narrow matrices would leave the chip idle with a thread walking the whole batch, where the time
// is the number of dependent rounds of loads (8 x 256 rows of 4000 columns: 35.9 us without a split),
// and wide ones lose nothing (8 x 128 rows of 100003 columns, both kernels with streaming loads: 147 us against
// 155; 318 with a column per thread, as rows that do not start on 16 bytes were read before.  Both kernels
// are bound by the two reads of the batch, 5.6-6.4 TB/s; workers taken in groups of 60-220 MB and
// columns in reverse, so that more of the second read comes from the last-level cache, were no faster).
// The last work-group of a worker adds up the losses instead, if they are asked for.
template <int SPLIT, bool STREAM>
__global__ __launch_bounds__(kThreads) void dense_colsum_kernel(GradArgs a_all) {
  constexpr int kRows = 16, kStage = 1024, kCols = kThreads / SPLIT;
  const GradArgs a = for_worker(a_all);
  __shared__ int4 s_row[kStage / 4];                      // -1: no row or id out of range, adds nothing
  __shared__ float4 s_coef[kStage / 4];
  __shared__ double s_part[(SPLIT - 1) * 4 * kCols];
  const int64_t n4 = (a.d + 3) / 4;
  if ((int64_t)blockIdx.x * kCols >= n4) {
    reduce_loss(a, s_part);
    return;
  }
  int32_t* s_row1 = reinterpret_cast<int32_t*>(s_row);
  float* s_coef1 = reinterpret_cast<float*>(s_coef);
  const int part = (int)threadIdx.x / kCols, col = (int)threadIdx.x % kCols;
  const int64_t j = ((int64_t)blockIdx.x * kCols + col) * 4;
  const bool live = j < a.d, whole = j + 3 < a.d;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int c0 = 0; c0 < a.B; c0 += kStage) {
    const int nb = a.B - c0 < kStage ? a.B - c0 : kStage;
    const int nb_pad = (nb + kRows - 1) / kRows * kRows;
    if (c0 > 0) __syncthreads();                          // the previous ids have been used
    for (int i = threadIdx.x; i < nb_pad; i += kThreads) {
      const int32_t r = i < nb ? a.rows[c0 + i] : -1;
      const bool ok = r >= 0 && r < a.n_rows;
      s_row1[i] = ok ? r : -1;
      s_coef1[i] = ok ? a.coef[c0 + i] : 0.0f;
    }
    __syncthreads();
    if (!live) continue;
    for (int b0 = part * kRows; b0 < nb_pad; b0 += SPLIT * kRows) {
      int32_t r[kRows];
      float cf32[kRows];
#pragma unroll
      for (int u = 0; u < kRows / 4; ++u) {
        const int4 rr = s_row[b0 / 4 + u];
        const float4 cc = s_coef[b0 / 4 + u];
        r[4 * u] = rr.x; r[4 * u + 1] = rr.y; r[4 * u + 2] = rr.z; r[4 * u + 3] = rr.w;
        cf32[4 * u] = cc.x; cf32[4 * u + 1] = cc.y; cf32[4 * u + 2] = cc.z; cf32[4 * u + 3] = cc.w;
      }
      floatx4 v[kRows];
      if (whole) {
#pragma unroll
        for (int u = 0; u < kRows; ++u) v[u] = row_load4<STREAM>(a.A + (int64_t)(r[u] >= 0 ? r[u] : 0) * a.d + j);
      } else {                                            // the last columns of a row of odd length
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
          const float* p = a.A + (int64_t)(r[u] >= 0 ? r[u] : 0) * a.d + j;
          v[u].x = p[0];
          v[u].y = j + 1 < a.d ? p[1] : 0.0f;
          v[u].z = j + 2 < a.d ? p[2] : 0.0f;
          v[u].w = 0.0f;
        }
      }
#pragma unroll
      for (int u = 0; u < kRows; ++u) {
        const double cf = (double)cf32[u];
        if (r[u] < 0) v[u] = floatx4{0.f, 0.f, 0.f, 0.f};
        acc[0] = fma(cf, (double)v[u].x, acc[0]);
        acc[1] = fma(cf, (double)v[u].y, acc[1]);
        acc[2] = fma(cf, (double)v[u].z, acc[2]);
        acc[3] = fma(cf, (double)v[u].w, acc[3]);
      }
    }
  }
  if (part > 0) {
#pragma unroll
    for (int e = 0; e < 4; ++e) s_part[((part - 1) * 4 + e) * kCols + col] = acc[e];
  }
  __syncthreads();
  if (part > 0) return;
#pragma unroll
  for (int e = 0; e < 4; ++e)
#pragma unroll
    for (int q = 0; q < SPLIT - 1; ++q) acc[e] += s_part[(q * 4 + e) * kCols + col];
  if (whole) {
    *reinterpret_cast<float4*>(a.g + j) = make_float4((float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]);
  } else if (live) {
    a.g[j] = (float)acc[0];
    if (j + 1 < a.d) a.g[j + 1] = (float)acc[1];
    if (j + 2 < a.d) a.g[j + 2] = (float)acc[2];
  }
}

__global__ __launch_bounds__(kThreads) void fill_zero_kernel(float* p_all, int64_t n,
                                                            int64_t stride) {
  float* p = p_all + (int64_t)blockIdx.y * stride;
  const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) * 4;
  if (i + 3 < n) *reinterpret_cast<float4*>(p + i) = make_float4(0.f, 0.f, 0.f, 0.f);
  else for (int e = 0; e < 4; ++e) if (i + e < n) p[i + e] = 0.0f;
}

// one wave per batch row: margin, coef, loss; also clears the accumulator at the row's columns.
// ZERO_G: the work-groups of a worker first share out the zero-fill of its gradient vector (the
// stores drain while the latency-bound margins are computed); otherwise fill_zero_kernel ran before.
template <bool ZERO_G>
__global__ __launch_bounds__(kThreads) void csr_margin_kernel(GradArgs a_all) {
  const GradArgs a = for_worker(a_all);
  if (ZERO_G) {
    const int64_t n4 = a.d / 4;
    const int64_t per = (n4 + gridDim.x - 1) / gridDim.x;
    const int64_t lo = (int64_t)blockIdx.x * per, hi = lo + per < n4 ? lo + per : n4;
    float4* g4 = reinterpret_cast<float4*>(a.g);
    for (int64_t i = lo + threadIdx.x; i < hi; i += kThreads) g4[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (blockIdx.x == 0 && threadIdx.x < (a.d & 3)) a.g[4 * n4 + threadIdx.x] = 0.0f;
  }
  const int b = blockIdx.x * kWaves + threadIdx.x / kWave;
  if (b >= a.B) return;
  const int lane = threadIdx.x % kWave;
  const int64_t r = a.rows[b];
  const bool ok = r >= 0 && r < a.n_rows;
  double s = 0.0;
  if (ok) {
    const int64_t k0 = a.indptr[r], k1 = a.indptr[r + 1];
    for (int64_t k = k0 + lane; k < k1; k += kWave) {
      const uint32_t c = (uint32_t)a.indices[k];
      if (c < (uint64_t)a.d) {
        s = fma((double)a.A[k], (double)a.x[c], s);
        a.acc[c] = 0.0;
      }
    }
  }
  for (int off = 1; off < kWave; off <<= 1) s += shfl_xor_f64(s, off);
  if (lane == 0) {
    float c = 0.0f; double l = 0.0;
    if (ok) logistic_terms((float)s, a.y[r], a.B, &c, &l);
    a.coef[b] = c; a.loss_part[b] = l;
  }
}

template <bool FINALIZE>
__global__ __launch_bounds__(kThreads) void csr_scatter_kernel(GradArgs a_all) {
  const GradArgs a = for_worker(a_all);
  const int b = blockIdx.x * kWaves + threadIdx.x / kWave;
  if (b >= a.B) return;
  const int lane = threadIdx.x % kWave;
  const int64_t r = a.rows[b];
  if (r < 0 || r >= a.n_rows) return;
  const double cf = (double)a.coef[b];
  const int64_t k0 = a.indptr[r], k1 = a.indptr[r + 1];
  for (int64_t k = k0 + lane; k < k1; k += kWave) {
    const uint32_t c = (uint32_t)a.indices[k];
    if (c >= (uint64_t)a.d) continue;
    if (FINALIZE) a.g[c] = (float)a.acc[c];
    else unsafeAtomicAdd(&a.acc[c], cf * (double)a.A[k]);
  }
}

// ---- CSR rows, up to 2^22 columns: two launches, no global atomics -------------------------------
//
// A batch touches few of the d columns, at random.  An accumulator in memory costs three or four cache
// lines per entry (clear, atomic addition, read back, g) beside a zero-filled g.  Here instead
//
//   csr_bin     a work-group per group of rows (a multiple of 16, 16 lanes per row) forms their margins,
//               coefficients and losses, counts the entries per range of 2^LOGW columns, and writes the
//               entries -- value, batch row, column in its range -- to the group's part of the
//               workspace, ordered by range, with a table of where each range begins;
//   csr_gather  a work-group per range of a worker collects the groups' entries of its range, adds
//               coefficient * value into 2^LOGW binary64 accumulators in LDS and writes its part of g
//               in one piece, zeros included.
//
// A group whose entries do not fit its part of the workspace (all groups of a worker together have room for
// some 98 000 + d entries) leaves a mark, and csr_gather reads the group's rows themselves and takes what
// lies in its range.
//
// Ranges are as narrow as 256 of them allow (a counter per thread of csr_bin's work-group), at least 256
// columns, at most 16384 (128 KiB of LDS): narrow ones are more work-groups on short vectors (4 x 300
// rows of 150 entries, 5003 columns: 13.9 us with 256, 24 with 1024).  Beyond 2^22 columns the atomic form
// stays; at 2^22 (8 x 256 rows x 100) it takes 48 us, this one 39.
// Bound by the write of g (4 d bytes per worker) and, for few rows, by the chains of dependent loads (row
// id, row bounds, columns, x; table, entry, coefficient).  Atomic form -> this, batched calls: 16 x 256
// rows x 100 entries, d = 2^20 52.9 -> 26.4 us (csr_bin 10, csr_gather 16; 64 MiB of g alone take 11);
// 4 workers 21.0 -> 14.3; 16 x 384 x 200, d = 2^18 108 -> 32; 4 x 64 x 50, d = 4096 9.7 -> 9.4.
constexpr int kBinThreads = 256, kMaxRanges = 256, kMaxGroups = 64, kRowLanes = 16;
constexpr int kMinLogWidth = 8, kMaxLogWidth = 14;
constexpr uint32_t kOverflow = 0xffffffffu;
// The number of entries is known on the device only, so the line is drawn by the rows: the form is taken while
// the groups have room for kRowEntries entries per row (or for every column).  Without that line a
// batch that did not fit was read again by each of up to 256 ranges, in us, atomic form / no line / now:
// 1 x 65536 rows x 100, d = 2^20 787 / 3347 / 787; 4 of them 2660 / 5186 / 2668; 1 x 65536 x 50, d = 4096
// 627 / 4086 / 625; 8 x 4096 x 100, d = 2^17 302 / 528 / 302; 1 x 1700 x 200 there 53 / 123 / 52; and what is
// given up: 8 x 1700 x 100 there 132 / 34 / 132.  8 x 8192 x 100, d = 2^20 is just on this side: 631 / 117 / 120.
// Longer rows that overflow nevertheless cost up to twice the atomic form with one worker and 1.3 times with
// eight: 1 x 256 x 2000, d = 2^17 81 -> 157, 8 workers 267 -> 325; 1 x 8192 x 200, d = 2^20 194 -> 390.
// With room for less than kWideGather per row the gathering work-groups have 1024 threads, which reading again takes
// less ill (1 x 4096 x 1000, d = 2^20 981 -> 620; 2003 columns, 1 x 384 x 500 58 -> 40, 8 workers 91 -> 60);
// else 512 (16 x 256 x 100, d = 2^20 27.5 against 33.4).
constexpr int64_t kRowEntries = 128, kWideGather = 512;

// more entries than a worker's part of the workspace can hold
constexpr int64_t max_entries() {
  return (int64_t)(workspace_of(int64_t(kMaxRanges) << kMaxLogWidth, true) / sizeof(uint2));
}

struct BinArgs {
  uint32_t* table;           // [groups][ranges + 1], first range's entry kOverflow if the group did not fit
  uint2* entries;            // [groups][capacity]: value bits, batch row << 14 | column in range
  int64_t ws_stride_bytes;
  int groups, rows_per_group, ranges, log_width;
  uint32_t capacity;
};

__device__ __forceinline__ BinArgs for_worker(BinArgs b) {
  const int64_t m = blockIdx.y;
  b.table = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(b.table) + m * b.ws_stride_bytes);
  b.entries = reinterpret_cast<uint2*>(reinterpret_cast<char*>(b.entries) + m * b.ws_stride_bytes);
  return b;
}

__device__ __forceinline__ double row16_sum_f64(double v) {
  v += dpp_f64<kDppQuadXor1>(v);
  v += dpp_f64<kDppQuadXor2>(v);
  v += dpp_f64<kDppRowHalfMirror>(v);
  v += dpp_f64<kDppRowMirror>(v);
  return v;
}

// Up to 128 entries of a row, eight per lane of its team: column ids (0xffffffff: none), values.
constexpr int kAhead = 8;
struct RowChunk {
  uint32_t c[kAhead];
  float v[kAhead];
};
__device__ __forceinline__ void load_columns(const GradArgs& a, int64_t k, int64_t k1, uint32_t (&c)[kAhead]) {
#pragma unroll
  for (int u = 0; u < kAhead; ++u)
    c[u] = k + kRowLanes * u < k1 ? (uint32_t)a.indices[k + kRowLanes * u] : 0xffffffffu;
}
__device__ __forceinline__ void load_chunk(const GradArgs& a, int64_t k, int64_t k1, RowChunk& q) {
  load_columns(a, k, k1, q.c);
#pragma unroll
  for (int u = 0; u < kAhead; ++u) q.v[u] = k + kRowLanes * u < k1 ? a.A[k + kRowLanes * u] : 0.0f;
}

// ONE_ROW: a team has one row, whose row bounds and first 128 entries stay in registers between the
// counting and the writing (the time of small batches is the chain of dependent loads).
template <bool ONE_ROW>
__global__ __launch_bounds__(kBinThreads) void csr_bin_kernel(GradArgs a_all, BinArgs b_all) {
  const GradArgs a = for_worker(a_all);
  const BinArgs b = for_worker(b_all);
  __shared__ uint32_t count[kMaxRanges];
  __shared__ uint32_t place[kMaxRanges];                 // where the range's entries without a rank go
  __shared__ uint32_t wave_total[kBinThreads / kWave];
  constexpr int kTeams = kBinThreads / kRowLanes, kStep = kRowLanes * kAhead;
  const int t = threadIdx.x, lane = t % kRowLanes, team = t / kRowLanes;
  const int group = blockIdx.x;
  const int first = group * b.rows_per_group;
  const int last = first + b.rows_per_group < a.B ? first + b.rows_per_group : a.B;
  const uint32_t d = (uint32_t)a.d;
  count[t] = 0u;
  place[t] = 0u;
  __syncthreads();
  RowChunk q;
  uint32_t rank[kAhead];                                 // of the chunk in registers, among the range's
  int64_t k0 = 0, k1 = 0;
  double s = 0.0;
  bool ok = false;
  float label = 0.0f;
  int64_t listed = 0;                                    // entries of the team's rows, whatever their columns
  const auto row_bounds = [&](int i) {
    const int64_t r = i < last ? a.rows[i] : -1;
    ok = r >= 0 && r < a.n_rows;
    k0 = ok ? a.indptr[r] : 0;
    k1 = ok ? a.indptr[r + 1] : 0;
    label = ok ? a.y[r] : 0.0f;
  };
  const auto count_chunk = [&](bool ranked) {
    float x[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) x[u] = q.c[u] < d ? a.x[q.c[u]] : 0.0f;
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (q.c[u] < d) {
        if (ranked) rank[u] = atomicAdd(&count[q.c[u] >> b.log_width], 1u);
        else atomicAdd(&place[q.c[u] >> b.log_width], 1u);
      }
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (q.c[u] < d) s = fma((double)q.v[u], (double)x[u], s);
  };
  // coefficient and loss of row i from the team's margin, by two lanes
  const auto finish_row = [&](int i) {
    if (i < last && lane < 2) {
      float coef = 0.0f; double loss = 0.0;
      if (ok) logistic_terms((float)s, label, a.B, &coef, &loss);
      if (lane == 0) a.coef[i] = coef;
      else a.loss_part[i] = loss;
    }
  };
  if (ONE_ROW) {
    row_bounds(first + team);
    listed = k1 - k0;
    for (int64_t k = k1 - k0 > kStep ? k0 + kStep + lane : k1; k < k1; k += kStep) {       // beyond the first chunk
      load_chunk(a, k, k1, q);
      count_chunk(false);
    }
    load_chunk(a, k0 + lane, k1, q);
    count_chunk(true);
    s = row16_sum_f64(s);
  } else {
    for (int i = first + team; i < last; i += kTeams) {
      row_bounds(i);
      listed += k1 - k0;
      s = 0.0;
      for (int64_t k = k0 + lane; k < k1; k += kStep) {
        load_chunk(a, k, k1, q);
        count_chunk(false);
      }
      s = row16_sum_f64(s);
      finish_row(i);
    }
  }
  __syncthreads();
  // where each range begins in the group's part
  const uint32_t ranked = count[t], mine = ranked + place[t];
  uint32_t incl = mine;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t o = __shfl_up(incl, off, kWave);
    if (t % kWave >= off) incl += o;
  }
  // The counters are 32 bits wide: they hold the group's entries as long as no team alone has more than the
  // group's part of the workspace takes, and a group with such a team does not fit in any case.
  static_assert(kTeams * (max_entries() + 1) < (int64_t(1) << 32), "a group that passes the test cannot wrap its counters");
  const bool too_many = __any(listed > (int64_t)b.capacity);
  if (t % kWave == kWave - 1) wave_total[t / kWave] = too_many ? b.capacity + 1u : incl;
  __syncthreads();
  uint32_t before = incl - mine, total = 0;
#pragma unroll
  for (int w = 0; w < kBinThreads / kWave; ++w) {
    if (w < t / kWave) before += wave_total[w];
    total += wave_total[w];
  }
  uint32_t* table = b.table + (int64_t)group * (b.ranges + 1);
  const bool fits = total <= b.capacity;                 // the same for the whole work-group
  if (t < b.ranges) table[t] = !fits && t == 0 ? kOverflow : before;
  if (t == 0) table[b.ranges] = total;
  count[t] = before;
  place[t] = before + ranked;
  __syncthreads();
  uint2* entries = b.entries + (int64_t)group * b.capacity;
  const uint32_t in_range = (1u << b.log_width) - 1u;
  const auto write_chunk = [&](int i, bool is_ranked) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u)
      if (q.c[u] < d) {
        const uint32_t of = q.c[u] >> b.log_width;
        const uint32_t at = is_ranked ? count[of] + rank[u] : atomicAdd(&place[of], 1u);
        entries[at] = make_uint2(__float_as_uint(q.v[u]), ((uint32_t)i << 14) | (q.c[u] & in_range));
      }
  };
  if (ONE_ROW) {
    if (fits) {
      write_chunk(first + team, true);
      for (int64_t k = k1 - k0 > kStep ? k0 + kStep + lane : k1; k < k1; k += kStep) {
        load_chunk(a, k, k1, q);
        write_chunk(first + team, false);
      }
    }
    finish_row(first + team);
  } else if (fits) {
    for (int i = first + team; i < last; i += kTeams) {
      row_bounds(i);
      for (int64_t k = k0 + lane; k < k1; k += kStep) {
        load_chunk(a, k, k1, q);
        write_chunk(i, false);
      }
    }
  }
}


template <int LOGW, int THREADS>
__global__ __launch_bounds__(THREADS) void csr_gather_kernel(GradArgs a_all, BinArgs b_all) {
  constexpr int kWidth = 1 << LOGW, kThr = THREADS, kTeams = kThr / kRowLanes;
  const GradArgs a = for_worker(a_all);
  const BinArgs b = for_worker(b_all);
  __shared__ double acc[kWidth];
  __shared__ int overflow;
  static_assert(kThr / kWave <= kWidth, "room for the waves' sums");
  const int t = threadIdx.x, lane = t % kRowLanes, team = t / kRowLanes;
  const uint32_t range = blockIdx.x;
  if ((int)range >= b.ranges) {                            // a worker's extra work-group: the loss
    double s = 0.0;
    for (int i = t; i < a.B; i += kThr) s += a.loss_part[i];
    s = wave_sum_f64(s);
    if (t % kWave == 0) acc[t / kWave] = s;
    __syncthreads();
    if (t == 0) {
      double all = 0.0;
      for (int w = 0; w < kThr / kWave; ++w) all += acc[w];
      *a.loss_out = (float)(all / (double)a.B);
    }
    return;
  }
  // a team's first 64 entries of one group are on their way while the accumulators are cleared
  uint2 e[4];
  float coef[4];
  uint32_t lo = 0, hi = 0;
  bool marked = false;
  const uint2* entries = b.entries;
  const auto load_entries = [&](uint32_t i) {
#pragma unroll
    for (int u = 0; u < 4; ++u) e[u] = i + kRowLanes * u < hi ? entries[i + kRowLanes * u] : make_uint2(0u, 0u);
#pragma unroll
    for (int u = 0; u < 4; ++u) coef[u] = i + kRowLanes * u < hi ? a.coef[e[u].y >> 14] : 0.0f;
  };
  const auto open_group = [&](int g) {
    const uint32_t* table = b.table + (int64_t)g * (b.ranges + 1);
    const bool live = g < b.groups;
    const uint32_t first = live ? table[0] : 0u;
    lo = live ? table[range] : 0u;
    hi = live ? table[range + 1] : 0u;
    marked = first == kOverflow;
    if (marked) lo = hi = 0u;
    entries = b.entries + (int64_t)g * b.capacity;
    load_entries(lo + lane);
  };
  open_group(team);
  for (int i = t; i < kWidth / 2; i += kThr) reinterpret_cast<double2*>(acc)[i] = make_double2(0.0, 0.0);
  if (t == 0) overflow = 0;
  __syncthreads();
  for (int g = team; g < b.groups;) {
    if (marked && lane == 0) overflow = 1;
    for (uint32_t i = lo + lane; i < hi;) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (i + kRowLanes * u < hi)
          unsafeAtomicAdd(&acc[e[u].y & (kWidth - 1)], (double)coef[u] * (double)__uint_as_float(e[u].x));
      i += kRowLanes * 4;
      if (i < hi) load_entries(i);
    }
    g += kTeams;
    if (g < b.groups) open_group(g);
  }
  __syncthreads();
  if (overflow) {
    for (int i = team; i < a.B; i += kTeams) {
      const int64_t r = a.rows[i];
      if (r < 0 || r >= a.n_rows || b.table[(int64_t)(i / b.rows_per_group) * (b.ranges + 1)] != kOverflow) continue;
      const double coef = (double)a.coef[i];
      const int64_t k1 = a.indptr[r + 1];
      for (int64_t k = a.indptr[r] + lane; k < k1; k += kRowLanes * kAhead) {
        uint32_t c[kAhead];
        load_columns(a, k, k1, c);
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
          if (c[u] < (uint32_t)a.d && c[u] >> LOGW == range)
            unsafeAtomicAdd(&acc[c[u] & (kWidth - 1)], coef * (double)a.A[k + kRowLanes * u]);
      }
    }
    __syncthreads();
  }
  const int64_t c0 = (int64_t)range << LOGW;
  const int n = a.d - c0 < kWidth ? (int)(a.d - c0) : kWidth;
  float* g = a.g + c0;
  for (int i = 4 * t; i < n; i += 4 * kThr) {
    if (i + 3 < n) {
      *reinterpret_cast<float4*>(g + i) = make_float4((float)acc[i], (float)acc[i + 1], (float)acc[i + 2], (float)acc[i + 3]);
    } else {
      for (int e = 0; i + e < n; ++e) g[i + e] = (float)acc[i + e];
    }
  }
}

__global__ __launch_bounds__(kThreads) void loss_finalize_kernel(GradArgs a_all) {
  const GradArgs a = for_worker(a_all);
  __shared__ double lds_d[kWaves];
  reduce_loss(a, lds_d);
}

size_t grad_workspace_bytes(int64_t d, bool csr) { return workspace_of(d, csr); }

// The two-launch form for CSR rows; false if the vector is too long for its ranges or the batch has too many
// rows for the workspace.  A worker's part of
// the workspace holds [coefficients][losses][table][entries]: grad_workspace_bytes counts the first two
// for the largest batch, so some 98 000 entries fit beside the d of the accumulator.
static bool csr_launch(GradArgs a, int M, hipStream_t stream) {
  int log_width = kMinLogWidth;
  while (((a.d + (int64_t(1) << log_width) - 1) >> log_width) > kMaxRanges) ++log_width;
  if (log_width > kMaxLogWidth) return false;
  BinArgs b{};
  b.log_width = log_width;
  b.ranges = (int)((a.d + (int64_t(1) << log_width) - 1) >> log_width);
  const int teams = kBinThreads / kRowLanes;
  b.rows_per_group = teams * ((a.B + teams * kMaxGroups - 1) / (teams * kMaxGroups));
  b.groups = (a.B + b.rows_per_group - 1) / b.rows_per_group;
  char* const base = reinterpret_cast<char*>(a.coef);
  size_t at = align256((size_t)a.B * sizeof(float));
  a.loss_part = reinterpret_cast<double*>(base + at);
  at += align256((size_t)a.B * sizeof(double));
  b.table = reinterpret_cast<uint32_t*>(base + at);
  at += align256((size_t)b.groups * (b.ranges + 1) * sizeof(uint32_t));
  if (at > (size_t)a.ws_stride_bytes) return false;
  b.entries = reinterpret_cast<uint2*>(base + at);
  const size_t room = ((size_t)a.ws_stride_bytes - at) / sizeof(uint2) / (size_t)b.groups;
  b.capacity = room < (size_t)kOverflow ? (uint32_t)room : kOverflow - 1u;
  const int64_t per_row = (int64_t)b.capacity / b.rows_per_group;
  if (per_row < (a.d < kRowEntries ? a.d : kRowEntries)) return false;
  const bool wide = log_width >= 14 || per_row < kWideGather;
  b.ws_stride_bytes = a.ws_stride_bytes;
  const dim3 grid((unsigned)b.ranges + (a.loss_out ? 1u : 0u), (unsigned)M), groups((unsigned)b.groups, (unsigned)M);
  if (b.rows_per_group == teams) hipLaunchKernelGGL(csr_bin_kernel<true>, groups, dim3(kBinThreads), 0, stream, a, b);
  else hipLaunchKernelGGL(csr_bin_kernel<false>, groups, dim3(kBinThreads), 0, stream, a, b);
  switch (log_width) {
#define QA_GATHER(w, threads) hipLaunchKernelGGL((csr_gather_kernel<w, threads>), grid, dim3(threads), 0, stream, a, b)
#define QA_GATHER_EITHER(w) case w: if (wide) QA_GATHER(w, 1024); else QA_GATHER(w, 512); break
    QA_GATHER_EITHER(8); QA_GATHER_EITHER(9); QA_GATHER_EITHER(10);
    QA_GATHER_EITHER(11); QA_GATHER_EITHER(12); QA_GATHER_EITHER(13);
    case 14: QA_GATHER(14, 1024); break;
#undef QA_GATHER_EITHER
#undef QA_GATHER
    default: return false;
  }
  return true;
}

static int grad_launch(int format, const float* A_or_vals, const int64_t* indptr,
                       const int32_t* indices, int64_t n_rows, int64_t d, const float* y,
                       const int32_t* batch_rows, int32_t B, int32_t M, const float* x, float* g_out,
                       int64_t g_stride, float* loss_out, void* ws, size_t ws_bytes,
                       hipStream_t stream) {
  if (format != QA_DENSE && format != QA_CSR) return QA_ERR_INVALID_ARG;
  if (!A_or_vals || !y || !batch_rows || !x || !g_out) return QA_ERR_INVALID_ARG;
  if (format == QA_CSR && (!indptr || !indices)) return QA_ERR_INVALID_ARG;
  if (n_rows < 1 || d < 1 || d >= (int64_t(1) << 31) || B < 1 || B > kMaxBatch || M < 1 || M > 4096)
    return QA_ERR_INVALID_ARG;
  if (M > 1 && (g_stride < d || (g_stride % 4) != 0)) return QA_ERR_INVALID_ARG;
  if (!aligned(g_out, 16) || !aligned(A_or_vals, 4) || !aligned(x, 4) || !aligned(indptr, 8) ||
      !aligned(indices, 4) || !aligned(batch_rows, 4) || !aligned(loss_out, 4))
    return QA_ERR_ALIGNMENT;
  const bool csr = format == QA_CSR;
  const size_t per_worker = grad_workspace_bytes(d, csr);
  if (!ws || ws_bytes < per_worker * (size_t)M) return QA_ERR_WORKSPACE;
  if (!aligned(ws, 256)) return QA_ERR_ALIGNMENT;

  GradArgs a{};
  a.A = A_or_vals; a.indptr = indptr; a.indices = indices; a.n_rows = n_rows; a.d = d;
  a.y = y; a.rows = batch_rows; a.B = B; a.x = x; a.g = g_out; a.loss_out = loss_out;
  a.g_stride = g_stride; a.ws_stride_bytes = (int64_t)per_worker;
  char* p = static_cast<char*>(ws);
  a.coef = reinterpret_cast<float*>(p);        p += align256((size_t)kMaxBatch * sizeof(float));
  a.loss_part = reinterpret_cast<double*>(p);  p += align256((size_t)kMaxBatch * sizeof(double));
  a.acc = reinterpret_cast<double*>(p);

  const dim3 block(kThreads);
  const unsigned Mu = (unsigned)M;
  if (!csr) {
    const int64_t n4 = (d + 3) / 4;
    const unsigned extra = loss_out ? 1u : 0u;            // a work-group per worker for the loss
    const int64_t rows = n_rows < (int64_t)M * B ? n_rows : (int64_t)M * B;   // different ones, at most
    const bool streamed = rows > kStreamedBatch / d;
    if (d <= kShortRow)
      hipLaunchKernelGGL((streamed ? dense_margin_kernel<kWave, true> : dense_margin_kernel<kWave, false>),
                         dim3((B + kWaves - 1) / kWaves, Mu), block, 0, stream, a);
    else
      hipLaunchKernelGGL((streamed ? dense_margin_kernel<kThreads, true> : dense_margin_kernel<kThreads, false>),
                         dim3(B, Mu), block, 0, stream, a);
    const int64_t groups = (n4 + kWave - 1) / kWave;
    if (groups * M < kFewGroups && B > 64)
      hipLaunchKernelGGL((streamed ? dense_colsum_kernel<16, true> : dense_colsum_kernel<16, false>),
                         dim3((unsigned)((n4 + 15) / 16) + extra, Mu), block, 0, stream, a);
    else
      hipLaunchKernelGGL((streamed ? dense_colsum_kernel<4, true> : dense_colsum_kernel<4, false>),
                         dim3((unsigned)groups + extra, Mu), block, 0, stream, a);
    return launch_status();
  } else if (csr_launch(a, M, stream)) {
    return launch_status();
  } else {
    const dim3 grid_rows((B + kWaves - 1) / kWaves, Mu);
    // few rows for a long vector: the zero-fill gets a launch of its own
    const bool fused_fill = d / 4 <= (int64_t)grid_rows.x * kThreads * 32;
    if (fused_fill) {
      hipLaunchKernelGGL(csr_margin_kernel<true>, grid_rows, block, 0, stream, a);
    } else {
      hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)((d + 4 * kThreads - 1) / (4 * kThreads)), Mu),
                         block, 0, stream, g_out, d, g_stride);
      hipLaunchKernelGGL(csr_margin_kernel<false>, grid_rows, block, 0, stream, a);
    }
    hipLaunchKernelGGL((csr_scatter_kernel<false>), grid_rows, block, 0, stream, a);
    hipLaunchKernelGGL((csr_scatter_kernel<true>), grid_rows, block, 0, stream, a);
  }
  if (loss_out) hipLaunchKernelGGL(loss_finalize_kernel, dim3(1, Mu), block, 0, stream, a);
  return launch_status();
}

}  // namespace qa

extern "C" int qa_local_grad(int format, const float* A_or_vals, const int64_t* indptr,
                             const int32_t* indices, int64_t n_rows, int64_t d, const float* y,
                             const int32_t* batch_rows, int32_t B, const float* x, float* g_out,
                             float* loss_out, void* ws, size_t ws_bytes, void* stream) {
  return qa::grad_launch(format, A_or_vals, indptr, indices, n_rows, d, y, batch_rows, B, 1, x, g_out,
                         0, loss_out, ws, ws_bytes, static_cast<hipStream_t>(stream));
}

extern "C" int qa_local_grad_batched(int format, const float* A_or_vals, const int64_t* indptr,
                                     const int32_t* indices, int64_t n_rows, int64_t d,
                                     const float* y, const int32_t* batch_rows, int32_t B, int32_t M,
                                     const float* x, float* g_out, int64_t g_stride, float* loss_out,
                                     void* ws, size_t ws_bytes, void* stream) {
  return qa::grad_launch(format, A_or_vals, indptr, indices, n_rows, d, y, batch_rows, B, M, x, g_out,
                         g_stride, loss_out, ws, ws_bytes, static_cast<hipStream_t>(stream));
}
