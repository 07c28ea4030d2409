// Exact least-squares threshold (Section 3.4: rank the magnitudes and try each one as the
// threshold) for buckets longer than one 4096-tile and for one threshold over a whole vector, for
// gfx950.  The per-tile form lives with the quantizer; qa_quantize_pack with QA_THRESH_EXACT comes
// here when a bucket spans tiles.  Not on the method's hot path: Section 3.5 introduces the
// 0.75 mean|v| rule precisely to avoid this ranking.
//
// The objective of keeping the k largest is (their sum)^2 / k.  Ranking everything is avoided by
// refining a histogram of the bit patterns of |v| (which order like the magnitudes):
//
//   level 0   4096 bins of 2^19 patterns (16 per binade) over all non-zero magnitudes.  A bin holds
//             its count and the sum of its members' offsets from its lower end in units of the last
//             place: integers, so the bin's sum is exact and does not depend on the order of the
//             atomic additions.
//   scan      per bin, from the top: count and sum of everything kept when the cut lies at the bin's
//             lower end, the objective there, and a bound for every cut inside the bin: the j largest
//             of c members with sum c L + o in [L, H) sum to at most min(j H, o + j L), and
//             (A + B j)^2 / (K + j) is convex in j, so the bound is largest where the two meet,
//             j = o / (H - L).  Bins whose bound reaches the best edge survive, with the
//             next filled bin below each (it holds the largest magnitude not kept).
//   level 1.. the survivors are divided again, up to 4096 parts in all, until a bin is one pattern.
//             Then the best edge is the optimum (smallest k among equal objectives) and the
//             magnitude of the next filled bin is the threshold, compared with strictly.
//
// A smooth distribution leaves 2-4 bins per level: three levels, i.e. three reads of the gradient.
// Every sum is formed in binary64 from exact parts; candidates whose objectives agree to binary64
// rounding may be resolved differently from a strictly sequential summation (likely only beyond some
// 1e7 components per bucket; both kept sets are then optimal to that resolution).  A bucket that
// more than 2048 bins or five levels leave open (an objective constructed to be flat) is sorted by one
// work-group behind the levels.  Infinite members are kept alone, a NaN gives the threshold 0.
//
// Measured against a device-wide radix sort with four passes behind it (2^26 x 4 Gaussian components,
// thresholds and codes): one threshold per vector 6660 -> 850 us (three reads of the gradient at
// 5.2-5.4 TB/s and one for the codes), buckets of 65536 15.5 -> 1.1 ms, of 8192 15.9 -> 4.6 ms (bound by
// the scans, some 20 us per level and work-group); 9001 x 4 components 165 -> 43 us, 10^6 x 8 1258 -> 150.
#include "qa_common.h"

namespace qa {

constexpr int kLogBins = 12, kBins = 1 << kLogBins;
constexpr int kFirstShift = 31 - kLogBins;               // level 0: pattern >> 19
constexpr int kRanges = kBins / 2;
constexpr int kLevels = 5;
constexpr int kScanThreads = 1024, kScanWaves = kScanThreads / kWave, kPerThread = kBins / kScanThreads;
constexpr int kCountShift = 40;                          // LDS bin: count << 40 | sum of offsets
constexpr float kOpenMark = -1.0f;                       // threshold of a bucket still to be found
constexpr uint32_t kNonFinite = 0x7f800000u;

// The bins of one level, from the largest magnitudes down: `nr` ranges of 2^width patterns starting at
// lo[r], each divided into 2^sub bins of 2^shift patterns.  Bin position r * 2^sub + (2^sub - 1 - part).
struct LevelShape {
  int nr, width, sub, shift;
};
struct LevelRanges {
  uint32_t lo[kRanges];
  uint32_t count_before[kRanges];                        // magnitudes above the range: how many, their sum
  double sum_before[kRanges];
};

__device__ __forceinline__ uint32_t lower_end(const LevelShape& s, const uint32_t* lo, int pos) {
  const uint32_t part = (1u << s.sub) - 1u - ((uint32_t)pos & ((1u << s.sub) - 1u));
  return lo[pos >> s.sub] + (part << s.shift);
}

// position and offset of a pattern in level s, -1 if it lies in no range
// (which is not below the lowest)
__device__ __forceinline__ int bin_of(const LevelShape& s, const uint32_t* lo, uint32_t bits) {
  int r = 0;                                             // first range with lo[r] <= bits
  for (int n = s.nr; n > 1;) {
    const int half = n >> 1;
    r += lo[r + half - 1] > bits ? half : 0;
    n -= half;
  }
  const uint32_t rel = bits - lo[r];
  if (rel >> s.width) return -1;
  return (r << s.sub) + (int)((1u << s.sub) - 1u - (rel >> s.shift));
}

// ---- the scan of a level by a work-group of 1024 threads, four bins each ------------------------

struct ScanLds {
  LevelRanges ranges;                                    // in: this level's; out: the next level's
  double wave_f[kScanWaves];
  uint32_t wave_u[kScanWaves];
  int wave_i[kScanWaves];
  double best_obj[kScanWaves];
  uint32_t best_k[kScanWaves];
  int best_pos[kScanWaves];
  uint8_t survives[kScanThreads];                        // bit i: bin 4 t + i
  uint32_t threshold_bits;
};

// sum over the threads before this one; *total = over all
template <typename T>
__device__ __forceinline__ T scan_exclusive(T v, T* lds, T* total) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  T incl = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const T o = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += o;
  }
  __syncthreads();                                       // earlier readers of lds are done
  if (lane == kWave - 1) lds[wave] = incl;
  __syncthreads();
  T before = 0, all = 0;
  for (int w = 0; w < kScanWaves; ++w) {
    if (w < wave) before += lds[w];
    all += lds[w];
  }
  *total = all;
  // by the neighbour and not incl - v: exact in binary64 as well
  const T left = __shfl_up(incl, 1, kWave);
  return before + (lane ? left : (T)0);
}

// largest v over the threads before this one (0 if none); v >= 0
__device__ __forceinline__ int scan_exclusive_max(int v, int* lds) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  int incl = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int o = __shfl_up(incl, off, kWave);
    if (lane >= off && o > incl) incl = o;
  }
  __syncthreads();
  if (lane == kWave - 1) lds[wave] = incl;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wave; ++w) before = lds[w] > before ? lds[w] : before;
  const int left = __shfl_up(incl, 1, kWave);
  return lane && left > before ? left : before;
}

__device__ __forceinline__ double ulp_of(uint32_t bits) {      // of a finite positive pattern
  const int e = (int)(bits >> 23);
  return __hiloint2double(((e ? e : 1) - 150 + 1023) << 20, 0);
}

enum ScanResult { kScanRefine = 0, kScanDone = 1, kScanGiveUp = 2 };

// c, off: count and offset sum of this thread's bins 4 t .. 4 t + 3.  kScanDone: lds.threshold_bits
// holds the threshold; kScanRefine: *shape and lds.ranges are the next level's.  Work-group uniform.
__device__ __forceinline__ ScanResult scan_level(LevelShape* shape, bool first, const uint32_t (&c)[kPerThread],
                                                 const uint64_t (&off)[kPerThread], ScanLds& lds) {
  const LevelShape s = *shape;
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  const int nbins = s.nr << s.sub;
  uint32_t low[kPerThread];
  double sum[kPerThread];
  uint32_t cnt = 0;
  double mine = 0.0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int pos = kPerThread * t + i;
    low[i] = pos < nbins ? lower_end(s, lds.ranges.lo, pos) : 0u;
    sum[i] = c[i] ? fma((double)off[i], ulp_of(low[i]), (double)c[i] * (double)__uint_as_float(low[i])) : 0.0;
    cnt += c[i];
    mine += sum[i];
  }
  if (t == 0) lds.threshold_bits = 0u;
  if (first) {                                           // NaN members: in the top bins of level 0
    bool odd = false;
    if (t <= (int)((kBins - 1 - (kNonFinite >> kFirstShift)) / kPerThread))
#pragma unroll
      for (int i = 0; i < kPerThread; ++i)
        odd |= c[i] != 0 && (low[i] > kNonFinite || (low[i] == kNonFinite && off[i] != 0));
    if (__syncthreads_or(odd)) return kScanDone;
  }
  uint32_t total_cnt;
  double total_sum;
  uint32_t k_run = scan_exclusive(cnt, lds.wave_u, &total_cnt);
  double s_run = scan_exclusive(mine, lds.wave_f, &total_sum);
  if (total_cnt == 0) return kScanDone;                  // nothing but zeros
  // what lies before a range in this scan is replaced by what lies above it in the bucket
  if (!first) {
    uint32_t k_at = k_run;
    double s_at = s_run;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const int pos = kPerThread * t + i;
      if (pos < nbins && (pos & ((1 << s.sub) - 1)) == 0) {
        lds.ranges.count_before[pos >> s.sub] -= k_at;
        lds.ranges.sum_before[pos >> s.sub] -= s_at;
      }
      k_at += c[i];
      s_at += sum[i];
    }
    __syncthreads();
  }
  double s_before[kPerThread], edge[kPerThread], inner[kPerThread];
  uint32_t k_before[kPerThread];
  double best = -1.0;
  uint32_t best_k = 0;
  int best_pos = -1;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int pos = kPerThread * t + i;
    k_before[i] = k_run;
    s_before[i] = s_run;
    if (!first && pos < nbins) {
      k_before[i] += lds.ranges.count_before[pos >> s.sub];
      s_before[i] += lds.ranges.sum_before[pos >> s.sub];
    }
    const double k1 = (double)(k_before[i] + c[i]), s1 = s_before[i] + sum[i];
    edge[i] = c[i] ? s1 * s1 / k1 : -1.0;
    inner[i] = -1.0;
    if (c[i] > 1 && off[i] != 0 && s.shift > 0) {
      const double width = ulp_of(low[i]) * (double)(1u << s.shift);
      const double j = (double)off[i] / (double)(1u << s.shift);
      const double s_in = s_before[i] + j * ((double)__uint_as_float(low[i]) + width);
      inner[i] = s_in * s_in / ((double)k_before[i] + j);
    }
    if (edge[i] > best) { best = edge[i]; best_k = k_before[i] + c[i]; best_pos = pos; }
    k_run += c[i];
    s_run += sum[i];
  }
  // the best edge, smallest k among equal ones (later positions keep more)
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double ob = __shfl_xor(best, o, kWave);
    const uint32_t ok = __shfl_xor(best_k, o, kWave);
    const int op = __shfl_xor(best_pos, o, kWave);
    if (ob > best || (ob == best && ok < best_k)) { best = ob; best_k = ok; best_pos = op; }
  }
  if (lane == 0) { lds.best_obj[wave] = best; lds.best_k[wave] = best_k; lds.best_pos[wave] = best_pos; }
  __syncthreads();
  best = lds.best_obj[0]; best_k = lds.best_k[0]; best_pos = lds.best_pos[0];
  for (int w = 1; w < kScanWaves; ++w)
    if (lds.best_obj[w] > best || (lds.best_obj[w] == best && lds.best_k[w] < best_k)) {
      best = lds.best_obj[w]; best_k = lds.best_k[w]; best_pos = lds.best_pos[w];
    }
  const double bar = best * (1.0 - 1e-11);               // far above the rounding of the binary64 sums
  const bool infinite = best > 1e300;                    // infinite members: they alone are kept (the smallest k)
  uint32_t survives = 0;
  int last = 0;                                          // 1 + position of this thread's last filled bin
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    if (edge[i] >= bar || inner[i] >= bar) survives |= 1u << i;
    if (c[i]) last = kPerThread * t + i + 1;
  }
  if (infinite) survives = best_pos / kPerThread == t ? 1u << (best_pos % kPerThread) : 0u;
  lds.survives[t] = (uint8_t)survives;
  int previous = scan_exclusive_max(last, lds.wave_i);   // (barriers inside: survives[] is visible)
  if (s.shift == 0) {                                    // bins are single patterns: this is the optimum
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if (c[i]) {
        if (previous == best_pos + 1) lds.threshold_bits = low[i];
        previous = kPerThread * t + i + 1;
      }
    __syncthreads();
    return kScanDone;
  }
  uint32_t keep = 0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i)
    if (c[i]) {
      const int q = previous - 1;
      const bool follows = q >= 0 && ((lds.survives[q / kPerThread] >> (q % kPerThread)) & 1u);
      if (((survives >> i) & 1u) || follows) keep |= 1u << i;
      previous = kPerThread * t + i + 1;
    }
  uint32_t n;
  uint32_t at = scan_exclusive((uint32_t)__popc(keep), lds.wave_u, &n);
  if (n > (uint32_t)kRanges) return kScanGiveUp;
  // (the scan's barriers lie between the last read of this level's ranges and the writes below)
#pragma unroll
  for (int i = 0; i < kPerThread; ++i)
    if ((keep >> i) & 1u) {
      lds.ranges.lo[at] = low[i];
      lds.ranges.count_before[at] = k_before[i];
      lds.ranges.sum_before[at] = s_before[i];
      ++at;
    }
  int sub = kLogBins - (n > 1 ? 32 - __clz((int)(n - 1)) : 0);
  if (sub > s.shift) sub = s.shift;
  shape->nr = (int)n; shape->width = s.shift; shape->sub = sub; shape->shift = s.shift - sub;
  __syncthreads();
  return kScanRefine;
}

__device__ __forceinline__ LevelShape first_shape() { return LevelShape{1, 31, kLogBins, kFirstShift}; }

// ---- buckets of up to 65536 components: a work-group each, all levels in LDS ----------------------

struct WideArgs {
  const float* g;
  int64_t g_stride, d, bucket_len, nb;
  float* thresholds;
  int64_t scale_stride;
  int m0;                                                // first worker of this launch
  char* state;                                           // per (worker, bucket): see below
  uint32_t* sort_keys;                                   // two arrays of d keys
};

// The bucket (at most 256 KiB) is read from memory once and by the later levels from the caches: kept
// in registers, 64 components per thread, it leaves no room for the scan.  Beyond 65536 the levels
// become launches: a work-group alone would leave the chip idle, and the state of every (bucket,
// worker) has to fit the workspace.
constexpr int kResidentMost = 65536;
template <typename F>
__device__ __forceinline__ void for_each_pattern(const float* g, int64_t lo, int64_t hi, int threads, F f) {
  typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
  constexpr int kAhead = 8;                              // 16-byte loads in flight per thread
  int64_t i = lo + 4 * (int)threadIdx.x;
  for (; i + 4 * threads * (kAhead - 1) + 3 < hi; i += 4 * threads * kAhead) {
    uintx4 q[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) q[j] = *reinterpret_cast<const uintx4*>(g + i + 4 * threads * j);
#pragma unroll
    for (int j = 0; j < kAhead; ++j) { f(q[j].x); f(q[j].y); f(q[j].z); f(q[j].w); }
  }
  for (; i < hi; i += 4 * threads)
    for (int e = 0; e < 4; ++e)
      if (i + e < hi) f(__float_as_uint(g[i + e]));
}

// One level's histogram in LDS; patterns of zeros are left out.
__device__ __forceinline__ void add_first(unsigned long long* hist, uint32_t raw) {
  const uint32_t bits = raw & 0x7fffffffu;
  if (bits)
    atomicAdd(hist + (kBins - 1 - (bits >> kFirstShift)),
              (1ull << kCountShift) | (unsigned long long)(bits & ((1u << kFirstShift) - 1u)));
}
struct Envelope {
  uint32_t lo, len;
};
__device__ __forceinline__ Envelope envelope_of(const LevelShape& s, const uint32_t* lo) {
  return Envelope{lo[s.nr - 1], lo[0] - lo[s.nr - 1] + (1u << s.width)};
}
__device__ __forceinline__ void add_in_ranges(unsigned long long* hist, const LevelShape& s, const uint32_t* lo,
                                              const Envelope& env, uint32_t raw) {
  const uint32_t bits = raw & 0x7fffffffu;
  if (bits - env.lo >= env.len) return;
  const int pos = bin_of(s, lo, bits);
  // (ranges start on multiples of 2^shift: the low bits are the offset in the bin)
  if (pos >= 0 && bits)
    atomicAdd(hist + pos, (1ull << kCountShift) | (unsigned long long)(bits & ((1u << s.shift) - 1u)));
}

__global__ __launch_bounds__(kScanThreads) void exact_resident_kernel(WideArgs a) {
  __shared__ ScanLds lds;
  __shared__ unsigned long long hist[kBins];
  const int t = threadIdx.x;
  const int64_t k = blockIdx.x, lo = k * a.bucket_len;
  const int m = blockIdx.y;
  const int64_t hi = lo + a.bucket_len < a.d ? lo + a.bucket_len : a.d;
  const float* g = a.g + (int64_t)m * a.g_stride;
  LevelShape shape = first_shape();
  if (t == 0) lds.ranges.lo[0] = 0u;
  ScanResult result = kScanGiveUp;
  for (int level = 0; level < kLevels; ++level) {
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) hist[i * kScanThreads + t] = 0ull;
    __syncthreads();
    if (level == 0) {
      for_each_pattern(g, lo, hi, kScanThreads, [&](uint32_t raw) { add_first(hist, raw); });
    } else {
      const Envelope env = envelope_of(shape, lds.ranges.lo);
      for_each_pattern(g, lo, hi, kScanThreads,
                       [&](uint32_t raw) { add_in_ranges(hist, shape, lds.ranges.lo, env, raw); });
    }
    __syncthreads();
    uint32_t c[kPerThread];
    uint64_t off[kPerThread];
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const unsigned long long h = hist[kPerThread * t + i];
      c[i] = (uint32_t)(h >> kCountShift);
      off[i] = h & ((1ull << kCountShift) - 1ull);
    }
    result = scan_level(&shape, level == 0, c, off, lds);
    if (result != kScanRefine) break;
  }
  if (t == 0)
    a.thresholds[(int64_t)m * a.scale_stride + k] =
        result == kScanDone ? __uint_as_float(lds.threshold_bits) : kOpenMark;
}

// ---- longer buckets: the levels are launches, the histogram lies in global memory -----------------

constexpr int kChunkTiles = 32;                          // tiles of one bucket per work-group
constexpr int kHistThreads = 512;

struct alignas(256) WideState {
  LevelShape shape;
  int done;
  uint32_t count[kBins];
  unsigned long long offset[kBins];
  LevelRanges ranges;
};

__global__ __launch_bounds__(kScanThreads) void exact_wide_init_kernel(WideArgs a) {
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + blockIdx.x;
  for (int i = threadIdx.x; i < kBins; i += kScanThreads) { st->count[i] = 0u; st->offset[i] = 0ull; }
  if (threadIdx.x == 0) { st->shape = first_shape(); st->done = 0; st->ranges.lo[0] = 0u; }
}

// One chunk's magnitudes into the level's histogram: LDS first, filled bins added to global memory.
// Bound by the read of the gradient (4 bytes per component and level).
template <bool FIRST>
__global__ __launch_bounds__(kHistThreads) void exact_wide_hist_kernel(WideArgs a, int64_t chunks) {
  __shared__ unsigned long long hist[kBins];
  __shared__ uint32_t lo_of[kRanges];
  const int64_t k = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + k;
  if (st->done) return;
  const int t = threadIdx.x;
  const LevelShape shape = st->shape;
  for (int i = t; i < kBins; i += kHistThreads) hist[i] = 0ull;
  if (!FIRST) {
    for (int i = t; i < shape.nr; i += kHistThreads) lo_of[i] = st->ranges.lo[i];
  }
  __syncthreads();
  const int64_t bucket_lo = k * a.bucket_len;
  const int64_t bucket_hi = bucket_lo + a.bucket_len < a.d ? bucket_lo + a.bucket_len : a.d;
  const int64_t lo = bucket_lo + chunk * (int64_t)(kChunkTiles * kTile);
  const int64_t end = lo + kChunkTiles * kTile;
  const int64_t hi = end < bucket_hi ? end : bucket_hi;
  const float* g = a.g + (int64_t)(a.m0 + (int)blockIdx.y) * a.g_stride;
  if (FIRST) {
    for_each_pattern(g, lo, hi, kHistThreads, [&](uint32_t raw) { add_first(hist, raw); });
  } else {
    const Envelope env = envelope_of(shape, lo_of);
    for_each_pattern(g, lo, hi, kHistThreads, [&](uint32_t raw) { add_in_ranges(hist, shape, lo_of, env, raw); });
  }
  __syncthreads();
  for (int b = t; b < kBins; b += kHistThreads) {
    const unsigned long long h = hist[b];
    if (h) {
      atomicAdd(&st->count[b], (uint32_t)(h >> kCountShift));
      atomicAdd(&st->offset[b], h & ((1ull << kCountShift) - 1ull));
    }
  }
}

__global__ __launch_bounds__(kScanThreads) void exact_wide_scan_kernel(WideArgs a, int level) {
  __shared__ ScanLds lds;
  __shared__ LevelShape shape_out;
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + blockIdx.x;
  if (st->done) return;
  const int t = threadIdx.x;
  LevelShape shape = st->shape;
  for (int i = t; i < shape.nr; i += kScanThreads) {
    lds.ranges.lo[i] = st->ranges.lo[i];
    if (level) {
      lds.ranges.count_before[i] = st->ranges.count_before[i];
      lds.ranges.sum_before[i] = st->ranges.sum_before[i];
    }
  }
  uint32_t c[kPerThread];
  uint64_t off[kPerThread];
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    const int b = kPerThread * t + i;
    c[i] = st->count[b];
    off[i] = st->offset[b];
    if (c[i]) { st->count[b] = 0u; st->offset[b] = 0ull; }        // clear for the next level
  }
  __syncthreads();
  ScanResult result = scan_level(&shape, level == 0, c, off, lds);
  if (result == kScanRefine && level + 1 < kLevels) {
    for (int i = t; i < shape.nr; i += kScanThreads) {
      st->ranges.lo[i] = lds.ranges.lo[i];
      st->ranges.count_before[i] = lds.ranges.count_before[i];
      st->ranges.sum_before[i] = lds.ranges.sum_before[i];
    }
    if (t == 0) st->shape = shape;
  } else if (t == 0) {
    st->done = 1;
    a.thresholds[(int64_t)(a.m0 + (int)blockIdx.y) * a.scale_stride + blockIdx.x] =
        result == kScanDone ? __uint_as_float(lds.threshold_bits) : kOpenMark;
  }
}

// ---- what is still open: a plain sort by one work-group -------------------------------------------
//
// One work-group per bucket looks at its M thresholds; for a worker whose bucket is still marked it
// sorts the magnitudes (descending, four stable passes of eight bits between two key arrays) and
// walks the objective.  Only for inputs built to defeat the levels: an objective that is the same
// number for thousands of cuts to 1e-11.  Some 6 ns per component and worker, a cliff: 2^16 components
// 0.53 ms, 2^22 23.8 ms, where a device-wide sort of every gradient took 0.08 and 0.23 (256 threads, eight
// passes of four bits, each counted on its own: 1.23 and 117 ms).  Chip-wide passes would be launches that
// every call pays for.

__device__ __forceinline__ uint32_t sort_key(uint32_t raw) { return 0x7fffffffu - (raw & 0x7fffffffu); }

__global__ __launch_bounds__(kScanThreads) void exact_sort_open_kernel(WideArgs a, int M) {
  constexpr int kDigitBits = 8, kDigits = 1 << kDigitBits, kPasses = 4, kKeys = 16, kChunk = kScanThreads * kKeys,
                kRun = 8;
  __shared__ uint32_t digit_base[kPasses][kDigits];
  __shared__ uint32_t digit_of_wave[kScanWaves][kDigits];
  __shared__ uint32_t lds_u[kScanWaves];
  __shared__ double lds_d[kScanWaves];
  __shared__ double lds_o[kScanWaves];
  __shared__ long long lds_k[kScanWaves];
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  const int64_t k = blockIdx.x, lo = k * a.bucket_len;
  const int64_t n = (lo + a.bucket_len < a.d ? lo + a.bucket_len : a.d) - lo;
  bool open = false;                                     // any worker's, all looked at together
  for (int m = t; m < M; m += kScanThreads) open |= a.thresholds[(int64_t)m * a.scale_stride + k] == kOpenMark;
  if (!__syncthreads_or(open)) return;
  uint32_t* const keys0 = a.sort_keys + lo;
  uint32_t* const keys1 = a.sort_keys + a.d + lo;
  for (int m = 0; m < M; ++m) {
    float* thr = a.thresholds + (int64_t)m * a.scale_stride + k;
    if (*thr != kOpenMark) continue;                     // the same value for every thread
    const uint32_t* g = reinterpret_cast<const uint32_t*>(a.g + (int64_t)m * a.g_stride + lo);
    for (int i = t; i < kPasses * kDigits; i += kScanThreads) digit_base[i / kDigits][i % kDigits] = 0u;
    __syncthreads();
    for (int64_t i = t; i < n; i += kScanThreads) {      // the digits of all passes are counted at once
      const uint32_t key = sort_key(g[i]);
      keys0[i] = key;
#pragma unroll
      for (int p = 0; p < kPasses; ++p) atomicAdd(&digit_base[p][(key >> (kDigitBits * p)) & (kDigits - 1)], 1u);
    }
    __syncthreads();
    for (int p = 0; p < kPasses; ++p) {                  // counts -> places of the first key of each digit
      uint32_t total;
      const uint32_t first = scan_exclusive(t < kDigits ? digit_base[p][t] : 0u, lds_u, &total);
      if (t < kDigits) digit_base[p][t] = first;
    }
    __syncthreads();
    for (int pass = 0; pass < kPasses; ++pass) {
      const uint32_t* src = pass & 1 ? keys1 : keys0;
      uint32_t* dst = pass & 1 ? keys0 : keys1;
      for (int64_t i0 = 0; i0 < n; i0 += kChunk) {
        // a wave's keys are 1024 consecutive ones, 64 at a time, so that equal digits keep their order
        uint32_t key[kKeys], at[kKeys];
        for (int i = t; i < kScanWaves * kDigits; i += kScanThreads) digit_of_wave[i / kDigits][i % kDigits] = 0u;
#pragma unroll
        for (int j = 0; j < kKeys; ++j) {
          const int64_t i = i0 + wave * (kWave * kKeys) + j * kWave + lane;
          key[j] = i < n ? src[i] : 0u;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kKeys; ++j) {
          const bool live = i0 + wave * (kWave * kKeys) + j * kWave + lane < n;
          const uint32_t digit = (key[j] >> (kDigitBits * pass)) & (kDigits - 1);
          uint64_t same = __ballot(live);
#pragma unroll
          for (int q = 0; q < kDigitBits; ++q) {
            const uint64_t ones = __ballot((digit >> q) & 1u);
            same &= (digit >> q) & 1u ? ones : ~ones;
          }
          const uint32_t rank = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
          at[j] = live ? digit_of_wave[wave][digit] + rank : 0xffffffffu;
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          if (live && rank == 0u) digit_of_wave[wave][digit] += (uint32_t)__popcll(same);
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        if (t < kDigits) {                               // places of the waves' digits in the output
          uint32_t run = digit_base[pass][t];
          for (int w = 0; w < kScanWaves; ++w) { const uint32_t v = digit_of_wave[w][t]; digit_of_wave[w][t] = run; run += v; }
          digit_base[pass][t] = run;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kKeys; ++j)
          if (at[j] != 0xffffffffu) dst[digit_of_wave[wave][(key[j] >> (kDigitBits * pass)) & (kDigits - 1)] + at[j]] = key[j];
        __syncthreads();
      }
    }
    // keys0 holds the magnitudes in descending order: objective of every cut
    double best = -1.0, running = 0.0;
    long long best_k = 0;
    for (int64_t i0 = 0; i0 < n; i0 += kScanThreads * kRun) {
      double v[kRun], sum = 0.0;
      uint32_t key[kRun + 1];
#pragma unroll
      for (int j = 0; j <= kRun; ++j) {
        const int64_t i = i0 + (int64_t)t * kRun + j;
        key[j] = i < n ? keys0[i] : 0x7fffffffu;         // past the end: magnitude 0
      }
#pragma unroll
      for (int j = 0; j < kRun; ++j) { v[j] = (double)__uint_as_float(0x7fffffffu - key[j]); sum += v[j]; }
      double incl = sum;
      for (int o = 1; o < kWave; o <<= 1) {
        const double p = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += p;
      }
      __syncthreads();
      if (lane == kWave - 1) lds_d[wave] = incl;
      __syncthreads();
      double before = running, total = 0.0;
      for (int w = 0; w < kScanWaves; ++w) { if (w < wave) before += lds_d[w]; total += lds_d[w]; }
      const double left = __shfl_up(incl, 1, kWave);
      before += lane ? left : 0.0;
#pragma unroll
      for (int j = 0; j < kRun; ++j) {
        before += v[j];
        const int64_t kk = i0 + (int64_t)t * kRun + j + 1;
        if (kk <= n && v[j] > 0.0 && key[j + 1] != key[j]) {
          const double obj = before * before / (double)kk;
          if (obj > best) { best = obj; best_k = kk; }
        }
      }
      running += total;
    }
    for (int o = 1; o < kWave; o <<= 1) {
      const double b2 = __shfl_xor(best, o, kWave);
      const long long k2 = __shfl_xor(best_k, o, kWave);
      if (b2 > best || (b2 == best && k2 < best_k)) { best = b2; best_k = k2; }
    }
    if (lane == 0) { lds_o[wave] = best; lds_k[wave] = best_k; }
    __syncthreads();
    if (t == 0) {
      for (int w = 0; w < kScanWaves; ++w)
        if (lds_o[w] > best || (lds_o[w] == best && lds_k[w] < best_k)) { best = lds_o[w]; best_k = lds_k[w]; }
      *thr = best >= 0.0 && best_k < n ? __uint_as_float(0x7fffffffu - keys0[best_k]) : 0.0f;
    }
    __syncthreads();                                     // the next worker reuses keys and LDS
  }
}

// ---- host side ---------------------------------------------------------------------------------

static inline size_t xalign(size_t v) { return (v + 255) & ~size_t(255); }

static bool bucket_spans_tiles(const qa_layout* L) {
  return L->bucket == 0 ? tiles_of(L->d) > 1 : L->bucket > kTile;
}

// Bytes this file's passes need beyond the quantizer's own workspace: two arrays of keys for the sort of
// what the levels leave open, which share their place with the levels' state (some 100 KiB per
// bucket and worker; workers are taken in groups that fit).
size_t exact_wide_workspace_bytes(const qa_layout* L) {
  if (!bucket_spans_tiles(L)) return 0;
  const size_t d = (size_t)L->d, nt = (size_t)tiles_of(L->d);
  return xalign(d * 8) + 4 * xalign(nt * 8) + xalign(d * 8 + d + (size_t(4) << 20));
}

int exact_thresholds_wide(const qa_layout* L, const float* g, int64_t g_stride, float* thresholds,
                          void* ws, size_t ws_bytes, hipStream_t stream) {
  if (!bucket_spans_tiles(L)) return QA_ERR_INVALID_ARG;
  if (L->d >= (int64_t(1) << 32)) return QA_ERR_TOO_LARGE;
  if (!ws || ws_bytes < exact_wide_workspace_bytes(L) || !aligned(ws, 256)) return QA_ERR_WORKSPACE;
  WideArgs a{};
  a.g = g; a.g_stride = g_stride; a.d = L->d;
  a.bucket_len = L->bucket ? L->bucket : L->d;
  a.nb = buckets_of(L->d, L->bucket);
  a.thresholds = thresholds; a.scale_stride = L->scale_stride;
  a.state = static_cast<char*>(ws);
  a.sort_keys = static_cast<uint32_t*>(ws);
  const int64_t longest = a.bucket_len < L->d ? a.bucket_len : L->d;
  if (longest <= kResidentMost) {
    hipLaunchKernelGGL(exact_resident_kernel, dim3((unsigned)a.nb, (unsigned)L->M), dim3(kScanThreads), 0, stream, a);
  } else {
    const int64_t chunks = (longest + kChunkTiles * kTile - 1) / (kChunkTiles * kTile);
    const int64_t fit = (int64_t)(ws_bytes / (sizeof(WideState) * (size_t)a.nb));
    if (fit < 1 || a.nb * chunks > 0x7fffffffLL) return QA_ERR_WORKSPACE;
    for (int64_t m0 = 0; m0 < L->M; m0 += fit) {
      const unsigned here = (unsigned)(L->M - m0 < fit ? L->M - m0 : fit);
      a.m0 = (int)m0;
      const dim3 pairs((unsigned)a.nb, here), parts((unsigned)(a.nb * chunks), here);
      hipLaunchKernelGGL(exact_wide_init_kernel, pairs, dim3(kScanThreads), 0, stream, a);
      for (int level = 0; level < kLevels; ++level) {
        if (level == 0)
          hipLaunchKernelGGL(exact_wide_hist_kernel<true>, parts, dim3(kHistThreads), 0, stream, a, chunks);
        else
          hipLaunchKernelGGL(exact_wide_hist_kernel<false>, parts, dim3(kHistThreads), 0, stream, a, chunks);
        hipLaunchKernelGGL(exact_wide_scan_kernel, pairs, dim3(kScanThreads), 0, stream, a, level);
      }
    }
  }
  hipLaunchKernelGGL(exact_sort_open_kernel, dim3((unsigned)a.nb), dim3(kScanThreads), 0, stream, a, (int)L->M);
  return launch_status();
}

}  // namespace qa
