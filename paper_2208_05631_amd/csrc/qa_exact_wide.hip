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
// A smooth distribution leaves 2-4 bins per level: three levels, i.e. three reads of the gradient and one for the
// codes; long buckets of such a distribution take one read (below).
// Every sum is formed in binary64 from exact parts; candidates whose objectives agree to binary64
// rounding may be resolved differently from a strictly sequential summation (likely only beyond some
// 1e7 components per bucket; both kept sets are then optimal to that resolution).  A bucket that
// more than 2048 bins or five levels leave open (an objective constructed to be flat) is sorted by one
// work-group behind the levels.  Infinite members are kept alone, a NaN gives the threshold 0.
//
// Thresholds and codes, us, levels as launches with a scan launch each and two launches for the codes -> now:
//   one read, 2^26 x 4 Gaussian / 5 %-dense Laplace / 10 %-dense Student-t components, one scale per vector:
//     844 797 803 -> 308 310 328 (213 of it the read at 5.4 TB/s); 2^24 x 4 264 230 235 -> 126 138 148
//   levels, Gaussian components: 10^6 x 8 150 -> 87, 100003 119 -> 64; buckets of 2^18, 2^26 x 4 967 -> 857, 2^24 x 4 272 -> 259
//   where the sample is in vain: Cauchy components 2^26 x 4 772 -> 756, 2^24 x 4 221 -> 232, 2^22 x 8 138 -> 169, 2^26 x 4
//     in buckets of 2^21 778 -> 874; ternary 2^26 x 4 2036 -> 2090.  One component 10^9 times as large as the others, which the
//     sample misses and the proof does not allow (the gradient is read once more): 2^26 x 4 775 -> 755, 2^22 x 8 138 -> 178
//   up to 65536 components, a work-group per bucket: 2^26 x 4 in buckets of 65536 1091 -> 972, of 8192 4583 -> 4120
//     (bound by the scans, some 8 us per level and work-group)
#include "qa_common.h"
#include "qa_exact_window.h"

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
  uint32_t threshold_bits, kept_count;                   // kScanDone of single patterns: what is kept
  double kept_sum;
};

__device__ __forceinline__ uint32_t wave_scan(uint32_t v) { return wave_scan_u32(v); }
__device__ __forceinline__ double wave_scan(double v) { return wave_scan_f64(v); }
// sum over the threads before this one; *total = over all
template <typename T>
__device__ __forceinline__ T scan_exclusive(T v, T* lds, T* total) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const T incl = wave_scan(v);
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

// num / den to a few units in the last place of binary64, a fifth of the division's instructions: for objectives
// that are only compared with some 1e-11 to spare.
__device__ __forceinline__ double quick_ratio(double num, double den) {
  double y = __builtin_amdgcn_rcp(den);
  y = fma(fma(-den, y, 1.0), y, y);
  y = fma(fma(-den, y, 1.0), y, y);
  return num * y;
}
__device__ __forceinline__ double sum_of_bin(uint32_t c, uint64_t off, uint32_t low) {
  return c ? fma((double)off, ulp_of(low), (double)c * (double)__uint_as_float(low)) : 0.0;
}

// c, off: count and offset sum of this thread's bins 4 t .. 4 t + 3.  kScanDone: lds.threshold_bits
// holds the threshold; kScanRefine: *shape and lds.ranges are the next level's.  Work-group uniform.
// One work-group per bucket: bound by its instructions (16 waves on four SIMDs), so no division but at the last level
// (10 us a level with two per bin and sums by shuffles, 7 so).
__device__ __forceinline__ ScanResult scan_level(LevelShape* shape, bool first, const uint32_t (&c)[kPerThread],
                                                 const uint64_t (&off)[kPerThread], ScanLds& lds) {
  const LevelShape s = *shape;
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  const int nbins = s.nr << s.sub;
  uint32_t low[kPerThread], cnt = 0;
  double sum[kPerThread], mine = 0.0;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    low[i] = kPerThread * t + i < nbins ? lower_end(s, lds.ranges.lo, kPerThread * t + i) : 0u;
    sum[i] = sum_of_bin(c[i], off[i], low[i]);
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
  const uint32_t k_start = scan_exclusive(cnt, lds.wave_u, &total_cnt);
  const double s_start = scan_exclusive(mine, lds.wave_f, &total_sum);
  if (total_cnt == 0) return kScanDone;                  // nothing but zeros
  // what lies before a range in this scan is replaced by what lies above it in the bucket
  if (!first) {
    uint32_t k_at = k_start;
    double s_at = s_start;
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
  // f(i, count and sum above the bin) for this thread's filled bins
  const auto for_filled = [&](auto f) {
    uint32_t k_run = k_start;
    double s_run = s_start;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i)
      if (c[i]) {
        const int r = (kPerThread * t + i) >> s.sub;
        f(i, first ? k_run : k_run + lds.ranges.count_before[r], first ? s_run : s_run + lds.ranges.sum_before[r]);
        k_run += c[i];
        s_run += sum[i];
      }
  };
  double best = -1.0;
  uint32_t best_k = 0;
  int best_pos = -1;
  for_filled([&](int i, uint32_t k_before, double s_before) {
    const double s1 = s_before + sum[i], k1 = (double)(k_before + c[i]);
    const double edge = s.shift == 0 ? s1 * s1 / k1 : quick_ratio(s1 * s1, k1);
    if (edge > best) { best = edge; best_k = k_before + c[i]; best_pos = kPerThread * t + i; }
  });
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
  const double bins = (double)(1u << s.shift), per_bin = 1.0 / bins;
  for_filled([&](int i, uint32_t k_before, double s_before) {
    const double s1 = s_before + sum[i], j = (double)off[i] * per_bin;
    const double s_in = fma(j, fma(ulp_of(low[i]), bins, (double)__uint_as_float(low[i])), s_before);
    if (s1 * s1 >= bar * (double)(k_before + c[i]) ||
        (c[i] > 1 && off[i] != 0 && s.shift > 0 && s_in * s_in >= bar * ((double)k_before + j)))
      survives |= 1u << i;
    last = kPerThread * t + i + 1;
    if (last == best_pos + 1) { lds.kept_count = best_k; lds.kept_sum = s1; }
  });
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
  // this level's ranges are read for the last time before any is written
  uint32_t count[kPerThread];
  double above[kPerThread];
  for_filled([&](int i, uint32_t k_before, double s_before) { count[i] = k_before; above[i] = s_before; });
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kPerThread; ++i)
    if ((keep >> i) & 1u) {
      lds.ranges.lo[at] = low[i];
      lds.ranges.count_before[at] = count[i];
      lds.ranges.sum_before[at] = above[i];
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
  float* scales;
  int64_t scale_stride;
  uint32_t* codes;
  int64_t code_stride;
  double* part_sum;                                      // [m of this launch][bucket][chunk]
  uint32_t* part_cnt;
  int m0;                                                // first worker of this launch
  char* state;                                           // per (worker, bucket): see below
  uint32_t* sort_keys;                                   // two arrays of d keys
};

// The bucket (at most 256 KiB) is read from memory once and by the later levels from the caches: kept
// in registers, 64 components per thread, it leaves no room for the scan.  Beyond 65536 the levels
// become launches: a work-group alone would leave the chip idle, and the state of every (bucket,
// worker) has to fit the workspace.
constexpr int kResidentMost = 65536, kComputeUnits = 256;
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

// CROWDED: two work-groups per compute unit, at the price of a scan with spills (2^26 x 4 components, buckets of 65536
// 1041 -> 972 us, of 8192 4230 -> 4120; four buckets of 9001 on their own 40 -> 48).
template <bool CROWDED>
__global__ __launch_bounds__(kScanThreads) __attribute__((amdgpu_waves_per_eu(CROWDED ? 8 : 4))) void exact_resident_kernel(WideArgs a) {
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
//
// Work-groups of 1024 threads take a chunk each (4 to 128 tiles); the one of a bucket that finishes last scans
// the level.  From 512 tiles on (2048 in all workers' buckets) and up to some 30 workers (a list of each has to fit
// the workspace) the bucket is read once in full, like the quantizer's own long buckets:
//
//   sample    level 0 over a quarter of the components, at most 2^20, spread in pieces of 256.  At the optimum the
//             threshold is half the mean of what is kept (adding a to a sum S of k raises S^2 / k as long as
//             a > S / 2k), so the place where S - 2 t K changes sign beside the sample's best edge is found
//             between the bins.
//   probe     the same sample against that threshold: S - 2 t K, 256 by 256.  Its slope gives a Newton step,
//             the differences between neighbours the standard error; four of them to either side
//             make the bracket.
//   pass      all components, once: those above the bracket are coded as kept, all others as 0, and those inside
//             are listed with their places.  Its histogram is finest around the bracket.  (With four standard errors
//             to a side the list holds a fifth less than with five, and since what is listed is coded 0 until it is
//             settled, only its kept components, some half, are atomics then: 27.7 to 11.9 us for 2^26 x 4 Gaussian
//             components, the whole call 316 to 303 us; the wider bracket 307.)
//   prove     the scan's bounds show that no cut outside the bracket can be the optimum, or the levels go on over the
//             whole gradient from the bins that survive.
//   level     as above, over the list instead of the gradient; some 250 000 of 2^26 Gaussian components.
//   settle    the codes of the listed components.
//
// The last work-group reads what the others have added by atomic operations of the device's scope, each wave
// having waited for its own before the ticket was drawn; nothing else crosses work-groups inside a launch.

constexpr int kPassThreads = kScanThreads, kPassComponents = kPassThreads * 16;
constexpr int kMostChunkTiles = 128, kBracketedTiles = 32;   // at most 2^19 components: counts and offset sums fit a bin
// Buckets of fewer tiles than this, or than this in all workers' buckets, are not sampled.  Levels alone / with the
// sample, us, Gaussian, 5 %-dense Laplace and Cauchy components (the last ones' optimum keeps too few for a
// bracket): 2^22 x 2 92 75 71 / 87 98 90; 2^23 101 84 79 / 86 99 97; 2^21 x 8 113 94 91 / 91 99 107; 2^22 x 8 164 140 135 /
// 111 116 169; 2^23 x 4 165 141 135 / 99 105 153; 2^24 x 4 259 222 216 / 126 138 232; 2^26 x 4 in buckets of 2^21 808 758
// 740 / 508 502 874.  The second line lies where dense gradients gain; sparse ones gain from four times as many tiles on.
constexpr int64_t kSampledTiles = 512, kSampledInAll = 2048;
constexpr int kUnit = 4 * kWave, kMostOften = 4, kUnitsPerWave = 4, kUnitsPerGroup = kUnitsPerWave * kScanWaves;
constexpr int kMostUnits = kRanges / 2 * kUnitsPerWave;   // two sums of each wave in LevelRanges::sum_before
constexpr int kProofBins = 2048, kProofPerThread = kProofBins / kScanThreads;
constexpr int kFarAbove = 512, kFarBelow = kProofBins - kNearBins - kMostNear - kFarAbove;
constexpr int kStage = 4096;                             // components of a chunk inside the bracket, at most
constexpr double kMostOpen = 0.015;                      // share of the components inside the bracket
constexpr int kListGroups = 64;                          // work-groups of a bucket that walk its list

enum WideMode { kWholeGradient = 0, kBracketed = 1, kListed = 2 };

struct alignas(256) WideState {
  LevelShape shape;
  int first;                                             // level 0 comes next
  int mode, done;
  uint32_t ticket;
  float guess;                                           // threshold that the sample's histogram gives, 0 if none
  // around the bracket [below, above): near0 = first of the bins of 2^18 that are divided into 2^near_shift
  uint32_t near0, near_shift, below, above;
  uint32_t listed, list_failed;
  uint32_t kept, around;                                 // of the probe
  uint32_t count[kBins];
  unsigned long long offset[kBins];
  LevelRanges ranges;                                    // before the first level: sum_before holds the probe's tiles
};

struct WideList {
  uint2* entries;                                        // [pair][capacity]: place in the bucket, pattern
  uint32_t capacity;
};

template <typename T>
__device__ __forceinline__ T device_load(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void device_store(T* p, T v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Whether this work-group is the last of n to arrive; every wave's atomic operations have reached memory.
__device__ __forceinline__ bool arrives_last(uint32_t* ticket, uint32_t n, uint32_t* lds) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    *lds = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1u ? 1u : 0u;
  __syncthreads();
  return *lds != 0u;
}

__global__ __launch_bounds__(kScanThreads) void exact_wide_init_kernel(WideArgs a) {
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + blockIdx.x;
  for (int i = threadIdx.x; i < kBins; i += kScanThreads) { st->count[i] = 0u; st->offset[i] = 0ull; }
  if (threadIdx.x == 0) {
    st->shape = first_shape();
    st->first = 1;
    st->mode = kWholeGradient;
    st->done = 0;
    st->ticket = 0u;
    st->guess = 0.0f;
    st->listed = st->list_failed = st->kept = st->around = 0u;
    st->ranges.lo[0] = 0u;
  }
}

// bins of the work-group -> the bucket's
template <int N>
__device__ __forceinline__ void flush_bins(const unsigned long long* hist, WideState* st) {
  for (int b = threadIdx.x; b < N; b += kPassThreads) {
    const unsigned long long h = hist[b];
    if (h) {
      atomicAdd(&st->count[b], (uint32_t)(h >> kCountShift));
      const unsigned long long o = h & ((1ull << kCountShift) - 1ull);
      if (o) atomicAdd(&st->offset[b], o);
    }
  }
}

// the bucket's bins -> bins `at` of this thread; they are cleared for the next level
template <int N>
__device__ __forceinline__ void take_bins(WideState* st, const int (&at)[N], uint32_t (&c)[N], uint64_t (&off)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) { c[i] = device_load(&st->count[at[i]]); off[i] = device_load(&st->offset[at[i]]); }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (c[i]) { st->count[at[i]] = 0u; st->offset[at[i]] = 0ull; }
}

// The sample: units of 256 consecutive components (a KiB), one of every `every`, not always the same of its group: every
// fourth (kMostOften), or fewer, so that a bucket has kMostUnits of them at most; a wave takes kUnitsPerWave.
struct SampleArgs {
  int64_t every;                                         // one unit of so many
  int units, groups;                                     // of a full bucket; work-groups per bucket
};
// units of bucket k
__device__ __forceinline__ int units_of(const WideArgs& a, const SampleArgs& sa, int64_t k) {
  const int64_t all = (a.d - k * a.bucket_len) / kUnit / sa.every;
  return all < sa.units ? (int)all : sa.units;
}
// this lane's four components of unit i of n, zeros beyond
__device__ __forceinline__ uint4 load_unit(const float* g, const SampleArgs& sa, int64_t i, int n) {
  const int64_t unit = i * sa.every + (i * 29) % sa.every;
  return i < n ? *reinterpret_cast<const uint4*>(g + unit * kUnit + 4 * (threadIdx.x % kWave)) : make_uint4(0, 0, 0, 0);
}

__global__ __launch_bounds__(kPassThreads) void exact_wide_sample_kernel(WideArgs a, SampleArgs sa) {
  __shared__ union { unsigned long long hist[kBins]; ScanLds scan; } lds;
  __shared__ uint32_t last;
  __shared__ float guess;
  const int64_t k = blockIdx.x / sa.groups, part = blockIdx.x % sa.groups;
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + k;
  const int t = threadIdx.x, n = units_of(a, sa, k);
  const float* g = a.g + (int64_t)(a.m0 + (int)blockIdx.y) * a.g_stride + k * a.bucket_len;
  const int64_t i0 = part * kUnitsPerGroup + t / kWave * kUnitsPerWave;
  for (int i = t; i < kBins; i += kPassThreads) lds.hist[i] = 0ull;
  __syncthreads();
  uint4 q[kUnitsPerWave];
#pragma unroll
  for (int j = 0; j < kUnitsPerWave; ++j) q[j] = load_unit(g, sa, i0 + j, n);
#pragma unroll
  for (int j = 0; j < kUnitsPerWave; ++j) {
    add_first(lds.hist, q[j].x); add_first(lds.hist, q[j].y); add_first(lds.hist, q[j].z); add_first(lds.hist, q[j].w);
  }
  __syncthreads();
  flush_bins<kBins>(lds.hist, st);
  if (!arrives_last(&st->ticket, (uint32_t)sa.groups, &last)) return;
  const LevelShape s = first_shape();
  const uint32_t zero = 0u;
  uint32_t c[kPerThread], low[kPerThread], cnt = 0;
  uint64_t off[kPerThread];
  double sum[kPerThread], mine = 0.0;
  int at[kPerThread];
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) at[i] = kPerThread * t + i;
  take_bins(st, at, c, off);
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) {
    low[i] = lower_end(s, &zero, at[i]);
    sum[i] = sum_of_bin(c[i], off[i], low[i]);
    cnt += c[i];
    mine += sum[i];
  }
  uint32_t all_cnt;
  double all_sum;
  const uint32_t k_before = scan_exclusive(cnt, lds.scan.wave_u, &all_cnt);
  const double s_before = scan_exclusive(mine, lds.scan.wave_f, &all_sum);
  double best = -1.0;
  int best_pos = 0;
  double k1 = (double)k_before, s1 = s_before;
#pragma unroll
  for (int i = 0; i < kPerThread; ++i)
    if (c[i]) {
      k1 += (double)c[i];
      s1 += sum[i];
      const double edge = quick_ratio(s1 * s1, k1);
      if (edge > best) { best = edge; best_pos = at[i]; }
    }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double ob = __shfl_xor(best, o, kWave);
    const int op = __shfl_xor(best_pos, o, kWave);
    if (ob > best || (ob == best && op < best_pos)) { best = ob; best_pos = op; }
  }
  __syncthreads();
  if (t % kWave == 0) { lds.scan.best_obj[t / kWave] = best; lds.scan.best_pos[t / kWave] = best_pos; }
  if (t == 0) guess = 0.0f;
  __syncthreads();
  best = lds.scan.best_obj[0]; best_pos = lds.scan.best_pos[0];
  for (int w = 1; w < kScanWaves; ++w)
    if (lds.scan.best_obj[w] > best) { best = lds.scan.best_obj[w]; best_pos = lds.scan.best_pos[w]; }
  // S - 2 t K at both ends of the bins beside the best edge
  if (best > 0.0 && best < 1e300 && kPerThread * t <= best_pos + 1 && kPerThread * t + kPerThread > best_pos - 1) {
    k1 = (double)k_before; s1 = s_before;
#pragma unroll
    for (int i = 0; i < kPerThread; ++i) {
      const double L = (double)__uint_as_float(low[i]), H = L + ulp_of(low[i]) * (double)(1u << kFirstShift);
      const double above = s1 - 2.0 * H * k1;
      k1 += (double)c[i];
      s1 += sum[i];
      const double below = s1 - 2.0 * L * k1;
      if (c[i] && at[i] >= best_pos - 1 && at[i] <= best_pos + 1 && above < 0.0 && below >= 0.0)
        guess = (float)(L + (H - L) * (below / (below - above)));
    }
  }
  __syncthreads();
  if (t == 0) { st->guess = guess; st->ticket = 0u; }
}

__global__ __launch_bounds__(kPassThreads) void exact_wide_probe_kernel(WideArgs a, SampleArgs sa) {
  __shared__ double wave_s[kScanWaves], wave_d[kScanWaves];
  __shared__ uint32_t wave_k[kScanWaves], wave_n[kScanWaves];
  __shared__ uint32_t last;
  const int64_t k = blockIdx.x / sa.groups, part = blockIdx.x % sa.groups;
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + k;
  const float guess = st->guess;
  // (the histogram's bins must lie below the infinities and above the denormals)
  if (!(guess > 1e-25f && guess < 1e30f)) return;
  const int t = threadIdx.x, n = units_of(a, sa, k);
  const float* g = a.g + (int64_t)(a.m0 + (int)blockIdx.y) * a.g_stride + k * a.bucket_len;
  const int64_t i0 = part * kUnitsPerGroup + t / kWave * kUnitsPerWave;
  const float lo = guess * 0.98f, hi = guess * 1.02f;
  const double twice = 2.0 * (double)guess;
  double excess = 0.0, diff = 0.0, previous = 0.0;       // of S - 2 t K; the same in every lane
  uint32_t kept = 0, around = 0;
  uint4 q[kUnitsPerWave];
#pragma unroll
  for (int j = 0; j < kUnitsPerWave; ++j) q[j] = load_unit(g, sa, i0 + j, n);
#pragma unroll
  for (int j = 0; j < kUnitsPerWave; ++j) {
    const uint32_t raw[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
    double u = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = fabsf(__uint_as_float(raw[e]));
      u += x > guess ? (double)x - twice : 0.0;
      kept += (uint32_t)__popcll(__ballot(x > guess));
      around += (uint32_t)__popcll(__ballot(x > lo && x <= hi));
    }
    u = wave_sum_f64(u);
    if (i0 + j < n) {
      excess += u;
      if (j > 0) diff += (u - previous) * (u - previous);
      previous = u;
    }
  }
  const int64_t w = part * kScanWaves + t / kWave;
  if (t % kWave == 0) {
    device_store(&st->ranges.sum_before[2 * w], excess);
    device_store(&st->ranges.sum_before[2 * w + 1], diff);
    wave_k[t / kWave] = kept;
    wave_n[t / kWave] = around;
  }
  __syncthreads();
  if (t == 0) {
    for (int v = 1; v < kScanWaves; ++v) { kept += wave_k[v]; around += wave_n[v]; }
    atomicAdd(&st->kept, kept);
    atomicAdd(&st->around, around);
  }
  if (!arrives_last(&st->ticket, (uint32_t)sa.groups, &last)) return;
  excess = diff = 0.0;
  for (int j = t; j < sa.groups * kScanWaves; j += kPassThreads) {
    excess += device_load(&st->ranges.sum_before[2 * j]);
    diff += device_load(&st->ranges.sum_before[2 * j + 1]);
  }
  excess = wave_sum_f64(excess);
  diff = wave_sum_f64(diff);
  if (t % kWave == 0) { wave_s[t / kWave] = excess; wave_d[t / kWave] = diff; }
  __syncthreads();
  if (t == 0) {
    excess = diff = 0.0;
    for (int v = 0; v < kScanWaves; ++v) { excess += wave_s[v]; diff += wave_d[v]; }
    st->ticket = 0u;
    const double K = (double)device_load(&st->kept), N = (double)device_load(&st->around), t0 = (double)guess;
    const int pairs = n - (n + kUnitsPerWave - 1) / kUnitsPerWave;   // neighbours within a wave
    // d/dt (S - 2 t K) = p t - 2 K with p the number of components per unit of t
    const double slope = 2.0 * K - N / 0.04;
    if (pairs >= 64 && K >= 256.0 && N >= 64.0 && slope > 0.2 * K) {
      const double step = excess / slope;
      const double half = 4.0 * sqrt((double)n * diff / (2.0 * (double)pairs)) / slope + 0.02 * fabs(step) + 1e-4 * t0;
      const double open = N / 0.04 * (2.0 * half / t0) / ((double)n * (double)kUnit);
      if (half < 0.12 * t0 && fabs(step) < 0.05 * t0 && open < kMostOpen) {
        const uint32_t below = __float_as_uint((float)(t0 + step - half)), above = __float_as_uint((float)(t0 + step + half));
        const NearWindow w = near_window(below, __float_as_uint((float)(t0 + step)), above);
        if (w.shift) {
          st->below = below; st->above = above; st->near0 = w.near0; st->near_shift = w.shift;
          st->mode = kBracketed;
        }
      }
    }
  }
}

// The bins of the one pass over a bracketed bucket, ascending: kFarBelow of 2^18 patterns, kNearBins of 2^shift in
// the place of `near` such ones around the bracket, kFarAbove of 2^18.  The number of a bin is that of its 2^18
// plus the near ones that begin before it, two clamps and an addition: inside the near part a number in every
// 2^(18 - shift) + 1 stays unused.  Sums of offsets are relative to the multiple of 2^18 below.
struct NearShape {
  uint32_t near0;
  int near, shift, base;                                 // base: upper bits of the lowest bin
  int reciprocal;                                        // 2^18 / (2^(18 - shift) + 1), rounded up
};
__device__ __forceinline__ NearShape near_shape(const WideState* st) {
  const int shift = (int)st->near_shift;
  const int parts = 1 << (kFarShift - shift);
  return NearShape{st->near0, kNearBins >> (kFarShift - shift), shift, (int)st->near0 - kFarBelow, (1 << 18) / (parts + 1) + 1};
}
// lower end and log2 width of bin `slot`
__device__ __forceinline__ uint32_t bracketed_low(const NearShape& ns, int slot, int* log_width) {
  const int v = slot - kFarBelow, parts = 1 << (kFarShift - ns.shift);
  const int q = v * ns.reciprocal >> 18;                 // v / (parts + 1) for the numbers that are near
  const bool near = v >= 0 && q < ns.near;
  *log_width = near ? ns.shift : kFarShift;
  return near ? ((ns.near0 + (uint32_t)q) << kFarShift) + ((uint32_t)(v - q * (parts + 1)) << ns.shift)
              : (uint32_t)(ns.base + slot - (v < 0 ? 0 : kNearBins)) << kFarShift;
}

// Scan of the one pass.  kListed: no cut outside the bracket can be the optimum, and lds.ranges and *shape are the
// next level's, bins inside the bracket.  kWholeGradient: some can, and the next level's are bins of 2^17
// patterns; or, *restart, the bins do not say enough.  n: components of the bucket.
__device__ __forceinline__ WideMode scan_bracketed(LevelShape* shape, bool* restart, WideState* st, int64_t n, ScanLds& lds) {
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  const NearShape ns = near_shape(st);
  const uint32_t below = st->below, above = st->above;
  const bool complete = st->list_failed == 0u;
  uint32_t c[kProofPerThread], low[kProofPerThread], cnt = 0;
  uint64_t off[kProofPerThread];
  int at[kProofPerThread], wide[kProofPerThread];
  double sum[kProofPerThread], mine = 0.0;
#pragma unroll
  for (int i = 0; i < kProofPerThread; ++i) at[i] = kProofBins - 1 - (kProofPerThread * t + i);
  take_bins(st, at, c, off);
#pragma unroll
  for (int i = 0; i < kProofPerThread; ++i) {
    low[i] = bracketed_low(ns, at[i], &wide[i]);
    off[i] -= (uint64_t)c[i] * (uint64_t)(low[i] & ((1u << kFarShift) - 1u));   // from now on relative to the lower end
    sum[i] = sum_of_bin(c[i], off[i], low[i]);
    cnt += c[i];
    mine += sum[i];
  }
  uint32_t total_cnt;
  double total_sum;
  const uint32_t k_before = scan_exclusive(cnt, lds.wave_u, &total_cnt);
  const double s_before = scan_exclusive(mine, lds.wave_f, &total_sum);
  // the best edge
  double best = -1.0, k1 = (double)k_before, s1 = s_before;
#pragma unroll
  for (int i = 0; i < kProofPerThread; ++i)
    if (c[i]) {
      k1 += (double)c[i];
      s1 += sum[i];
      const double edge = quick_ratio(s1 * s1, k1);
      best = edge > best ? edge : best;
    }
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const double ob = __shfl_xor(best, o, kWave);
    best = ob > best ? ob : best;
  }
  if (lane == 0) lds.best_obj[wave] = best;
  __syncthreads();
  best = lds.best_obj[0];
#pragma unroll
  for (int w = 1; w < kScanWaves; ++w) best = lds.best_obj[w] > best ? lds.best_obj[w] : best;
  const double bar = best * (1.0 - 1e-11);
  uint32_t survives = 0;
  int last = 0;
  k1 = (double)k_before; s1 = s_before;
#pragma unroll
  for (int i = 0; i < kProofPerThread; ++i)
    if (c[i]) {
      const double bins = (double)(1u << wide[i]), j = (double)off[i] * (wide[i] == kFarShift ? 1.0 / (1u << kFarShift) : 1.0 / bins);
      const double s_in = fma(j, fma(ulp_of(low[i]), bins, (double)__uint_as_float(low[i])), s1);
      const bool within = c[i] > 1 && off[i] != 0 && s_in * s_in >= bar * (k1 + j);
      k1 += (double)c[i];
      s1 += sum[i];
      if (within || s1 * s1 >= bar * k1) survives |= 1u << i;
      last = kProofPerThread * t + i + 1;
    }
  lds.survives[t] = (uint8_t)survives;
  int previous = scan_exclusive_max(last, lds.wave_i);   // (barriers inside: survives[] is visible)
  uint32_t keep = 0;
  bool unknown = false, outside = false;
#pragma unroll
  for (int i = 0; i < kProofPerThread; ++i)
    if (c[i]) {
      const int pos = kProofPerThread * t + i, q = previous - 1;
      unknown |= at[i] == kFarBelow + ns.near + kFarAbove - 1 + kNearBins;   // the topmost bin takes all above it too
      const bool follows = q >= 0 && ((lds.survives[q / kProofPerThread] >> (q % kProofPerThread)) & 1u);
      if (((survives >> i) & 1u) || follows) {
        keep |= 1u << i;
        outside |= wide[i] != ns.shift || low[i] < below || low[i] + (1u << ns.shift) > above;
      }
      previous = pos + 1;
    }
  if (t == kScanThreads - 1) {
    // The last filled bin of all: what follows it may be too small for the histogram.  Any j of those add less than
    // j * tiny: (S + j tiny)^2 / (K + j) is convex in j, so its ends bound it.
    const int q = previous - 1;
    unknown |= q < 0 || ((lds.survives[q / kProofPerThread] >> (q % kProofPerThread)) & 1u);
    const double rest = (double)(n - (int64_t)total_cnt), tiny = (double)__uint_as_float((uint32_t)ns.base << kFarShift);
    const double s_all = total_sum + rest * tiny;
    unknown |= !(s_all * s_all < bar * ((double)total_cnt + rest));
  }
  *restart = __syncthreads_or(unknown || !(best > 0.0) || !(best < 1e300)) != 0;
  if (*restart) return kWholeGradient;
  const bool inside = __syncthreads_or(outside) == 0;
  if (!inside) {
    // whole bins of 2^18 patterns, taken at their topmost number
    uint32_t* const wanted = lds.ranges.lo;              // free until the ranges are written
    static_assert(kFarBelow + kMostNear + kFarAbove <= kRanges, "a word for each");
    for (int i = t; i < kRanges; i += kScanThreads) wanted[i] = 0u;
    __syncthreads();
    const int parts = 1 << (kFarShift - ns.shift);
#pragma unroll
    for (int i = 0; i < kProofPerThread; ++i)
      if ((keep >> i) & 1u) wanted[(int)(low[i] >> kFarShift) - ns.base] = 1u;
    __syncthreads();
    keep = 0;
#pragma unroll
    for (int i = 0; i < kProofPerThread; ++i) {
      const int far = (int)(low[i] >> kFarShift) - ns.base;
      const bool head = wide[i] == kFarShift || (low[i] >> ns.shift) % (uint32_t)parts == (uint32_t)parts - 1u;
      // (an unused number reads as the lowest part of the next 2^18)
      if (head && far >= 0 && far < kRanges && wanted[far])
        keep |= 1u << i;
      low[i] &= ~((1u << kFarShift) - 1u);
    }
    __syncthreads();
  }
  uint32_t kept_bins;
  uint32_t to = scan_exclusive((uint32_t)__popc(keep), lds.wave_u, &kept_bins);
  if (kept_bins > (uint32_t)kRanges) { *restart = true; return kWholeGradient; }
  uint32_t k_at = k_before;
  double s_at = s_before;
#pragma unroll
  for (int i = 0; i < kProofPerThread; ++i) {
    if ((keep >> i) & 1u) {
      lds.ranges.lo[to] = low[i];
      lds.ranges.count_before[to] = k_at;
      lds.ranges.sum_before[to] = s_at;
      ++to;
    }
    k_at += c[i];
    s_at += sum[i];
  }
  const int width = inside ? ns.shift : kFarShift;
  int sub = kLogBins - (kept_bins > 1 ? 32 - __clz((int)(kept_bins - 1)) : 0);
  sub = sub < width ? sub : width;
  shape->nr = (int)kept_bins; shape->width = width; shape->sub = sub; shape->shift = width - sub;
  __syncthreads();
  return inside && complete ? kListed : kWholeGradient;
}

// Four groups of four components of this thread: components i0 + 4096 j + 4 t of the bucket's part that ends at hi;
// f(j, raw[4]) for each, in order.
template <typename F>
__device__ __forceinline__ void for_four_groups(const float* g, int64_t i0, int64_t hi, F f) {
  typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
  uintx4 q[4];
  if (i0 + kPassComponents <= hi) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      q[j] = __builtin_nontemporal_load(reinterpret_cast<const uintx4*>(g + i0 + 4 * ((int)threadIdx.x + j * kPassThreads)));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int64_t i = i0 + 4 * ((int)threadIdx.x + j * kPassThreads);
#pragma unroll
      for (int e = 0; e < 4; ++e) q[j][e] = i + e < hi ? __float_as_uint(g[i + e]) : 0u;
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t raw[4] = {q[j].x, q[j].y, q[j].z, q[j].w};
    f(j, raw);
  }
}
// The same thread's code bytes of those four groups -> the word that it stores: word 256 (t & 3) + t / 4 of the
// sixteen thousand components.
__device__ __forceinline__ void add_code_byte(int j, uint32_t byte, uint32_t* mine) {
  const int t = threadIdx.x;
  uint32_t w = byte << (8 * (t & 3));
  w |= (uint32_t)dpp_i32<kDppQuadXor1>((int)w);
  w |= (uint32_t)dpp_i32<kDppQuadXor2>((int)w);
  if ((t & 3) == j) *mine = w;
}

__device__ __forceinline__ int clamp_i32(int v, int lo, int hi) {
  int out;
  asm("v_med3_i32 %0, %1, %2, %3" : "=v"(out) : "v"(v), "v"(lo), "v"(hi));
  return out;
}
// a if the condition is not 0, else b, by bits: a choice among an array's elements must not become an address
__device__ __forceinline__ uint32_t choose(int condition, uint32_t a, uint32_t b) {
  const uint32_t mask = condition ? 0xffffffffu : 0u;
  return (a & mask) | (b & ~mask);
}

// The one pass over a bracketed bucket: its chunk's codes, bins and list.
// Bound by the read of the gradient (4 bytes per component) and close behind it by instructions: 18 per component
// (2^26 x 4: 213 us, 5.4 TB/s; with 30 of them, a branch for the open ones at every component, 320).
__global__ __launch_bounds__(kPassThreads) void exact_wide_bracketed_kernel(WideArgs a, WideList list, int64_t chunks,
                                                                             int chunk_tiles) {
  __shared__ unsigned long long hist[kProofBins];
  __shared__ uint2 stage[kStage];
  __shared__ uint32_t n_stage, base_stage;
  const int64_t k = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int64_t pair = (int64_t)blockIdx.y * a.nb + k;
  WideState* st = reinterpret_cast<WideState*>(a.state) + pair;
  if (st->mode != kBracketed) return;
  const int t = threadIdx.x, m = a.m0 + (int)blockIdx.y;
  const int64_t bucket_lo = k * a.bucket_len, n = a.d - bucket_lo < a.bucket_len ? a.d - bucket_lo : a.bucket_len;
  const float* g = a.g + (int64_t)m * a.g_stride + bucket_lo;
  uint32_t* codes = a.codes + (int64_t)m * a.code_stride + bucket_lo / 16;
  const int64_t lo = chunk * (int64_t)chunk_tiles * kTile;
  const int64_t hi = lo + (int64_t)chunk_tiles * kTile < n ? lo + (int64_t)chunk_tiles * kTile : n;
  const NearShape ns = near_shape(st);
  // patterns are taken relative to `origin`, which puts the near bins' numbers and the lowest bin's together
  const uint32_t origin = (ns.near0 << kFarShift) + ((uint32_t)ns.base << ns.shift);
  const uint32_t open0 = st->below - origin, width = st->above - st->below;
  const int kept0 = (int)(st->above - origin), shift = ns.shift, top = (int)ns.near0 + ns.near + kFarAbove - 1;
  int near_lo = -ns.base, near_hi = kNearBins - ns.base;
  asm volatile("" : "+v"(near_lo), "+v"(near_hi));       // (an instruction takes one scalar operand)
  for (int i = t; i < kProofBins; i += kPassThreads) hist[i] = 0ull;
  if (t == 0) n_stage = 0u;
  __syncthreads();
  for (int64_t i0 = lo; i0 < hi; i0 += kPassComponents) {
    uint32_t mine = 0, fields = 0, raws[4][4];
    for_four_groups(g, i0, hi, [&](int j, const uint32_t (&raw)[4]) {
      uint32_t byte = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        raws[j][e] = raw[e];
        const uint32_t from = (raw[e] & 0x7fffffffu) - origin;
        const int x = (int)((raw[e] >> kFarShift) & ((1u << (31 - kFarShift)) - 1u));
        uint32_t kept = raw[e] >> 30 | 1u, field = from - open0 < width ? 2u : 0u;
        asm("" : "+v"(kept), "+v"(field));               // (selected, not branched to)
        field = (int)from >= kept0 ? kept : field;
        byte |= field << (2 * e);
        const uint32_t slot = (uint32_t)((x < top ? x : top) + clamp_i32((int)from >> shift, near_lo, near_hi));
        if (x >= ns.base)
          atomicAdd(reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(hist) + slot * 8u),
                    (1ull << kCountShift) | (unsigned long long)(raw[e] & ((1u << kFarShift) - 1u)));
      }
      fields |= byte << (8 * j);
      add_code_byte(j, byte, &mine);
    });
    const int64_t word = i0 / 16 + (t & 3) * (kPassThreads / 4) + (t >> 2);
    if (16 * word < hi) codes[word] = mine & (mine << 1 | 0x55555555u);   // 10 -> 00
    for (uint32_t left = (fields >> 1) & ~fields & 0x55555555u; left; left &= left - 1u) {
      const int f = __builtin_ctz(left) >> 1;            // component f % 4 of group f / 4
      uint32_t by[4];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        by[j] = choose(f & 2, choose(f & 1, raws[j][3], raws[j][2]), choose(f & 1, raws[j][1], raws[j][0]));
      const uint32_t raw = choose(f & 8, choose(f & 4, by[3], by[2]), choose(f & 4, by[1], by[0]));
      const uint32_t p = atomicAdd(&n_stage, 1u);
      if (p < (uint32_t)kStage)
        stage[p] = make_uint2((uint32_t)i0 + (uint32_t)(4 * (t + (f >> 2) * kPassThreads) + (f & 3)), raw);
    }
  }
  __syncthreads();
  const uint32_t listed = n_stage;
  if (t == 0) base_stage = listed ? atomicAdd(&st->listed, listed) : 0u;
  flush_bins<kProofBins>(hist, st);
  __syncthreads();
  uint2* entries = list.entries + pair * (int64_t)list.capacity + base_stage;
  if (listed <= (uint32_t)kStage && base_stage <= list.capacity && listed <= list.capacity - base_stage)
    for (uint32_t i = t; i < listed; i += kPassThreads) entries[i] = stage[i];
  else if (t == 0)
    st->list_failed = 1u;
}

// Its scan: the list replaces the gradient, or the next level reads it again, or the levels start from the beginning.
__global__ __launch_bounds__(kScanThreads) void exact_wide_prove_kernel(WideArgs a) {
  __shared__ ScanLds lds;
  const int64_t k = blockIdx.x;
  WideState* st = reinterpret_cast<WideState*>(a.state) + (int64_t)blockIdx.y * a.nb + k;
  if (st->mode != kBracketed) return;
  const int64_t n = a.d - k * a.bucket_len < a.bucket_len ? a.d - k * a.bucket_len : a.bucket_len;
  LevelShape shape;
  bool restart;
  const WideMode mode = scan_bracketed(&shape, &restart, st, n, lds);
  if (!restart) {
    for (int i = threadIdx.x; i < shape.nr; i += kScanThreads) {
      st->ranges.lo[i] = lds.ranges.lo[i];
      st->ranges.count_before[i] = lds.ranges.count_before[i];
      st->ranges.sum_before[i] = lds.ranges.sum_before[i];
    }
  }
  if (threadIdx.x == 0) {
    st->mode = mode;
    if (!restart) { st->shape = shape; st->first = 0; }
    else st->ranges.lo[0] = 0u;
  }
}

// One level of a bucket: its chunk's magnitudes, or its part of the list, into the histogram, LDS first, filled
// bins added to global memory; the last work-group scans.
// Bound by the read of the gradient (4 bytes per component) and, in short buckets, by the scan.  CROWDED: two
// work-groups per compute unit, at the price of a scan with spills, where there are more work-groups than units
// (2^26 x 4, buckets of 2^18 951 -> 857 us, ternary components 2145 -> 2098); with a unit for each the spills only
// cost (100003 67.5 -> 64.2, 10^6 x 8 91 -> 87).
template <bool CROWDED>
__global__ __launch_bounds__(kPassThreads) __attribute__((amdgpu_waves_per_eu(CROWDED ? 8 : 4))) void exact_wide_level_kernel(WideArgs a, WideList list, int64_t chunks,
                                                                         int chunk_tiles, int last_level) {
  __shared__ union {
    struct { unsigned long long hist[kBins]; uint32_t lo_of[kRanges]; } pass;
    ScanLds scan;
  } lds;
  __shared__ uint32_t last;
  const int64_t k = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int64_t pair = (int64_t)blockIdx.y * a.nb + k;
  WideState* st = reinterpret_cast<WideState*>(a.state) + pair;
  if (st->done) return;
  const int t = threadIdx.x, m = a.m0 + (int)blockIdx.y;
  const bool first = st->first != 0, in_list = st->mode == kListed;
  uint32_t arrivals = (uint32_t)chunks;
  if (in_list) {
    if (chunk >= kListGroups) return;
    if (arrivals > (uint32_t)kListGroups) arrivals = (uint32_t)kListGroups;
  }
  const int64_t bucket_lo = k * a.bucket_len, n = a.d - bucket_lo < a.bucket_len ? a.d - bucket_lo : a.bucket_len;
  const float* g = a.g + (int64_t)m * a.g_stride + bucket_lo;
  const int64_t lo = chunk * (int64_t)chunk_tiles * kTile;
  const int64_t hi = lo + (int64_t)chunk_tiles * kTile < n ? lo + (int64_t)chunk_tiles * kTile : n;
  unsigned long long* hist = lds.pass.hist;
  LevelShape shape = st->shape;
  for (int i = t; i < kBins; i += kPassThreads) hist[i] = 0ull;
  for (int i = t; i < shape.nr; i += kPassThreads) lds.pass.lo_of[i] = st->ranges.lo[i];
  __syncthreads();
  if (first) {
    for (int64_t i0 = lo; i0 < hi; i0 += kPassComponents)
      for_four_groups(g, i0, hi, [&](int, const uint32_t (&raw)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) add_first(hist, raw[e]);
      });
  } else {
    const Envelope env = envelope_of(shape, lds.pass.lo_of);
    if (in_list) {
      const uint2* entries = list.entries + pair * (int64_t)list.capacity;
      const uint32_t listed = st->listed;
      for (uint32_t i = (uint32_t)chunk * kPassThreads + t; i < listed; i += 4 * arrivals * kPassThreads) {
        uint32_t raw[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) raw[j] = i + j * arrivals * kPassThreads < listed ? entries[i + j * arrivals * kPassThreads].y : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) add_in_ranges(hist, shape, lds.pass.lo_of, env, raw[j]);
      }
    } else {
      for (int64_t i0 = lo; i0 < hi; i0 += kPassComponents)
        for_four_groups(g, i0, hi, [&](int, const uint32_t (&raw)[4]) {
#pragma unroll
          for (int e = 0; e < 4; ++e) add_in_ranges(hist, shape, lds.pass.lo_of, env, raw[e]);
        });
    }
  }
  __syncthreads();
  flush_bins<kBins>(hist, st);
  if (!arrives_last(&st->ticket, arrivals, &last)) return;
  ScanLds& scan = lds.scan;
  for (int i = t; i < shape.nr; i += kPassThreads) {
    scan.ranges.lo[i] = st->ranges.lo[i];
    if (!first) {
      scan.ranges.count_before[i] = st->ranges.count_before[i];
      scan.ranges.sum_before[i] = st->ranges.sum_before[i];
    }
  }
  uint32_t c[kPerThread];
  uint64_t off[kPerThread];
  int at[kPerThread];
#pragma unroll
  for (int i = 0; i < kPerThread; ++i) at[i] = kPerThread * t + i;
  take_bins(st, at, c, off);
  __syncthreads();
  const ScanResult result = scan_level(&shape, first, c, off, scan);
  if (result == kScanRefine && !last_level) {
    for (int i = t; i < shape.nr; i += kPassThreads) {
      st->ranges.lo[i] = scan.ranges.lo[i];
      st->ranges.count_before[i] = scan.ranges.count_before[i];
      st->ranges.sum_before[i] = scan.ranges.sum_before[i];
    }
    if (t == 0) { st->shape = shape; st->first = 0; }
  } else if (t == 0) {
    st->done = 1;
    a.thresholds[(int64_t)m * a.scale_stride + k] = result == kScanDone ? __uint_as_float(scan.threshold_bits) : kOpenMark;
    if (in_list && result == kScanDone)
      a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(scan.kept_sum, scan.kept_count);
  }
  if (t == 0) st->ticket = 0u;
}

// Codes and scale by the threshold: of a listed bucket the open components' (its scale is known), of others all.
__global__ __launch_bounds__(kPassThreads) void exact_wide_codes_kernel(WideArgs a, WideList list, int64_t chunks, int chunk_tiles) {
  __shared__ double lds_d[kScanWaves], lds_c[kScanWaves];
  __shared__ uint32_t lds_u[kScanWaves];
  __shared__ uint32_t last;
  const int64_t k = blockIdx.x / chunks, chunk = blockIdx.x % chunks;
  const int64_t pair = (int64_t)blockIdx.y * a.nb + k;
  WideState* st = reinterpret_cast<WideState*>(a.state) + pair;
  const int t = threadIdx.x, m = a.m0 + (int)blockIdx.y;
  const int64_t bucket_lo = k * a.bucket_len;
  uint32_t* codes = a.codes + (int64_t)m * a.code_stride + bucket_lo / 16;
  const float D = a.thresholds[(int64_t)m * a.scale_stride + k];
  if (st->mode == kListed) {
    const uint2* entries = list.entries + pair * (int64_t)list.capacity;
    const uint32_t listed = st->listed;
    for (uint32_t i = (uint32_t)chunk * kPassThreads + t; i < listed; i += (uint32_t)chunks * kPassThreads) {
      const uint2 e = entries[i];
      const uint32_t code = ternary_field(__uint_as_float(e.y), D);
      if (code) atomicOr(&codes[e.x >> 4], code << (2 * (e.x & 15u)));   // the pass has left 0
    }
    return;
  }
  const float* g = a.g + (int64_t)m * a.g_stride + bucket_lo;
  const int64_t n = a.d - bucket_lo < a.bucket_len ? a.d - bucket_lo : a.bucket_len;
  const int64_t lo = chunk * (int64_t)chunk_tiles * kTile;
  const int64_t hi = lo + (int64_t)chunk_tiles * kTile < n ? lo + (int64_t)chunk_tiles * kTile : n;
  double s = 0.0;
  uint32_t c = 0;
  for (int64_t i0 = lo; i0 < hi; i0 += kPassComponents) {
    uint32_t mine = 0;
    for_four_groups(g, i0, hi, [&](int j, const uint32_t (&raw)[4]) {
      uint32_t byte = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float v = __uint_as_float(raw[e]), av = fabsf(v);
        byte |= ternary_field(v, D) << (2 * e);
        s += av > D ? (double)av : 0.0;
        c += av > D ? 1u : 0u;
      }
      add_code_byte(j, byte, &mine);
    });
    const int64_t word = i0 / 16 + (t & 3) * (kPassThreads / 4) + (t >> 2);
    if (16 * word < hi) codes[word] = mine;
  }
  s = wave_sum_f64(s);
  c = wave_sum_u32(c);
  if (t % kWave == 0) { lds_d[t / kWave] = s; lds_u[t / kWave] = c; }
  __syncthreads();
  const int64_t first_part = pair * chunks;
  if (t == 0) {
    double S = 0.0;
    uint32_t C = 0;
    for (int w = 0; w < kScanWaves; ++w) { S += lds_d[w]; C += lds_u[w]; }
    device_store(&a.part_sum[first_part + chunk], S);
    device_store(&a.part_cnt[first_part + chunk], C);
  }
  if (!arrives_last(&st->ticket, (uint32_t)chunks, &last)) return;
  double S = 0.0, C = 0.0;                               // counts are integers < 2^53: exact in binary64
  for (int64_t i = t; i < chunks; i += kPassThreads) {
    S += device_load(&a.part_sum[first_part + i]);
    C += (double)device_load(&a.part_cnt[first_part + i]);
  }
  S = wave_sum_f64(S);
  C = wave_sum_f64(C);
  if (t % kWave == 0) { lds_d[t / kWave] = S; lds_c[t / kWave] = C; }
  __syncthreads();
  if (t == 0) {
    S = C = 0.0;
    for (int w = 0; w < kScanWaves; ++w) { S += lds_d[w]; C += lds_c[w]; }
    a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(S, (uint64_t)C);
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

__global__ __launch_bounds__(kScanThreads) void exact_sort_open_kernel(WideArgs a, int M) {   // workers m0 .. m0 + M - 1
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
  for (int m = t; m < M; m += kScanThreads)
    open |= a.thresholds[(int64_t)(a.m0 + m) * a.scale_stride + k] == kOpenMark;
  if (!__syncthreads_or(open)) return;
  uint32_t* const keys0 = a.sort_keys + lo;
  uint32_t* const keys1 = a.sort_keys + a.d + lo;
  for (int m = a.m0; m < a.m0 + M; ++m) {
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
      // its sums are not known: coded as a whole
      if (a.state) (reinterpret_cast<WideState*>(a.state) + (int64_t)(m - a.m0) * a.nb + k)->mode = kWholeGradient;
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
// what the levels leave open, then the levels' state (some 100 KiB per bucket and worker) and the lists of what
// lies inside a bracket; workers are taken in groups that fit.
size_t exact_wide_workspace_bytes(const qa_layout* L) {
  if (!bucket_spans_tiles(L)) return 0;
  const size_t d = (size_t)L->d, nt = (size_t)tiles_of(L->d);
  return xalign(d * 8) + 4 * xalign(nt * 8) + xalign(d * 8 + d + (size_t(4) << 20));
}

// Thresholds, and for buckets of more than 65536 components codes and scales too (*coded): part_sum, part_cnt of the
// quantizer's own workspace hold a chunk's sums.
int exact_thresholds_wide(const qa_layout* L, const float* g, int64_t g_stride, uint32_t* codes, float* scales,
                          float* thresholds, double* part_sum, uint32_t* part_cnt, void* ws, size_t ws_bytes,
                          bool* coded, hipStream_t stream) {
  if (!bucket_spans_tiles(L)) return QA_ERR_INVALID_ARG;
  if (L->d >= (int64_t(1) << 32)) return QA_ERR_TOO_LARGE;
  if (!ws || ws_bytes < exact_wide_workspace_bytes(L) || !aligned(ws, 256)) return QA_ERR_WORKSPACE;
  WideArgs a{};
  a.g = g; a.g_stride = g_stride; a.d = L->d;
  a.bucket_len = L->bucket ? L->bucket : L->d;
  a.nb = buckets_of(L->d, L->bucket);
  a.thresholds = thresholds; a.scales = scales; a.scale_stride = L->scale_stride;
  a.codes = codes; a.code_stride = L->code_stride;
  a.part_sum = part_sum; a.part_cnt = part_cnt;
  a.sort_keys = static_cast<uint32_t*>(ws);
  const int64_t longest = a.bucket_len < L->d ? a.bucket_len : L->d;
  *coded = longest > kResidentMost;
  if (!*coded) {
    const dim3 pairs((unsigned)a.nb, (unsigned)L->M);
    if (a.nb * L->M > kComputeUnits) hipLaunchKernelGGL(exact_resident_kernel<true>, pairs, dim3(kScanThreads), 0, stream, a);
    else hipLaunchKernelGGL(exact_resident_kernel<false>, pairs, dim3(kScanThreads), 0, stream, a);
    hipLaunchKernelGGL(exact_sort_open_kernel, dim3((unsigned)a.nb), dim3(kScanThreads), 0, stream, a, (int)L->M);
    return launch_status();
  }
  const size_t keys = xalign((size_t)L->d * 8), room = ws_bytes - keys;
  a.state = static_cast<char*>(ws) + keys;
  const int64_t fit = (int64_t)(room / (sizeof(WideState) * (size_t)a.nb));
  if (fit < 1) return QA_ERR_WORKSPACE;
  const int64_t group = fit < L->M ? fit : L->M;
  const size_t states = sizeof(WideState) * (size_t)(a.nb * group);
  WideList list{};
  list.entries = reinterpret_cast<uint2*>(a.state + states);
  const int64_t tiles = tiles_of(longest), capacity = (int64_t)((room - states) / sizeof(uint2)) / (a.nb * group);
  list.capacity = (uint32_t)(capacity < longest ? capacity : longest);
  SampleArgs sa{};
  // A list holds a 32nd of its bucket, twice what a bracket may leave open: a quarter of a byte per component and
  // worker, of the 9 that there are per component.  So more than some 30 workers of one long vector (fewer with a
  // short last bucket) are not sampled.
  const bool sampled = tiles >= kSampledTiles && tiles * a.nb * L->M >= kSampledInAll && capacity >= longest / 32;
  const int64_t units = longest / kUnit;
  sa.every = (units + kMostUnits - 1) / kMostUnits;
  if (sa.every < kMostOften) sa.every = kMostOften;
  sa.units = (int)(units / sa.every);
  sa.groups = (sa.units + kUnitsPerGroup - 1) / kUnitsPerGroup;
  // Chunks: a work-group per compute unit, whole passes of its threads.  Two of them cost more in bins added to memory
  // than they gain: 10^6 x 8 114 -> 87 us, 2^21 x 8 113 -> 99, 2^24 x 4 Cauchy components 267 -> 232; chunks that only double
  // leave half the chip idle just beyond a power of two: 2^25 + 5 Cauchy components 177 -> 152.
  constexpr int64_t kPassTiles = kPassComponents / kTile;
  const int64_t each = a.nb * group < kComputeUnits ? kComputeUnits / (a.nb * group) : 1;
  const int64_t per = ((tiles + each - 1) / each + kPassTiles - 1) / kPassTiles * kPassTiles;
  const int chunk_tiles = (int)(per < kMostChunkTiles ? per : kMostChunkTiles);
  const int64_t chunks = (tiles + chunk_tiles - 1) / chunk_tiles, short_chunks = (tiles + kBracketedTiles - 1) / kBracketedTiles;
  if (a.nb * chunks > 0x7fffffffLL || a.nb * short_chunks > 0x7fffffffLL) return QA_ERR_WORKSPACE;
  for (int64_t m0 = 0; m0 < L->M; m0 += group) {
    const unsigned here = (unsigned)(L->M - m0 < group ? L->M - m0 : group);
    a.m0 = (int)m0;
    const dim3 pairs((unsigned)a.nb, here), parts((unsigned)(a.nb * chunks), here), block(kPassThreads);
    const auto level_kernel = a.nb * chunks * here > kComputeUnits ? exact_wide_level_kernel<true>
                                                                      : exact_wide_level_kernel<false>;
    hipLaunchKernelGGL(exact_wide_init_kernel, pairs, block, 0, stream, a);
    if (sampled) {
      const dim3 samples((unsigned)(a.nb * sa.groups), here);
      hipLaunchKernelGGL(exact_wide_sample_kernel, samples, block, 0, stream, a, sa);
      hipLaunchKernelGGL(exact_wide_probe_kernel, samples, block, 0, stream, a, sa);
      hipLaunchKernelGGL(exact_wide_bracketed_kernel, dim3((unsigned)(a.nb * short_chunks), here), block, 0, stream, a, list,
                         short_chunks, kBracketedTiles);
      hipLaunchKernelGGL(exact_wide_prove_kernel, pairs, block, 0, stream, a);
    }
    for (int level = 0; level < kLevels; ++level)
      hipLaunchKernelGGL(level_kernel, parts, block, 0, stream, a, list, chunks, chunk_tiles,
                         level == kLevels - 1 ? 1 : 0);
    hipLaunchKernelGGL(exact_sort_open_kernel, dim3((unsigned)a.nb), block, 0, stream, a, (int)here);
    hipLaunchKernelGGL(exact_wide_codes_kernel, parts, block, 0, stream, a, list, chunks, chunk_tiles);
  }
  return launch_status();
}

}  // namespace qa
