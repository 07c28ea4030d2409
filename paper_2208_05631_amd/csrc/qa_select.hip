// Indicator, selection and sparse encoding (Section 3.2, equations "select" and "ind";
// Algorithm 1 worker block and server decode; Encode paragraph: 32 + d + 2k bits) for gfx950.
//
//   indicator_kernel          : I_i = (x_i != 0) or (x^_i != 0), x^ being the worker's own QCMD/QRDA
//                               update from its full-precision gradient; one bit per coordinate,
//                               formed with wave ballots (64 consecutive coordinates per ballot).
//   quantize_selected_kernel  : per 4096-tile, threshold/scale over the marked components only and
//                               their 2-bit codes compacted in index order (prefix sum of the
//                               marks, extract table, LDS bit stream); _few_ for few tiles.
//   decode_selected_kernel    : S^{-1}: spreads the compact codes back to the dense 2-bit layout
//                               that the fused steps read.
//   select_codes_kernel       : S applied to a coded message (the server's push): the inverse.
// (The steps that read sparse messages directly live with the step kernel.)
#include "qa_common.h"
#include "qa_sparse.h"

namespace qa {

struct SelArgs {
  const float* g; int64_t g_stride;
  const float* x; const float* G; const float* z;
  uint32_t* ind; const uint32_t* ind_in; int64_t ind_stride;
  uint32_t* sel_codes; const uint32_t* sel_in; uint32_t* dense; int64_t code_stride;
  int64_t dense_stride;        // words between workers in `dense` (the decoder's output)
  uint32_t* counts; float* scales; float* thresholds; int64_t scale_stride;
  int64_t d, W, NW;            // coordinates, dense code words, indicator words
  int M, method;
  float eta, lam_eta, delta, t_lam, thr_coef;
  // buckets other than one 4096-tile (the general kernels below)
  int seg;                     // threads per bucket inside a tile: bucket/16 for 64 <= bucket <= 4096
  int64_t nb, ntiles, tiles_per_bucket, area_words;   // buckets spanning several tiles
  uint32_t* ws_count; double* ws_s1; double* ws_s2; uint32_t* ws_c2; int64_t* ws_start; float* ws_thr;
  uint2* ws_open;              // one-read quantizer: kOpenSlots open components of every tile
  int64_t samples;             // one-read quantizer: sampled tiles per bucket (at most)
};

// Granularity of a sparse message's buckets: one 4096-tile each; 64 .. 2048 coordinates, inside a
// tile (bucket j of a tile = the segment of seg = bucket/16 consecutive code words, its compact
// stream starts at word j*seg of the tile's 256 words); or spanning several tiles.
enum SelKind { kSelTile, kSelLocal, kSelMulti };

// The worker's own would-be parameter from gradient component g (same operation order as the
// update of the fused steps).
__device__ __forceinline__ float local_update(const SelArgs& a, float g, float x, float G, float z) {
  const float g2 = g * g;
  const float Gh = G + g2;
  const float H = a.delta + sqrtf(Gh);
  if (a.method == 0) {
    const float step = (a.eta * g) / H;
    const float u = x - step;
    const float tau = a.lam_eta / H;
    const float r = fabsf(u) - tau;
    return r > 0.0f ? copysignf(r, u) : 0.0f;
  }
  const float zh = z + g;
  const float r = fabsf(zh) - a.t_lam;
  const float mag = (a.eta * r) / H;
  return r > 0.0f ? -copysignf(mag, zh) : 0.0f;
}

// Whether the worker's own update is non-zero, decided without square root or division whenever
// that is provably the same as evaluating local_update():
//   QCMD with x == 0:  x^ != 0  <=>  fl(a/H) > fl(b/H),  a = |fl(eta*g)|, b = fl(lambda*eta).
//     Correctly rounded division by the same H > 0 is monotone, so a <= b gives "zero"; and if
//     a > b*(1+2^-21) while b/H is a normal number, the two quotients differ by more than their
//     rounding errors (2^-24 relative each), which gives "non-zero".
//   QRDA:  r = fl(|fl(z+g)| - t*lambda) is formed exactly as in the update; r <= 0 gives "zero",
//     and r > 0 gives "non-zero" unless (eta*r)/H underflows to 0.
//   H <= delta + max(1, G + g*g) bounds the quotients away from the subnormal range.
// Everything else (ties within the margin, possible underflow, NaN/Inf) is left undecided and
// the caller evaluates the closed form itself.
// Written without branches: every lane runs the same straight-line code.
template <int METHOD>
__device__ __forceinline__ bool quick_indicator(const SelArgs& a, float g, float x, float G, float z,
                                                bool* mark) {
  const bool xnz = x != 0.0f;
  const float s2 = G + g * g;
  const bool valid = s2 >= 0.0f;                         // false for NaN or an invalid accumulator
  const float tiny = (a.delta + (s2 > 1.0f ? s2 : 1.0f)) * 0x1p-100f;
  bool m, decided;
  if (METHOD == 0) {
    const float av = fabsf(a.eta * g), b = a.lam_eta;
    m = av > b;
    decided = (av <= b) | ((av > b * 1.0000005f) & (b >= tiny));
  } else {
    const float zh = z + g;
    const float r = fabsf(zh) - a.t_lam;
    m = r > 0.0f;
    decided = !m | (a.eta * r >= tiny);
  }
  *mark = xnz | m;
  return xnz | (valid & decided);
}

// Rare path: the 1024 coordinates of one wave for worker m, all through the closed form.
__device__ __forceinline__ void indicator_slab_exact(const SelArgs& a, int m, int64_t base, int lane) {
  const float* g = a.g + (int64_t)m * a.g_stride;
  uint32_t* out = a.ind + (int64_t)m * a.ind_stride;
#pragma unroll 1
  for (int j = 0; j < 16; ++j) {
    const int64_t c = base + j * 64 + lane;
    bool mark = false;
    if (c < a.d) {
      const float x = a.x[c];
      const float xh = local_update(a, g[c], x, a.G[c], a.method == 1 ? a.z[c] : 0.0f);
      mark = x != 0.0f || xh != 0.0f;
    }
    const uint64_t bits = __ballot(mark);
    const int64_t w0 = (base + j * 64) / 32;
    if (lane < 2 && w0 + lane < a.NW) out[w0 + lane] = (uint32_t)(bits >> (32 * lane));
  }
}

// wave w of the work-group owns coordinates [w*1024, (w+1)*1024) of the tile, lane l the
// coordinates j*64 + l (j = 0..15): each ballot is 64 consecutive indicator bits.
// Slab that lies wholly below d: no clamps or masks; the next worker's gradient is requested
// before the current one is examined; ballot j (64 indicator bits) is kept by lane j, and lanes
// 0..15 store the slab's 128 bytes.  STREAM: gradients that the last-level cache cannot hold are streamed
// (8 workers x 2^27: QCMD 992 -> 948 us, 8 x 10^8: QRDA 826 -> 814); x, G and z as well: no faster.  Those it
// holds are kept for the quantizer that follows (4 x 4 M, one scale, indicator to update: 86.8 us, streamed 89.5).
constexpr int64_t kStreamedGradients = int64_t(1) << 26;   // components of all workers: 256 MB
template <bool STREAM>
__device__ __forceinline__ float gradient_load(const float* p) { return STREAM ? __builtin_nontemporal_load(p) : *p; }
template <int METHOD, bool STREAM>
__device__ __forceinline__ void indicator_wave_full(const SelArgs& a, int64_t base, int lane) {
  const float* px = a.x + base + lane;
  const float* pG = a.G + base + lane;
  const float* pz = METHOD == 1 ? a.z + base + lane : px;  // z may be null for QCMD
  float x[16], G[16], z[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    x[j] = px[j * 64];
    G[j] = pG[j * 64];
    z[j] = METHOD == 1 ? pz[j * 64] : 0.0f;
  }
  const float* pg = a.g + base + lane;
  uint32_t* out = a.ind + base / 32 + 2 * lane;
  float gn[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) gn[j] = gradient_load<STREAM>(pg + j * 64);
  for (int m = 0; m < a.M; ++m) {
    float gv[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) gv[j] = gn[j];
    if (m + 1 < a.M) {                                   // the next worker's gradient, ahead of use
      const float* pn = pg + (int64_t)(m + 1) * a.g_stride;
#pragma unroll
      for (int j = 0; j < 16; ++j) gn[j] = gradient_load<STREAM>(pn + j * 64);
    }
    bool undecided = false;
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      bool mark = false;
      undecided |= !quick_indicator<METHOD>(a, gv[j], x[j], G[j], z[j], &mark);
      const uint64_t bits = __ballot(mark);
      lo = lane == j ? (uint32_t)bits : lo;
      hi = lane == j ? (uint32_t)(bits >> 32) : hi;
    }
    if (__any(undecided)) {
      indicator_slab_exact(a, m, base, lane);
    } else if (lane < 16) {
      out[(int64_t)m * a.ind_stride] = lo;
      out[(int64_t)m * a.ind_stride + 1] = hi;
    }
  }
}

// Three waves per SIMD: measured best for this access pattern (2: 2.15 ms, 3: 1.91, 4: 1.98,
// 6-8: 2.00 at d = 2^28, M = 8); the kernel needs only 58-77 registers and would otherwise run 6-8.
template <int METHOD, bool STREAM>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(3, 3)))
void indicator_kernel(SelArgs a) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t base = (int64_t)blockIdx.x * kTile + wave * 1024;
  if (base + 1024 <= a.d) indicator_wave_full<METHOD, STREAM>(a, base, lane);
  else if (base < a.d)                                   // the vector ends inside this slab: closed form
    for (int m = 0; m < a.M; ++m) indicator_slab_exact(a, m, base, lane);
}

__global__ __launch_bounds__(kThreads) void indicator_or_kernel(SelArgs a) {
  const int64_t w = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (w >= a.NW) return;
  uint32_t v = 0u;
  for (int m = 0; m < a.M; ++m) v |= a.ind_in[(int64_t)m * a.ind_stride + w];
  a.ind[w] = v;
}

// Exclusive prefix sum of `v` over the 256 threads and the total; two barriers.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* lds_w, uint32_t* total) {
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const uint32_t incl = wave_scan_u32(v);
  __syncthreads();
  if (lane == kWave - 1) lds_w[wave] = incl;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    const uint32_t s = lds_w[w];
    if (w < wave) before += s;
    tot += s;
  }
  *total = tot;
  return before + incl - v;
}

// the 16 indicator bits of coordinates [16t, 16t+16) of tile `tile`
__device__ __forceinline__ uint32_t mask16_of(const uint32_t* ind, int64_t NW, int64_t tile, int t) {
  const int64_t w = tile * (kTile / 32) + t / 2;
  const uint32_t word = w < NW ? ind[w] : 0u;
  return (word >> (16 * (t & 1))) & 0xFFFFu;
}


// A wave decodes kDecodeTiles consecutive 4096-tiles, phase by phase for all of them (their loads
// are independent and overlap).  Within a tile lane l holds code words j*64 + l (j = 0..3), so
// that each store instruction of the wave writes 256 consecutive bytes.  The position of a
// word's first marked component in the tile's compact stream is the number of marked components
// before it: a wave scan per j plus the totals of the earlier j.  The codes are spread to their
// fields four components at a time through the deposit table (copied to LDS once per block).
constexpr int kDecodeTiles = 2;

// kSelMulti: buckets that span tiles (and one scale per message of a long vector): a tile's codes
// start at code `start` of its bucket's stream, start being the tile's entry of the scan in the
// workspace: word start/16 of the bucket's area, code start%16 of that word.
// kSelLocal: a word's codes are counted from the start of its own bucket's stream, i.e. its
// position in the tile minus the position of the bucket's first word (same j and a lane of the
// wave for buckets up to 1024 coordinates, lane 0 of an even j for 2048).
template <int KIND>
__global__ __launch_bounds__(kThreads) void decode_selected_kernel(SelArgs a) {
  __shared__ uint8_t lut[16 * 256];
  reinterpret_cast<uint4*>(lut)[threadIdx.x] = reinterpret_cast<const uint4*>(kDepositLut.v)[threadIdx.x];
  const int lane = threadIdx.x % kWave;
  const int64_t tile0 = ((int64_t)blockIdx.x * kWaves + threadIdx.x / kWave) * kDecodeTiles;
  const int m = blockIdx.y;
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride;
  uint32_t mask[kDecodeTiles][4], incl[kDecodeTiles][4];
#pragma unroll
  for (int u = 0; u < kDecodeTiles; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int wl = j * 64 + lane;                        // code word within the tile
      const int64_t iw = (tile0 + u) * (kTile / 32) + wl / 2;
      const uint32_t word = iw < a.NW ? ind[iw] : 0u;
      mask[u][j] = (word >> (16 * (wl & 1))) & 0xFFFFu;
    }
#pragma unroll
  for (int u = 0; u < kDecodeTiles; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // bits at or beyond d are not components: ignoring them keeps every read of the compact
      // stream inside the words that exist for this tile
      const int64_t left = a.d - ((tile0 + u) * kTile + (int64_t)(j * 64 + lane) * 16);
      if (left < 16) mask[u][j] = left > 0 ? (mask[u][j] & ((1u << left) - 1u)) : 0u;
      incl[u][j] = wave_scan_u32((uint32_t)__popc(mask[u][j]));
    }
  uint32_t win_lo[kDecodeTiles][4], win_hi[kDecodeTiles][4], sh[kDecodeTiles][4];
#pragma unroll
  for (int u = 0; u < kDecodeTiles; ++u) {
    // clamped for tiles beyond the vector: their masks are 0, so nothing is read through it
    const int64_t tile = (tile0 + u) * kTile < a.d ? tile0 + u : 0;
    const uint32_t* sel = a.sel_in + (int64_t)m * a.code_stride;
    uint32_t start = 0;                                  // marked components in earlier j
    if (KIND == kSelMulti) {
      const int64_t first = a.ws_start[(int64_t)m * a.ntiles + tile];
      sel += (tile / a.tiles_per_bucket) * a.area_words + (first >> 4);
      start = (uint32_t)(first & 15);
    } else {
      sel += tile * kTileWords;
    }
    uint32_t ex[4];                                      // marked components of the tile before the word
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      ex[j] = start + incl[u][j] - (uint32_t)__popc(mask[u][j]);
      start += (uint32_t)__builtin_amdgcn_readlane((int)incl[u][j], kWave - 1);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      // the word's n <= 16 codes are codes before .. before+n-1 of the compact stream `src`:
      // word before/16 and, only if they cross a word boundary, the next one; both lie below
      // ceil(K/16) <= the words that exist for the stream (K = its marked components)
      const uint32_t n = (uint32_t)__popc(mask[u][j]);
      uint32_t before = ex[j];
      const uint32_t* src = sel;
      if (KIND == kSelLocal) {
        const int s0 = (j * 64 + lane) & ~(a.seg - 1);     // first code word of the bucket
        const uint32_t e0 = a.seg <= kWave ? (uint32_t)__shfl((int)ex[j], lane & ~(a.seg - 1), kWave)
                                           : (uint32_t)__builtin_amdgcn_readlane((int)ex[j & ~1], 0);
        before = ex[j] - e0;
        src = sel + s0;
      }
      const uint32_t w0 = before / 16;
      sh[u][j] = 2 * (before % 16);
      win_lo[u][j] = n != 0u ? src[w0] : 0u;
      win_hi[u][j] = (before % 16) + n > 16u ? src[w0 + 1] : 0u;
    }
  }
  __syncthreads();                                       // the table is in LDS
#pragma unroll
  for (int u = 0; u < kDecodeTiles; ++u)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t win = win_lo[u][j] >> sh[u][j];
      if (sh[u][j]) win |= win_hi[u][j] << (32 - sh[u][j]);
      uint32_t out = 0;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const uint32_t nib = (mask[u][j] >> (4 * q)) & 15u;
        out |= (uint32_t)lut[nib * 256 + (win & 0xFFu)] << (8 * q);
        win >>= 2 * __popc(nib);
      }
      const int64_t w = (tile0 + u) * kTileWords + j * 64 + lane;
      if (w < a.W) (a.dense + (int64_t)m * a.dense_stride)[w] = out;
    }
}

// Extract table, the inverse of the deposit table: entry [nib][s] packs the 2-bit fields of byte s
// at the set bits of nib towards bit 0 (lowest set bit first).
constexpr DepositLut make_extract_lut() {
  DepositLut t{};
  for (int nib = 0; nib < 16; ++nib)
    for (int s = 0; s < 256; ++s) {
      uint32_t out = 0;
      int n = 0;
      for (int b = 0; b < 4; ++b)
        if ((nib >> b) & 1) { out |= (((uint32_t)s >> (2 * b)) & 3u) << (2 * n); ++n; }
      t.v[nib * 256 + s] = (uint8_t)out;
    }
  return t;
}
__device__ const DepositLut kExtractLut = make_extract_lut();


__device__ __forceinline__ void wave_fence() {           // order of a wave's own LDS accesses
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Q(S(g, I)) for buckets of 4096: a wave per tile, which reads it 16 bytes per lane side by side (float4
// j*64 + lane, j = 0..15) and holds it in registers for both sums.  Unmarked components become 0 and add nothing; the fields of a
// float4 go through the extract table, the four lanes of a quad join theirs to the codes of one
// indicator half-word, and every fourth round each lane appends one half-word's codes to the wave's stream.
// Bound by the read of the gradient where few are marked, by that and vector instructions where most are (1380 per tile, three quarters of the issue slots;
// with four waves per tile, 16 consecutive components per lane and a branch per component 2000).  8 workers x 10^8, 7 / 30 / 97 %
// marked: 640 -> 570, 665 -> 592, 675 -> 640 us; with the words stored through the cache, 97 %, another 3 %.
struct SelTileLds {
  uint2 words[kTile / 32];                               // indicator word, marked components before it
  uint32_t stream[kTileWords + 2];
};
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(4))) void quantize_selected_kernel(SelArgs a) {
  __shared__ uint8_t lut[16 * 256];
  __shared__ SelTileLds lds_all[kWaves];
  reinterpret_cast<uint4*>(lut)[threadIdx.x] = reinterpret_cast<const uint4*>(kExtractLut.v)[threadIdx.x];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t tile = (int64_t)blockIdx.x * kWaves + wave;
  const int m = blockIdx.y;
  SelTileLds& lds = lds_all[wave];
  __syncthreads();                                       // the table is in LDS
  if (tile * kTile >= a.d) return;
  const float* g = a.g + (int64_t)m * a.g_stride + tile * kTile;
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride + tile * (kTile / 32);
  const int64_t live = a.d - tile * kTile, words_here = a.NW - tile * (kTile / 32);
  uint32_t iv[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) iv[h] = 2 * lane + h < words_here ? ind[2 * lane + h] : 0u;
  typedef float floatx4 __attribute__((ext_vector_type(4)));
  floatx4 v[16];
  if (live >= kTile) {
    const floatx4* src = reinterpret_cast<const floatx4*>(g) + lane;
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = __builtin_nontemporal_load(src + j * kWave);
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int i = (j * kWave + lane) * 4 + e;
        v[j][e] = i < live ? g[i] : 0.0f;
      }
  }
  const uint32_t n0 = (uint32_t)__popc(iv[0]), n1 = (uint32_t)__popc(iv[1]);
  const uint32_t incl = wave_scan_u32(n0 + n1);
  const uint32_t K = (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
  lds.words[2 * lane] = make_uint2(iv[0], incl - n0 - n1);
  lds.words[2 * lane + 1] = make_uint2(iv[1], incl - n1);
#pragma unroll
  for (int j = 0; j < 4; ++j) lds.stream[j * kWave + lane] = 0u;
  if (lane < 2) lds.stream[kTileWords + lane] = 0u;
  wave_fence();

  const uint32_t sh = 4 * (lane & 7);                    // of the lane's four bits in its indicator word
  uint32_t nibs[2] = {0u, 0u};                           // those of round j: bits 4*(j & 7) of nibs[j / 8]
  double s1[2] = {0.0, 0.0};
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const uint32_t nib = (lds.words[8 * j + (lane >> 3)].x >> sh) & 15u;
    nibs[j / 8] |= nib << (4 * (j & 7));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int marked = (int)(nib << (31 - e)) >> 31;   // 0 or all ones
      v[j][e] = __int_as_float(__float_as_int(v[j][e]) & marked);
      s1[e & 1] += (double)fabsf(v[j][e]);
    }
  }
  const double S1 = wave_sum_f64(s1[0] + s1[1]);
  const float Delta = K ? threshold_from_sum(S1, a.thr_coef, (int64_t)K) : 0.0f;

  double s2[2] = {0.0, 0.0};
  uint32_t c2 = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t mine = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = 4 * i + r;
      uint32_t b = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float av = fabsf(v[j][e]);
        const bool keep = av > Delta;                    // Delta is not negative, or NaN
        s2[e & 1] += (double)(keep ? av : 0.0f);
        const uint32_t pat = 1u | ((__float_as_uint(v[j][e]) >> 30) & 2u);
        b |= (keep ? pat : 0u) << (2 * e);
      }
      c2 += (uint32_t)__popc(b & 0x55u);
      const uint32_t nib = (nibs[j / 8] >> (4 * (j & 7))) & 15u;
      const uint32_t n = (uint32_t)__popc(nib), pair = n + (uint32_t)dpp_i32<kDppQuadXor1>((int)n);
      const uint32_t other = (uint32_t)dpp_i32<kDppQuadXor2>((int)pair);
      const uint32_t before = ((lane & 1) ? pair - n : 0u) + ((lane & 2) ? other : 0u);   // codes of the quad's earlier lanes
      uint32_t w = (uint32_t)lut[nib * 256 + b] << (2 * before);
      w |= (uint32_t)dpp_i32<kDppQuadXor1>((int)w);
      w |= (uint32_t)dpp_i32<kDppQuadXor2>((int)w);
      if ((lane & 3) == r) mine = w;
      // the round's additions here: moved behind the last round they keep every compare mask alive, which spills
      asm volatile("" : "+v"(s2[0]), "+v"(s2[1]));
    }
    const int half = 16 * (4 * i + (lane & 3)) + (lane >> 2);   // the half-word whose codes the lane holds
    const uint2 word = lds.words[half >> 1];
    const uint32_t low = word.x & 0xFFFFu;
    const uint32_t n = (uint32_t)__popc((half & 1) ? word.x >> 16 : low);
    const uint32_t before = word.y + ((half & 1) ? (uint32_t)__popc(low) : 0u);
    if (n) {
      const uint32_t w0 = before / 16, at = 2 * (before % 16);
      atomicOr(&lds.stream[w0], mine << at);
      if (at && 2 * n + at > 32) atomicOr(&lds.stream[w0 + 1], mine >> (32 - at));
    }
  }
  const double S2 = wave_sum_f64(s2[0] + s2[1]);
  c2 = wave_sum_u32(c2);
  wave_fence();
  uint32_t* out = a.sel_codes + (int64_t)m * a.code_stride + tile * kTileWords;
  const uint32_t nwords = (K + 15) / 16;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if ((uint32_t)(j * kWave + lane) < nwords) store_through(out + j * kWave + lane, lds.stream[j * kWave + lane]);
  if (lane == 0) {
    const int64_t at = (int64_t)m * a.scale_stride + tile;
    a.counts[at] = K;
    a.scales[at] = scale_from_sum(S2, c2);
    if (a.thresholds) a.thresholds[at] = Delta;
  }
}

// The same with four waves per tile, 16 consecutive components per thread, for calls whose tiles the chip takes in one
// round, where a wave's chain of instructions is the time (one tile 7.1 us as a wave, 4.0 so).  Alone / as a wave per tile, us,
// 7 % marked, tiles of all workers: 1500 7.6 / 10.0, 2048 9.3 / 10.0, 4096 16.0 / 17.3, 5000 18.2 / 18.3, 6000 21.0 / 20.7,
// 8000 26.7 / 25.6, 16000 49.6 / 46.0.  The magnitudes are added in another order: a threshold or scale may differ in its last bit.
constexpr int64_t kSelFewTiles = 5120;
__global__ __launch_bounds__(kThreads) void quantize_selected_few_kernel(SelArgs a) {
  __shared__ uint32_t stream[kTileWords + 1];
  __shared__ uint32_t lds_w[kWaves];
  __shared__ double lds_s1[kWaves];
  __shared__ double lds_s2[kWaves];
  __shared__ uint32_t lds_c[kWaves];
  const int t = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  const float* g = a.g + (int64_t)m * a.g_stride;
  const uint32_t mask = mask16_of(a.ind_in + (int64_t)m * a.ind_stride, a.NW, tile, t);
  const int64_t i0 = tile * kTile + 16 * (int64_t)t;

  float v[16];
  if (i0 + 16 <= a.d) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 f = *reinterpret_cast<const float4*>(g + i0 + 4 * q);
      v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = (i0 + j < a.d) ? g[i0 + j] : 0.0f;
  }
  stream[t] = 0u;
  if (t == 0) stream[kTileWords] = 0u;

  double s1 = 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if ((mask >> j) & 1u) s1 += (double)fabsf(v[j]);
  const uint32_t cnt = (uint32_t)__popc(mask);
  uint32_t K;
  const uint32_t before = block_exclusive_scan(cnt, lds_w, &K);
  const double S1 = block_sum_f64(s1, lds_s1);
  const float Delta = K ? threshold_from_sum(S1, a.thr_coef, (int64_t)K) : 0.0f;

  double s2 = 0.0;
  uint32_t c2 = 0, bits = 0, pos = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if ((mask >> j) & 1u) {
      const float av = fabsf(v[j]);
      if (av > Delta) { s2 += (double)av; ++c2; }
      bits |= ternary_field(v[j], Delta) << (2 * pos);
      ++pos;
    }
  }
  // append this thread's 2*cnt bits at bit 2*before of the tile's compact stream
  if (cnt) {
    const uint32_t word = before / 16, sh = 2 * (before % 16);
    atomicOr(&stream[word], bits << sh);
    if (sh && (2 * cnt + sh > 32)) atomicOr(&stream[word + 1], bits >> (32 - sh));
  }
  s2 = wave_sum_f64(s2);
  c2 = wave_sum_u32(c2);
  if ((t % kWave) == 0) { lds_s2[t / kWave] = s2; lds_c[t / kWave] = c2; }
  __syncthreads();
  const uint32_t nwords = (K + 15) / 16;
  if ((uint32_t)t < nwords) (a.sel_codes + (int64_t)m * a.code_stride)[tile * kTileWords + t] = stream[t];
  if (t == 0) {
    const double S2 = (lds_s2[0] + lds_s2[1]) + (lds_s2[2] + lds_s2[3]);
    const uint32_t C = lds_c[0] + lds_c[1] + lds_c[2] + lds_c[3];
    a.counts[(int64_t)m * a.scale_stride + tile] = K;
    a.scales[(int64_t)m * a.scale_stride + tile] = scale_from_sum(S2, C);
    if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + tile] = Delta;
  }
}

// A tile's stream word w, which ends or begins inside it, to memory or to the tile's head.
__device__ __forceinline__ void store_word(uint32_t* out, uint32_t w, uint32_t first, uint32_t bits, uint32_t* head) {
  if (w == 0 && first != 0) *head = bits;
  else store_through(out + w, bits);
}

// S applied to a coded message: one wave per 4096-tile, lane l holds code words j*64 + l of the
// tile (as in the decoder).  Each word's marked codes are packed through the extract table and
// appended at their position in the tile's compact stream, which is assembled in LDS (one area
// per wave) and written out in whole words.
// kSelMulti (buckets that span tiles): the tile's codes start at code start%16 of word start/16
// of the bucket's area (start from the scan in the workspace); its part of a word that begins in an
// earlier tile goes to the workspace for gsel_join_kernel, the other words are stored.
// kSelLocal (buckets inside a tile): bucket j's stream starts at word j*seg; its first
// ceil(K_j/16) words are written, and K_j by the bucket's first lane.
template <int KIND>
__global__ __launch_bounds__(kThreads) void select_codes_kernel(SelArgs a) {
  __shared__ uint8_t lut[16 * 256];
  __shared__ uint32_t stream_all[kWaves][kTileWords + 2];
  reinterpret_cast<uint4*>(lut)[threadIdx.x] = reinterpret_cast<const uint4*>(kExtractLut.v)[threadIdx.x];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  uint32_t* stream = stream_all[wave];
  const int64_t tile_raw = (int64_t)blockIdx.x * kWaves + wave;
  const bool exists = tile_raw * kTile < a.d;
  const int64_t tile = exists ? tile_raw : 0;            // clamped: every wave runs the same code
  const int m = blockIdx.y;
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride;
  const uint32_t* dense = a.sel_in + (int64_t)m * a.code_stride + tile * kTileWords;
  uint32_t mask[4], word[4], incl[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int wl = j * 64 + lane;
    const int64_t iw = tile * (kTile / 32) + wl / 2;
    const uint32_t iv = iw < a.NW ? ind[iw] : 0u;
    mask[j] = (iv >> (16 * (wl & 1))) & 0xFFFFu;
    const int64_t left = a.d - (tile * kTile + (int64_t)wl * 16);
    if (left < 16) mask[j] = left > 0 ? (mask[j] & ((1u << left) - 1u)) : 0u;
    const int64_t w = tile * kTileWords + wl;
    const uint32_t raw = w < a.W ? dense[wl] : 0u;
    const uint32_t lo = raw & 0x55555555u;
    word[j] = lo | (raw & (lo << 1));                    // reserved pattern 10 reads as 0
    stream[wl] = 0u;
  }
  if (lane < 2) stream[kTileWords + lane] = 0u;
#pragma unroll
  for (int j = 0; j < 4; ++j) incl[j] = wave_scan_u32((uint32_t)__popc(mask[j]));
  __syncthreads();                                       // table and zeroed streams are in LDS
  int64_t base = tile * kTileWords;
  uint32_t first = 0;
  if (KIND == kSelMulti) {
    const int64_t st = a.ws_start[(int64_t)m * a.ntiles + tile];
    base = (tile / a.tiles_per_bucket) * a.area_words + (st >> 4);
    first = (uint32_t)(st & 15);
  }
  uint32_t start = first, ex[4], total[4], in_bucket[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    total[j] = (uint32_t)__builtin_amdgcn_readlane((int)incl[j], kWave - 1);
    ex[j] = start + incl[j] - (uint32_t)__popc(mask[j]);
    start += total[j];
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t n = (uint32_t)__popc(mask[j]);
    uint32_t before = ex[j];
    if (KIND == kSelLocal) {
      const int s0 = (j * 64 + lane) & ~(a.seg - 1);       // first code word of the bucket
      uint32_t e0, Kb = n;
      if (a.seg <= kWave) {
        e0 = (uint32_t)__shfl((int)ex[j], lane & ~(a.seg - 1), kWave);
        for (int off = 1; off < a.seg; off <<= 1) Kb += (uint32_t)__shfl_xor((int)Kb, off, kWave);
      } else {
        e0 = (uint32_t)__builtin_amdgcn_readlane((int)ex[j & ~1], 0);
        Kb = total[j] + total[j ^ 1];
      }
      in_bucket[j] = Kb;
      before = 16u * (uint32_t)s0 + (ex[j] - e0);
    }
    uint32_t bits = 0, filled = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t nib = (mask[j] >> (4 * q)) & 15u;
      bits |= (uint32_t)lut[nib * 256 + ((word[j] >> (8 * q)) & 0xFFu)] << filled;
      filled += 2 * __popc(nib);
    }
    if (n) {
      const uint32_t w0 = before / 16, sh = 2 * (before % 16);
      atomicOr(&stream[w0], bits << sh);
      if (sh && 2 * n + sh > 32) atomicOr(&stream[w0 + 1], bits >> (32 - sh));
    }
  }
  __syncthreads();
  if (exists) {
    const uint32_t end = start, nwords = (end + 15) / 16;  // one past the tile's last code
    uint32_t* out = a.sel_codes + (int64_t)m * a.code_stride + base;
    if (KIND == kSelMulti) {
      uint32_t head = 0;
      if (end != first)
        for (uint32_t w = lane; w < nwords; w += kWave) store_word(out, w, first, stream[w], &head);   // at most 257
      if (lane == 0) a.ws_count[(int64_t)m * a.ntiles + tile] = head;
    } else if (KIND == kSelLocal) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int wl = j * 64 + lane, s0 = wl & ~(a.seg - 1);
        if ((uint32_t)(wl - s0) < (in_bucket[j] + 15) / 16) out[wl] = stream[wl];
        const int64_t kb = (tile * kTile + 16 * (int64_t)wl) / (16 * (int64_t)a.seg);
        if (wl == s0 && kb < a.nb) a.counts[(int64_t)m * a.scale_stride + kb] = in_bucket[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if ((uint32_t)(j * 64 + lane) < nwords) out[j * 64 + lane] = stream[j * 64 + lane];
      if (lane == 0) a.counts[(int64_t)m * a.scale_stride + tile] = end;
    }
  }
}

// ---- any bucket size -------------------------------------------------------------------------
//
// The decoder and S above take every granularity (their KIND parameter); the quantizer above is
// the one for one threshold/scale per 4096-tile.  Below: the quantizers of the other
// granularities and the passes that buckets spanning tiles need.
//   * buckets of 64 .. 2048 coordinates lie inside a tile: bucket j of a tile is the segment of
//     seg = bucket/16 consecutive code words, its compact stream starts at word j*seg of the
//     tile's 256 words, and a word's codes start at (selected components of its bucket before it);
//   * buckets above 4096, and one scale for a vector of several tiles (the 32 + d + 2k bit
//     message of the Encode paragraph), span tiles: a first pass counts every tile's selected
//     components, a scan per bucket turns the counts into each tile's first position in the
//     bucket's stream (kept in the workspace), and the tiles then place or fetch their codes
//     there.  Neighbouring tiles share stream words: the tile in which such a word begins stores
//     it, and a small kernel adds what the others have left in the workspace.

// the 16 indicator bits of the thread's coordinates, without those at or beyond d
__device__ __forceinline__ uint32_t live_mask16(const SelArgs& a, const uint32_t* ind, int64_t tile, int t) {
  const int64_t left = a.d - (tile * kTile + 16 * (int64_t)t);
  const uint32_t m = mask16_of(ind, a.NW, tile, t);
  return left >= 16 ? m : (left > 0 ? (m & ((1u << left) - 1u)) : 0u);
}

// the thread's 16 gradient components (coordinates 16t .. 16t+15 of the tile), 0 beyond d
__device__ __forceinline__ void load16(const float* __restrict__ g, int64_t d, int64_t i0, float v[16]) {
  if (i0 + 16 <= d) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 f = *reinterpret_cast<const float4*>(g + i0 + 4 * q);
      v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
    }
  } else {
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = (i0 + j < d) ? g[i0 + j] : 0.0f;
  }
}

// Where the thread's selected codes sit inside a tile whose buckets are segments of a.seg threads.
struct StreamPos {
  uint32_t pos;        // this thread's first selected code, counted from the tile's word 0
  uint32_t in_bucket;  // selected components of the thread's bucket
};

// n = number of selected components of this thread.  Contains barriers.
__device__ __forceinline__ StreamPos stream_position(const SelArgs& a, uint32_t n, uint32_t* lds_w,
                                                     uint32_t* lds_ex) {
  StreamPos p;
  const int t = threadIdx.x;
  uint32_t in_tile;
  const uint32_t ex = block_exclusive_scan(n, lds_w, &in_tile);
  lds_ex[t] = ex;
  if (t == 0) lds_ex[kThreads] = in_tile;
  __syncthreads();
  const int s0 = t & ~(a.seg - 1);
  p.in_bucket = lds_ex[s0 + a.seg] - lds_ex[s0];
  p.pos = 16u * (uint32_t)s0 + (ex - lds_ex[s0]);
  return p;
}

// OR `bits` (2*n bits) into the LDS stream at code position pos.
__device__ __forceinline__ void stream_append(uint32_t* stream, uint32_t pos, uint32_t n, uint32_t bits) {
  if (n == 0) return;
  const uint32_t word = pos / 16, sh = 2 * (pos % 16);
  atomicOr(&stream[word], bits << sh);
  if (sh && (2 * n + sh > 32)) atomicOr(&stream[word + 1], bits >> (32 - sh));
}

// pass 1 of the multi-tile quantizer: selected components of every tile and the sum of their
// magnitudes
__global__ __launch_bounds__(kThreads) void gsel_count_kernel(SelArgs a) {
  __shared__ uint32_t lds_w[kWaves];
  __shared__ double lds_d[kWaves];
  const int t = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  const uint32_t mask = live_mask16(a, a.ind_in + (int64_t)m * a.ind_stride, tile, t);
  uint32_t K;
  block_exclusive_scan((uint32_t)__popc(mask), lds_w, &K);
  float v[16];
  load16(a.g + (int64_t)m * a.g_stride, a.d, tile * kTile + 16 * (int64_t)t, v);
  double s1 = 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if ((mask >> j) & 1u) s1 += (double)fabsf(v[j]);
  const double S1 = block_sum_f64(s1, lds_d);
  if (t == 0) {
    a.ws_s1[(int64_t)m * a.ntiles + tile] = S1;
    a.ws_count[(int64_t)m * a.ntiles + tile] = K;
  }
}

// pass 1 without a gradient (decoder, S of a coded message): a wave counts kCountTiles
// consecutive tiles, lane l the indicator words 2l and 2l+1 of each tile (bits at or beyond d
// are not components).
constexpr int kCountTiles = 8;
__global__ __launch_bounds__(kThreads) void gsel_count_ind_kernel(SelArgs a) {
  const int lane = threadIdx.x % kWave;
  const int64_t tile0 = ((int64_t)blockIdx.x * kWaves + threadIdx.x / kWave) * kCountTiles;
  const int m = blockIdx.y;
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride;
  uint32_t c[kCountTiles];
#pragma unroll
  for (int u = 0; u < kCountTiles; ++u) {
    c[u] = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t iw = (tile0 + u) * (kTile / 32) + 2 * lane + h;
      uint32_t v = iw < a.NW ? ind[iw] : 0u;
      const int64_t left = a.d - 32 * iw;
      if (left < 32) v = left > 0 ? (v & ((1u << left) - 1u)) : 0u;
      c[u] += (uint32_t)__popc(v);
    }
  }
#pragma unroll
  for (int u = 0; u < kCountTiles; ++u) {
    const uint32_t K = wave_sum_u32(c[u]);
    if (lane == 0 && tile0 + u < a.ntiles) a.ws_count[(int64_t)m * a.ntiles + tile0 + u] = K;
  }
}

// pass 2: per (bucket, worker), in tile order: each tile's first position in the bucket's stream,
// the bucket's count and (with the tiles' sums) its threshold.  One work-group per bucket; a round
// takes THREADS x 8 consecutive tiles (thread t the 8 from t*8 on) with a running offset, so the
// order of the binary64 additions is fixed.  A wave for buckets of up to 512 tiles (one round), else 1024
// threads.  Bound by the rounds' chain of a load and a barrier: 8 x 32768 tiles 13 us, with 256 threads of 16 guarded loads 35.
constexpr int kScanRun = 8;
template <bool HAS_G, int THREADS>
__global__ __launch_bounds__(THREADS) void gsel_scan_kernel(SelArgs a) {
  constexpr int kScanThreads = THREADS, kScanWaves = THREADS / kWave;
  __shared__ uint32_t lds_w[kScanWaves];
  __shared__ double lds_d[kScanWaves];
  const int t = threadIdx.x, lane = t % kWave, wave = t / kWave;
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t t0 = k * a.tiles_per_bucket;
  const int64_t t1 = t0 + a.tiles_per_bucket < a.ntiles ? t0 + a.tiles_per_bucket : a.ntiles;
  const uint32_t* cnt = a.ws_count + (int64_t)m * a.ntiles;
  const double* s1p = a.ws_s1 + (int64_t)m * a.ntiles;
  int64_t* start = a.ws_start + (int64_t)m * a.ntiles;
  int64_t running = 0;
  double s1 = 0.0;
  for (int64_t i = t0; i < t1; i += (int64_t)kScanThreads * kScanRun) {
    const int64_t j0 = i + (int64_t)t * kScanRun;
    uint32_t c[kScanRun], mine = 0;
    double v[kScanRun];
    if (j0 + kScanRun <= t1) {                           // all loads together
#pragma unroll
      for (int u = 0; u < kScanRun; ++u) c[u] = cnt[j0 + u];
#pragma unroll
      for (int u = 0; u < kScanRun; ++u) v[u] = HAS_G ? s1p[j0 + u] : 0.0;
    } else {
#pragma unroll
      for (int u = 0; u < kScanRun; ++u) {
        c[u] = j0 + u < t1 ? cnt[j0 + u] : 0u;
        v[u] = HAS_G && j0 + u < t1 ? s1p[j0 + u] : 0.0;
      }
    }
#pragma unroll
    for (int u = 0; u < kScanRun; ++u) {
      mine += c[u];
      if (HAS_G) s1 += v[u];
    }
    const uint32_t incl = wave_scan_u32(mine);
    __syncthreads();                                     // the previous round's totals have been read
    if (lane == kWave - 1) lds_w[wave] = incl;
    __syncthreads();
    uint32_t ex = incl - mine, total = 0;                // at most 1024 x 8 x 4096 = 2^25
#pragma unroll
    for (int w = 0; w < kScanWaves; ++w) {
      const uint32_t x = lds_w[w];
      if (w < wave) ex += x;
      total += x;
    }
    int64_t from = running + ex;
    if (j0 + kScanRun <= t1) {
#pragma unroll
      for (int u = 0; u < kScanRun; ++u) { start[j0 + u] = from; from += c[u]; }
    } else {
#pragma unroll
      for (int u = 0; u < kScanRun; ++u) {
        if (j0 + u < t1) start[j0 + u] = from;
        from += c[u];
      }
    }
    running += total;
  }
  if (HAS_G) {
    s1 = wave_sum_f64(s1);
    if (lane == 0) lds_d[wave] = s1;
    __syncthreads();
  }
  if (t == 0) {
    a.counts[(int64_t)m * a.scale_stride + k] = (uint32_t)running;   // a bucket holds < 2^32 here
    if (HAS_G) {
      double S1 = 0.0;
      for (int w = 0; w < kScanWaves; ++w) S1 += lds_d[w];
      const float Delta = running ? threshold_from_sum(S1, a.thr_coef, running) : 0.0f;
      a.ws_thr[(int64_t)m * a.nb + k] = Delta;
      if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + k] = Delta;
    }
  }
}

// A word of the stream that several tiles share is stored by the tile it begins in; the others leave their
// part of it, their head, in the slot of their count, and this kernel adds the heads (where their bits are 0, or hold
// what the settling pass exchanges).  A thread per tile:
// 9 to 11 us for 8 workers x 2^27.  Two atomic ORs per tile among the stores of the coders themselves, into words zeroed
// before, cost 0.4 ms there (the quantizer 1.11 -> 0.70 ms without them, S of a coded message 0.25 -> 0.19 as a whole).
__global__ __launch_bounds__(kThreads) void gsel_join_kernel(SelArgs a) {
  const int64_t tile = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (tile >= a.ntiles) return;
  const int m = blockIdx.y;
  const int64_t k = tile / a.tiles_per_bucket, at = (int64_t)m * a.ntiles + tile;
  const uint32_t head = a.ws_count[at];
  if (head) atomicXor(&a.sel_codes[(int64_t)m * a.code_stride + k * a.area_words + (a.ws_start[at] >> 4)], head);
}
// Q(S(g, I)) for buckets of 64 .. 2048 coordinates: thread t = code word t of the tile, a bucket =
// a.seg consecutive threads.
__global__ __launch_bounds__(kThreads) void gsel_quantize_local_kernel(SelArgs a) {
  __shared__ uint32_t stream[kTileWords + 2];
  __shared__ uint32_t lds_w[kWaves];
  __shared__ uint32_t lds_ex[kThreads + 1];
  __shared__ double lds_d[kWaves];
  __shared__ uint32_t lds_u[kWaves];
  const int t = threadIdx.x;
  const int64_t tile = blockIdx.x;
  const int m = blockIdx.y;
  const float* g = a.g + (int64_t)m * a.g_stride;
  const uint32_t mask = live_mask16(a, a.ind_in + (int64_t)m * a.ind_stride, tile, t);
  float v[16];
  load16(g, a.d, tile * kTile + 16 * (int64_t)t, v);
  stream[t] = 0u;
  if (t < 2) stream[kTileWords + t] = 0u;
  const uint32_t n = (uint32_t)__popc(mask);
  const StreamPos p = stream_position(a, n, lds_w, lds_ex);   // barriers: stream is zero

  double s1 = 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if ((mask >> j) & 1u) s1 += (double)fabsf(v[j]);
  const double S1 = segment_sum(s1, a.seg, lds_d);
  const float Delta = p.in_bucket ? threshold_from_sum(S1, a.thr_coef, (int64_t)p.in_bucket) : 0.0f;
  double s2 = 0.0;
  uint32_t c2 = 0, bits = 0, k = 0;
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    if ((mask >> j) & 1u) {
      const float av = fabsf(v[j]);
      if (av > Delta) { s2 += (double)av; ++c2; }
      bits |= ternary_field(v[j], Delta) << (2 * k);
      ++k;
    }
  }
  stream_append(stream, p.pos, n, bits);
  __syncthreads();                                       // lds_d of the first sum has been read
  const double S2 = segment_sum(s2, a.seg, lds_d);
  const uint32_t C2 = segment_sum_u32(c2, a.seg, lds_u);
  __syncthreads();                                       // the stream is complete
  // the first ceil(K/16) words of each bucket's area, nothing else
  const int s0 = t & ~(a.seg - 1);
  uint32_t* row = a.sel_codes + (int64_t)m * a.code_stride + tile * kTileWords;
  if ((uint32_t)(t - s0) < (p.in_bucket + 15) / 16) row[t] = stream[t];
  if (t == s0) {
    const int64_t kb = (tile * kTile + 16 * (int64_t)t) / (16 * (int64_t)a.seg);
    if (kb < a.nb) {
      a.counts[(int64_t)m * a.scale_stride + kb] = p.in_bucket;
      a.scales[(int64_t)m * a.scale_stride + kb] = scale_from_sum(S2, C2);
      if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + kb] = Delta;
    }
  }
}

// Q(S(g, I)) of one tile for buckets that span tiles, by one wave (lane l holds code words j*64 + l
// of the tile, j = 0..3, as in the decoder): the tile's codes, in index order, in `stream` (LDS of
// the wave) from code position `first` on; the sums of |v| over the marked (BRACKET) and over the kept
// components and the latter's number per lane.  BRACKET: components up to `lo` get 0, above `hi` their
// code, those between the pattern 10.
// Bound by vector instructions (1500 per tile; 8 workers x 2^27: 0.77 ms without the list, 0.84 with it, which
// the settling pass returns four times over).  Slower were nontemporal loads (four lanes of a 64-byte stride share
// every line) and selecting in place of the branch around an unmarked component.
// Open components are listed, value and place in the tile's codes, as long as the tile's slots last.
constexpr uint32_t kOpenSlots = 16, kOpenUnlisted = 31;
struct TileCodes {
  double s1, s2;
  uint32_t c2, end, open;                                // end: one past the tile's last code
};
__device__ __forceinline__ void list_open(uint2* list, bool open, float x, uint32_t place, uint32_t* listed) {
  const uint64_t some = __ballot(open);
  if (some == 0) return;                                 // uniform
  const uint32_t slot = *listed + __builtin_amdgcn_mbcnt_hi((uint32_t)(some >> 32),
                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)some, 0u));
  if (open && slot < kOpenSlots) list[slot] = make_uint2(__float_as_uint(x), place);
  *listed += (uint32_t)__popcll(some);
}
template <bool BRACKET>
__device__ __forceinline__ TileCodes code_selected_tile(const SelArgs& a, int64_t tile, int m, uint32_t first,
                                                        float lo, float hi, uint32_t* stream, uint2* open_list) {
  const int lane = threadIdx.x % kWave;
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride;
  const float* g = a.g + (int64_t)m * a.g_stride;
#pragma unroll
  for (int j = 0; j < 4; ++j) stream[j * 64 + lane] = 0u;
  if (lane < 2) stream[kTileWords + lane] = 0u;
  wave_fence();
  TileCodes r{0.0, 0.0, 0u, first, 0u};
#pragma unroll 1
  for (int half = 0; half < 4; half += 2) {
    uint32_t mask[2], incl[2];
    float v[2][16];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int wl = (half + h) * 64 + lane;
      const int64_t iw = tile * (kTile / 32) + wl / 2;
      const uint32_t iv = iw < a.NW ? ind[iw] : 0u;
      mask[h] = (iv >> (16 * (wl & 1))) & 0xFFFFu;
      const int64_t left = a.d - (tile * kTile + (int64_t)wl * 16);
      if (left < 16) mask[h] = left > 0 ? (mask[h] & ((1u << left) - 1u)) : 0u;
      load16(g, a.d, tile * kTile + (int64_t)wl * 16, v[h]);
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) incl[h] = wave_scan_u32((uint32_t)__popc(mask[h]));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t n = (uint32_t)__popc(mask[h]);
      const uint32_t before = r.end + incl[h] - n;
      r.end += (uint32_t)__builtin_amdgcn_readlane((int)incl[h], kWave - 1);
      uint32_t bits = 0, filled = 0;
#pragma unroll
      for (int c = 0; c < 16; ++c) {
        bool open = false;
        const uint32_t place = before - first + filled / 2;
        if ((mask[h] >> c) & 1u) {
          const float av = fabsf(v[h][c]);
          uint32_t f;
          if (BRACKET) {
            r.s1 += (double)av;
            const bool keep = av > hi;
            if (keep) { r.s2 += (double)av; ++r.c2; }
            open = av > lo && !keep;
            f = keep ? 1u | ((__float_as_uint(v[h][c]) >> 30) & 2u) : (open ? 2u : 0u);
          } else {
            if (av > lo) { r.s2 += (double)av; ++r.c2; }
            f = ternary_field(v[h][c], lo);
          }
          bits |= f << filled;
          filled += 2;
        }
        if (BRACKET) list_open(open_list, open, v[h][c], place, &r.open);
      }
      if (n) {
        const uint32_t w0 = before / 16, sh = 2 * (before % 16);
        atomicOr(&stream[w0], bits << sh);
        if (sh && 2 * n + sh > 32) atomicOr(&stream[w0 + 1], bits >> (32 - sh));
      }
    }
  }
  r.s1 = wave_sum_f64(r.s1);
  r.s2 = wave_sum_f64(r.s2);
  r.c2 = wave_sum_u32(r.c2);
  wave_fence();
  return r;
}

// The same for a tile of at most kFewMarked marked components, in two steps that leave the others out: the
// wave reads the tile 16 bytes per lane side by side and drops the marked values into LDS at their place in
// the stream, then takes them 64 at a time, sixteen neighbours to a code word.  Unmarked values go to a slot
// that nobody reads: as many instructions as a branch, and the loads of LDS stay in one piece.  Bound by the
// read of the gradient: 8 workers x 2^27, 7 % marked, 0.69 ms for 4.4 GB (the other form 0.77).  The line: LDS
// for 1520 lets five work-groups share a CU, and two rounds of 64 cost more than the other form's words from
// there on (30 / 45 / 97 % marked, the whole call with a line at 1520 / 2032 / 4096: 900 / 934 / 1248, 1010 /
// 1034 / 1498 and 1068 / 1072 / 2368 us).
constexpr uint32_t kFewMarked = 1520, kFewCodes = 1536;  // with 15 codes of a shared first word
struct SelWaveLds {
  uint2 words[kTile / 32];                               // indicator word, codes before it
  union { float vals[kFewCodes + kWave]; uint32_t stream[kTileWords + 2]; };
};
template <bool BRACKET>
__device__ __forceinline__ TileCodes code_few_marked(const SelArgs& a, int64_t tile, int m, uint32_t first,
                                                     float lo, float hi, SelWaveLds& lds, uint32_t* out,
                                                     uint2* open_list, uint32_t* head) {
  const int lane = threadIdx.x % kWave;
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride;
  const float* g = a.g + (int64_t)m * a.g_stride;
  uint32_t iv[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t iw = tile * (kTile / 32) + 2 * lane + h;
    iv[h] = iw < a.NW ? ind[iw] : 0u;
    const int64_t left = a.d - 32 * iw;
    if (left < 32) iv[h] = left > 0 ? (iv[h] & ((1u << left) - 1u)) : 0u;
  }
  const uint32_t n0 = (uint32_t)__popc(iv[0]), n1 = (uint32_t)__popc(iv[1]);
  const uint32_t incl = wave_scan_u32(n0 + n1);
  const uint32_t ex = first + incl - n0 - n1;
  lds.words[2 * lane] = make_uint2(iv[0], ex);
  lds.words[2 * lane + 1] = make_uint2(iv[1], ex + n0);
  TileCodes r{0.0, 0.0, 0u, first + (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1), 0u};
  wave_fence();
  const uint32_t sh = 4 * (lane & 7), below = (1u << sh) - 1u;
  typedef float floatx4 __attribute__((ext_vector_type(4)));
#pragma unroll 1
  for (int j0 = 0; j0 < 16; j0 += 8) {
    floatx4 v[8];
    if ((tile + 1) * kTile <= a.d) {
      const floatx4* src = reinterpret_cast<const floatx4*>(g + tile * kTile) + j0 * kWave + lane;
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = __builtin_nontemporal_load(src + j * kWave);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t i = tile * kTile + ((j0 + j) * kWave + lane) * 4 + e;
          v[j][e] = i < a.d ? g[i] : 0.0f;
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const uint2 w = lds.words[8 * (j0 + j) + (lane >> 3)];
      const uint32_t nib = w.x >> sh;
      uint32_t pos = w.y + (uint32_t)__popc(w.x & below);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool marked = (nib & (1u << e)) != 0u;
        lds.vals[marked ? pos : kFewCodes + lane] = v[j][e];
        pos += marked ? 1u : 0u;
      }
    }
  }
  wave_fence();
  uint32_t mine = 0;
  const uint32_t nwords = r.end != first ? (r.end + 15) / 16 : 0u;
  for (uint32_t p0 = 0, q = 0; p0 < r.end; p0 += kWave, ++q) {
    const uint32_t p = p0 + lane;
    const float x = p >= first && p < r.end ? lds.vals[p] : 0.0f;
    const float av = fabsf(x);
    uint32_t f;
    if (BRACKET) {
      const bool keep = av > hi, open = av > lo && !keep;
      r.s1 += (double)av;
      r.s2 += (double)(keep ? av : 0.0f);
      r.c2 += (uint32_t)__popcll(__ballot(keep));
      f = keep ? 1u | ((__float_as_uint(x) >> 30) & 2u) : (open ? 2u : 0u);
      list_open(open_list, open, x, p - first, &r.open);
    } else {
      const bool keep = av > lo;
      r.s2 += (double)(keep ? av : 0.0f);
      r.c2 += (uint32_t)__popcll(__ballot(keep));
      f = ternary_field(x, lo);
    }
    uint32_t w = f << (2 * (lane & 15));                 // the sixteen codes of a word: a row of lanes
    w |= (uint32_t)dpp_i32<kDppQuadXor1>((int)w);
    w |= (uint32_t)dpp_i32<kDppQuadXor2>((int)w);
    w |= (uint32_t)dpp_i32<kDppRowHalfMirror>((int)w);
    w |= (uint32_t)dpp_i32<kDppRowMirror>((int)w);
    if ((uint32_t)(lane & 15) == (q & 15u)) mine = w;
    if ((q & 15u) == 15u || p0 + kWave >= r.end) {       // 64 words, or the last ones
      const uint32_t wl = (q >> 4) * kWave + 4 * (lane & 15) + (lane >> 4);
      if (wl < nwords) store_word(out, wl, first, mine, head);   // word 0: lane 0
    }
  }
  r.s1 = wave_sum_f64(r.s1);
  r.s2 = wave_sum_f64(r.s2);
  return r;
}

// The assembled codes of a tile to their place in the bucket's stream, its kept sum and count to the
// workspace.  BRACKET: the one pass of the one-read form below; else the threshold comes from pass 2.
// (Five waves per SIMD are what the LDS allows.)
template <bool BRACKET>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(5))) void gsel_quantize_multi_kernel(SelArgs a) {
  __shared__ SelWaveLds lds_all[kWaves];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const int64_t tile = (int64_t)blockIdx.x * kWaves + wave;
  if (tile >= a.ntiles) return;
  const int m = blockIdx.y;
  const int64_t at = (int64_t)m * a.ntiles + tile, k = tile / a.tiles_per_bucket;
  const int64_t st = a.ws_start[at];
  const uint32_t marked = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ws_count[at]);
  const uint32_t first = (uint32_t)(st & 15);
  const float thr = a.ws_thr[(int64_t)m * a.nb + k];
  const float lo = BRACKET ? a.scales[(int64_t)m * a.scale_stride + k] : thr;
  if (BRACKET && !(lo >= 0.0f)) {                        // no bracket: the marked sum only
    float v[2][16];
    uint32_t mask[4];
    double s1 = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) mask[j] = live_mask16(a, a.ind_in + (int64_t)m * a.ind_stride, tile, j * 64 + lane);
#pragma unroll 1
    for (int half = 0; half < 4; half += 2) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        load16(a.g + (int64_t)m * a.g_stride, a.d, tile * kTile + (int64_t)((half + h) * 64 + lane) * 16, v[h]);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t mk = half ? mask[2 + h] : mask[h];
#pragma unroll
        for (int c = 0; c < 16; ++c)
          if ((mk >> c) & 1u) s1 += (double)fabsf(v[h][c]);
      }
    }
    s1 = wave_sum_f64(s1);
    if (lane == 0) a.ws_s1[at] = s1;
    return;
  }
  uint32_t* out = a.sel_codes + (int64_t)m * a.code_stride + k * a.area_words + (st >> 4);
  TileCodes r;
  uint2* open_list = BRACKET ? a.ws_open + at * kOpenSlots : nullptr;
  uint32_t head = 0;
  if (marked <= kFewMarked) {
    r = code_few_marked<BRACKET>(a, tile, m, first, lo, thr, lds_all[wave], out, open_list, &head);
  } else {
    uint32_t* stream = lds_all[wave].stream;
    r = code_selected_tile<BRACKET>(a, tile, m, first, lo, thr, stream, open_list);
    const uint32_t nwords = (r.end + 15) / 16;
    for (uint32_t w = lane; w < nwords; w += kWave) store_word(out, w, first, stream[w], &head);   // at most 257 words
  }
  if (lane == 0) {
    a.ws_count[at] = head;                               // lane 0 has word 0
    if (BRACKET) a.ws_s1[at] = r.s1;
    a.ws_s2[at] = r.s2;
    a.ws_c2[at] = r.c2 | ((r.open <= kOpenSlots ? r.open : kOpenUnlisted) << 16);
  }
}

// ---- long buckets in one read -------------------------------------------------------------------
//
// As for the dense quantizer: the marked components' numbers come from the indicators alone, every 64th
// tile gives a bracket around the threshold (five standard errors to either side of the sampled ratio
// sum / number, at most 8 %), the one pass writes final codes outside the bracket and the pattern
// 10 inside it, and the settling pass looks the open components up once the threshold is known.
// Until the scales are known, scales[] carries the bracket's lower end (-1: there is none, and the pass forms
// the sum alone) and then whether it held the threshold (0 / 1), ws_thr its upper end and then the threshold.
constexpr int kSelSampleEvery = 64;
constexpr double kSelWidestBand = 0.08;

__device__ __forceinline__ int64_t sampled_tile(const SelArgs& a, int64_t k, int64_t i) {
  return k * a.tiles_per_bucket + i * kSelSampleEvery + (i * 29) % kSelSampleEvery;
}
__device__ __forceinline__ int64_t samples_of(const SelArgs& a, int64_t k) {
  const int64_t all = a.ntiles - k * a.tiles_per_bucket;
  return (all < a.tiles_per_bucket ? all : a.tiles_per_bucket) / kSelSampleEvery;
}

__global__ __launch_bounds__(kThreads) void gsel_sample_kernel(SelArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t k = blockIdx.x / a.samples, i = blockIdx.x % a.samples;
  const int m = blockIdx.y;
  if (i >= samples_of(a, k)) return;
  const int64_t tile = sampled_tile(a, k, i);
  const uint32_t mask = live_mask16(a, a.ind_in + (int64_t)m * a.ind_stride, tile, threadIdx.x);
  float v[16];
  load16(a.g + (int64_t)m * a.g_stride, a.d, tile * kTile + 16 * (int64_t)threadIdx.x, v);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j)
    if ((mask >> j) & 1u) s += (double)fabsf(v[j]);
  s = block_sum_f64(s, lds_d);
  if (threadIdx.x == 0) a.ws_s2[(int64_t)m * a.ntiles + k * a.samples + i] = s;
}

__global__ __launch_bounds__(kThreads) void gsel_band_kernel(SelArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const double* part = a.ws_s2 + (int64_t)m * a.ntiles + k * a.samples;
  const uint32_t* cnt = a.ws_count + (int64_t)m * a.ntiles;
  const int64_t n = samples_of(a, k);
  double sum = 0.0, num = 0.0, diff = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += kThreads) { sum += part[i]; num += (double)cnt[sampled_tile(a, k, i)]; }
  sum = segment_sum(sum, kThreads, lds_d);
  num = segment_sum(num, kThreads, lds_d);
  const double ratio = num > 0.0 ? sum / num : 0.0;
  // residuals against the ratio, neighbouring samples (trends along the vector drop out)
  for (int64_t i = threadIdx.x; i + 1 < n; i += kThreads) {
    const double e = (part[i + 1] - ratio * (double)cnt[sampled_tile(a, k, i + 1)]) -
                     (part[i] - ratio * (double)cnt[sampled_tile(a, k, i)]);
    diff += e * e;
  }
  diff = segment_sum(diff, kThreads, lds_d);
  if (threadIdx.x == 0) {
    float lo = -1.0f, hi = -1.0f;                        // no bracket
    if (n >= 16 && ratio > 0.0) {
      const double rel = 5.0 * sqrt(diff / (2.0 * (double)(n - 1)) * (double)n) / sum + 1e-6;
      const double mid = (double)a.thr_coef * ratio;
      if (rel < kSelWidestBand && mid < 1e38) { lo = (float)(mid * (1.0 - rel)); hi = (float)(mid * (1.0 + rel)); }
    }
    a.scales[(int64_t)m * a.scale_stride + k] = lo;
    a.ws_thr[(int64_t)m * a.nb + k] = hi;
  }
}

__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void gsel_threshold_kernel(SelArgs a) {
  __shared__ double lds_d[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t t0 = k * a.tiles_per_bucket;
  const int64_t t1 = t0 + a.tiles_per_bucket < a.ntiles ? t0 + a.tiles_per_bucket : a.ntiles;
  double s = strided_partial_sum(a.ws_s1 + (int64_t)m * a.ntiles, t0, t1);
  s = segment_sum(s, kThreads, lds_d);
  if (threadIdx.x == 0) {
    const int64_t K = a.counts[(int64_t)m * a.scale_stride + k];
    const float Delta = K ? threshold_from_sum(s, a.thr_coef, K) : 0.0f;
    float* lo = a.scales + (int64_t)m * a.scale_stride + k;
    float* thr = a.ws_thr + (int64_t)m * a.nb + k;
    if (*lo >= 0.0f) *lo = Delta >= *lo && Delta <= *thr ? 1.0f : 0.0f;
    *thr = Delta;
    if (a.thresholds) a.thresholds[(int64_t)m * a.scale_stride + k] = Delta;
  }
}

// A tile whose open components are not listed, by a wave.  With a bracket that held: each lane reads its
// words' codes back from the stream, finds the pattern 10, and exchanges it for the component's code in
// place; its head is not joined yet.  Without a bracket the tile is coded here, and with one that missed again; of a
// word that it shares with a neighbour then only its own bits change, the head's among them.
__device__ __forceinline__ void settle_tile(const SelArgs& a, int64_t tile, int m, SelWaveLds& lds) {
  const int lane = threadIdx.x % kWave;
  const int64_t slot = (int64_t)m * a.ntiles + tile, k = tile / a.tiles_per_bucket;
  const float D = a.ws_thr[(int64_t)m * a.nb + k], held = a.scales[(int64_t)m * a.scale_stride + k];
  const int64_t st = a.ws_start[slot];
  const uint32_t first = (uint32_t)(st & 15);
  uint32_t* out = a.sel_codes + (int64_t)m * a.code_stride + k * a.area_words + (st >> 4);
  if (held != 1.0f) {
    uint32_t head = 0;
    TileCodes r;
    uint32_t* stream = lds.stream;
    // without a bracket the count of the tile's marks is still in the head's slot
    const bool few = held < 0.0f && (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ws_count[slot]) <= kFewMarked;
    if (few) r = code_few_marked<false>(a, tile, m, first, D, 0.0f, lds, out, nullptr, &head);
    else r = code_selected_tile<false>(a, tile, m, first, D, 0.0f, stream, nullptr);
    const uint32_t nwords = (r.end + 15) / 16;
    if (!few && r.end != first)
      for (uint32_t w = lane; w < nwords; w += kWave) {
        uint32_t own = 0xffffffffu;
        if (w == 0 && first != 0) own &= 0xffffffffu << (2 * first);
        if (w == nwords - 1 && (r.end % 16) != 0) own &= ~(0xffffffffu << (2 * (r.end % 16)));
        if (held < 0.0f) store_word(out, w, first, stream[w], &head);
        else if (own == 0xffffffffu) out[w] = stream[w];
        else atomicXor(&out[w], (atomicOr(&out[w], 0u) ^ stream[w]) & own);
      }
    if (lane == 0) { a.ws_s2[slot] = r.s2; a.ws_c2[slot] = r.c2; a.ws_count[slot] = head; }
    return;
  }
  const uint32_t* ind = a.ind_in + (int64_t)m * a.ind_stride;
  const float* g = a.g + (int64_t)m * a.g_stride;
  uint32_t mask[4], at[4], open[4], any = 0, start = first;
  const uint32_t head = a.ws_count[slot];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int wl = j * 64 + lane;
    const int64_t iw = tile * (kTile / 32) + wl / 2;
    const uint32_t iv = iw < a.NW ? ind[iw] : 0u;
    mask[j] = (iv >> (16 * (wl & 1))) & 0xFFFFu;
    const int64_t left = a.d - (tile * kTile + (int64_t)wl * 16);
    if (left < 16) mask[j] = left > 0 ? (mask[j] & ((1u << left) - 1u)) : 0u;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t n = (uint32_t)__popc(mask[j]), incl = wave_scan_u32(n);
    at[j] = start + incl - n;
    start += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
    uint32_t lo = 0u, hi = 0u;
    const uint32_t w0 = at[j] / 16, sh = 2 * (at[j] % 16);
    if (n) lo = w0 == 0 ? out[0] | head : out[w0];
    if (sh && 2 * n + sh > 32) hi = out[w0 + 1];
    uint32_t bits = (lo >> sh) | (sh ? hi << (32 - sh) : 0u);
    if (n < 16) bits &= (1u << (2 * n)) - 1u;
    open[j] = (bits >> 1) & ~bits & 0x55555555u;         // low bit of every code 10
    any |= open[j];
  }
  const double s_before = a.ws_s2[slot];                 // the tile's sums, to be added to
  const uint32_t c_before = a.ws_c2[slot] & 0xFFFFu;
  double s = 0.0;
  uint32_t c = 0;
  while (__any(any != 0)) {                              // a code of every word at a time
    any = 0;
    float x[4];
    uint32_t f[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      f[j] = open[j] ? (uint32_t)(__ffs((int)open[j]) - 1) / 2 : 16u;    // the f-th marked component
      x[j] = 0.0f;
      if (f[j] < 16u) {
        uint32_t left = mask[j];
        for (uint32_t q = 0; q < f[j]; ++q) left &= left - 1u;
        x[j] = g[tile * kTile + (int64_t)(j * 64 + lane) * 16 + (__ffs((int)left) - 1)];
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (f[j] < 16u) {
        const float av = fabsf(x[j]);
        if (av > D) { s += (double)av; ++c; }
        const uint32_t place = at[j] + f[j];
        atomicXor(&out[place / 16], (2u ^ ternary_field(x[j], D)) << (2 * (place % 16)));
        open[j] &= open[j] - 1u;
        any |= open[j];
      }
  }
  s = wave_sum_f64(s);
  c = wave_sum_u32(c);
  if (lane == 0) { a.ws_s2[slot] = s_before + s; a.ws_c2[slot] = c_before + c; }
}

// A wave for four tiles, sixteen lanes for the listed components of each: everything that a tile needs is
// requested at once.  Tiles without a list follow one by one.  8 workers x 2^27: 30 us; reading
// every tile's marks and codes back took 180, a chain of dependent loads per tile.
__global__ __launch_bounds__(kThreads) void gsel_settle_kernel(SelArgs a) {
  __shared__ SelWaveLds lds_all[kWaves];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, e = lane % (int)kOpenSlots;
  constexpr int kTilesPerWave = kWave / (int)kOpenSlots;
  const int64_t tile0 = ((int64_t)blockIdx.x * kWaves + wave) * kTilesPerWave, tile = tile0 + lane / (int)kOpenSlots;
  const int m = blockIdx.y;
  bool listed = false, unlisted = false, keep = false;
  float av = 0.0f;
  double s_before = 0.0;
  uint32_t c_before = 0;
  const int64_t slot = (int64_t)m * a.ntiles + tile;
  if (tile < a.ntiles) {
    const int64_t k = tile / a.tiles_per_bucket;
    const float D = a.ws_thr[(int64_t)m * a.nb + k], held = a.scales[(int64_t)m * a.scale_stride + k];
    const int64_t st = a.ws_start[slot];
    const uint32_t c = a.ws_c2[slot];
    const uint2 entry = a.ws_open[slot * kOpenSlots + e];
    s_before = a.ws_s2[slot];
    c_before = c & 0xFFFFu;
    const uint32_t n = c >> 16;
    unlisted = held != 1.0f || n > kOpenSlots;
    listed = !unlisted && n > 0;
    if (listed && (uint32_t)e < n) {
      const float x = __uint_as_float(entry.x);
      av = fabsf(x);
      keep = av > D;
      const int64_t place = st + entry.y;
      uint32_t* area = a.sel_codes + (int64_t)m * a.code_stride + k * a.area_words;
      atomicXor(&area[place >> 4], (2u ^ ternary_field(x, D)) << (2 * (uint32_t)(place & 15)));
    }
  }
  double s = keep ? (double)av : 0.0;
  uint32_t c = keep ? 1u : 0u;
  s += dpp_f64<kDppQuadXor1>(s);       c += (uint32_t)dpp_i32<kDppQuadXor1>((int)c);
  s += dpp_f64<kDppQuadXor2>(s);       c += (uint32_t)dpp_i32<kDppQuadXor2>((int)c);
  s += dpp_f64<kDppRowHalfMirror>(s);  c += (uint32_t)dpp_i32<kDppRowHalfMirror>((int)c);
  s += dpp_f64<kDppRowMirror>(s);      c += (uint32_t)dpp_i32<kDppRowMirror>((int)c);
  if (listed && e == 0) { a.ws_s2[slot] = s_before + s; a.ws_c2[slot] = c_before + c; }
  for (uint64_t left = __ballot(unlisted && e == 0); left; left &= left - 1) {
    wave_fence();                                        // the stream of the tile before has been read
    settle_tile(a, tile0 + (__ffsll((unsigned long long)left) - 1) / (int)kOpenSlots, m, lds_all[wave]);
  }
}

// last pass of the multi-tile quantizer: scale of each (bucket, worker)
__global__ __launch_bounds__(kThreads) QA_FEW_WAVES void gsel_scale_kernel(SelArgs a) {
  __shared__ double lds_d[kWaves];
  __shared__ double lds_c[kWaves];
  const int64_t k = blockIdx.x;
  const int m = blockIdx.y;
  const int64_t t0 = k * a.tiles_per_bucket;
  const int64_t t1 = t0 + a.tiles_per_bucket < a.ntiles ? t0 + a.tiles_per_bucket : a.ntiles;
  double s, c;
  strided_partial_sums(a.ws_s2 + (int64_t)m * a.ntiles, a.ws_c2 + (int64_t)m * a.ntiles, t0, t1, &s, &c);
  s = segment_sum(s, kThreads, lds_d);
  c = segment_sum(c, kThreads, lds_c);
  if (threadIdx.x == 0) a.scales[(int64_t)m * a.scale_stride + k] = scale_from_sum(s, (uint64_t)c);
}

// Buckets of at least 4096 tiles (64 samples) are quantized in one read if all workers have 2^28 coordinates
// or more.  With a bracket it is the faster form from 2^27 on; without one (marks on components of very
// unequal sizes, one mark or none per tile) its small launches and the second coding come on top of two reads, and
// the line lies where that costs no more than a sixth and a bracket gains as much at least.  Two reads / one read with a bracket / one read without, us, for
// 7 % and for 97 % of the components marked: 8 workers x 2^27 1430 / 823 / 1518 and 1612 / 1060 / 1763,
// 8 x 2^25 357 / 226 / 395 and 407 / 357 / 471, 4 x 2^25 183 / 127 / 210 and 215 / 208 / 255, 2 x 2^25 98 / 80 / - and 100 /
// 119 / -.  Shorter buckets have wider brackets: 8 x 2^24 in buckets of 2^22 181 / 148 and 212 / 236.
constexpr int64_t kSelOneReadBucketTiles = 4096, kSelOneReadTiles = 65536;

// Which kernels serve a layout's sparse messages.
static SelKind sel_kind(const qa_layout* L) {
  if (L->bucket == kTile || (L->bucket == 0 && L->d <= kTile)) return kSelTile;   // the tuned kernels
  if (L->bucket != 0 && L->bucket < kTile) return kSelLocal;                        // buckets inside a tile
  return kSelMulti;                                                                 // buckets over several tiles
}

static bool sel_one_read(const qa_layout* L) {
  const int64_t ntiles = tiles_of(L->d), per = L->bucket ? L->bucket / kTile : ntiles;
  return sel_kind(L) == kSelMulti && per >= kSelOneReadBucketTiles && ntiles >= kSelOneReadBucketTiles &&
         ntiles * L->M >= kSelOneReadTiles && buckets_of(L->d, L->bucket) * (per / kSelSampleEvery) <= 0x7fffffffLL;
}

static inline size_t sel_align(size_t v) { return (v + 255) & ~size_t(255); }
template <bool HAS_G>
static void scan_launch(const SelArgs& a, int M, hipStream_t stream) {
  const dim3 buckets((unsigned)a.nb, (unsigned)M);
  if (a.tiles_per_bucket <= kWave * kScanRun)
    hipLaunchKernelGGL((gsel_scan_kernel<HAS_G, kWave>), buckets, dim3(kWave), 0, stream, a);
  else
    hipLaunchKernelGGL((gsel_scan_kernel<HAS_G, 1024>), buckets, dim3(1024), 0, stream, a);
}
static void join_launch(const SelArgs& a, int M, hipStream_t stream) {
  hipLaunchKernelGGL(gsel_join_kernel, dim3((unsigned)((a.ntiles + kThreads - 1) / kThreads), (unsigned)M),
                     dim3(kThreads), 0, stream, a);
}
static inline dim3 count_grid(const qa_layout* L) {
  return dim3((unsigned)((tiles_of(L->d) + kWaves * kCountTiles - 1) / (kWaves * kCountTiles)), (unsigned)L->M);
}

// Workspace of the multi-tile path: per (worker, tile) a count, two binary64 sums, a kept count and
// the tile's first position in its bucket's stream; per (worker, bucket) a threshold.  Quantizers that read
// once also list open components.
size_t select_workspace_bytes(const qa_layout* L) {
  if (sel_kind(L) != kSelMulti) return 0;
  const size_t mt = (size_t)L->M * (size_t)tiles_of(L->d);
  return sel_align(mt * 4) + 2 * sel_align(mt * 8) + sel_align(mt * 4) + sel_align(mt * 8) +
         sel_align((size_t)L->M * (size_t)buckets_of(L->d, L->bucket) * 4) +
         (sel_one_read(L) ? sel_align(mt * kOpenSlots * sizeof(uint2)) : 0);
}

static int check_select_layout(const qa_layout* L) {
  int rc = check_layout(L);
  if (rc != QA_OK) return rc;
  // a bucket's selected count is kept in 32 bits
  const int64_t blen = L->bucket ? L->bucket : L->d;
  if (blen >= (int64_t(1) << 32)) return QA_ERR_UNSUPPORTED;
  return QA_OK;
}

// Geometry of the general kernels and, for multi-tile buckets, the workspace pointers.
static int general_args(const qa_layout* L, SelArgs& a, void* ws, size_t ws_bytes) {
  const SelKind kind = sel_kind(L);
  a.nb = buckets_of(L->d, L->bucket);
  a.ntiles = tiles_of(L->d);
  a.seg = kind == kSelLocal ? L->bucket / 16 : kThreads;
  if (kind != kSelMulti) return QA_OK;
  const size_t need = select_workspace_bytes(L);
  if (!ws || ws_bytes < need) return QA_ERR_WORKSPACE;
  if (!aligned(ws, 256)) return QA_ERR_ALIGNMENT;
  a.tiles_per_bucket = L->bucket ? L->bucket / kTile : a.ntiles;
  a.area_words = L->bucket ? L->bucket / 16 : words_of(L->d);
  const size_t mt = (size_t)L->M * (size_t)a.ntiles;
  char* p = static_cast<char*>(ws);
  a.ws_count = reinterpret_cast<uint32_t*>(p); p += sel_align(mt * 4);
  a.ws_s1 = reinterpret_cast<double*>(p);      p += sel_align(mt * 8);
  a.ws_s2 = reinterpret_cast<double*>(p);      p += sel_align(mt * 8);
  a.ws_c2 = reinterpret_cast<uint32_t*>(p);    p += sel_align(mt * 4);
  a.ws_start = reinterpret_cast<int64_t*>(p);  p += sel_align(mt * 8);
  a.ws_thr = reinterpret_cast<float*>(p);      p += sel_align((size_t)L->M * (size_t)a.nb * 4);
  a.ws_open = sel_one_read(L) ? reinterpret_cast<uint2*>(p) : nullptr;
  return QA_OK;
}

static SelArgs base_args(const qa_layout* L) {
  SelArgs a{};
  a.d = L->d; a.W = words_of(L->d); a.NW = (L->d + 31) / 32; a.M = L->M;
  a.code_stride = L->code_stride; a.scale_stride = L->scale_stride; a.thr_coef = L->thr_coef;
  return a;
}

}  // namespace qa

extern "C" int qa_indicator(const qa_layout* layout, int method, const float* g, int64_t g_stride,
                            const float* x, const float* G, const float* z, int64_t t, float eta,
                            float lambda, float delta, uint32_t* ind_out, int64_t ind_stride,
                            void* stream) {
  using namespace qa;
  int rc = check_layout(layout);
  if (rc != QA_OK) return rc;
  if (method != 0 && method != 1) return QA_ERR_INVALID_ARG;
  if (!g || !x || !G || !ind_out || (method == 1 && !z)) return QA_ERR_INVALID_ARG;
  if (g_stride < layout->d || ind_stride < (layout->d + 31) / 32) return QA_ERR_INVALID_ARG;
  if (!(eta > 0.0f) || !(lambda >= 0.0f) || !(delta > 0.0f) || (method == 1 && t < 1))
    return QA_ERR_INVALID_ARG;
  if (!aligned(g, 4) || !aligned(x, 4) || !aligned(G, 4) || !aligned(z, 4) || !aligned(ind_out, 4))
    return QA_ERR_ALIGNMENT;
  SelArgs a = base_args(layout);
  a.method = method; a.g = g; a.g_stride = g_stride; a.x = x; a.G = G; a.z = z;
  a.ind = ind_out; a.ind_stride = ind_stride;
  a.eta = eta; a.lam_eta = lambda * eta; a.delta = delta; a.t_lam = (float)t * lambda;
  const dim3 grid((unsigned)tiles_of(layout->d)), block(kThreads);
  const bool streamed = layout->d * layout->M > kStreamedGradients;
  const auto kernel = method == 0 ? (streamed ? indicator_kernel<0, true> : indicator_kernel<0, false>)
                                  : (streamed ? indicator_kernel<1, true> : indicator_kernel<1, false>);
  hipLaunchKernelGGL(kernel, grid, block, 0, static_cast<hipStream_t>(stream), a);
  return launch_status();
}

namespace qa {
// does the fused step read this layout's sparse messages itself (one threshold/scale per tile)?
bool sparse_messages_fused(const qa_layout* L) { return sel_kind(L) == kSelTile; }
int check_sparse_layout(const qa_layout* L) { return check_select_layout(L); }

void indicator_or_launch(const qa_layout* layout, const uint32_t* ind, int64_t ind_stride,
                         uint32_t* ind_syn_out, hipStream_t stream) {
  SelArgs a = base_args(layout);
  a.ind_in = ind; a.ind_stride = ind_stride; a.ind = ind_syn_out;
  hipLaunchKernelGGL(indicator_or_kernel, dim3((unsigned)((a.NW + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, stream, a);
}
}  // namespace qa

extern "C" int qa_indicator_or(const qa_layout* layout, const uint32_t* ind, int64_t ind_stride,
                               uint32_t* ind_syn_out, void* stream) {
  using namespace qa;
  int rc = check_layout(layout);
  if (rc != QA_OK) return rc;
  if (!ind || !ind_syn_out || ind_stride < (layout->d + 31) / 32) return QA_ERR_INVALID_ARG;
  if (!aligned(ind, 4) || !aligned(ind_syn_out, 4)) return QA_ERR_ALIGNMENT;
  indicator_or_launch(layout, ind, ind_stride, ind_syn_out, static_cast<hipStream_t>(stream));
  return launch_status();
}

extern "C" int qa_quantize_pack_selected(const qa_layout* layout, const float* g, int64_t g_stride,
                                         const uint32_t* ind, int64_t ind_stride, uint32_t* sel_codes,
                                         uint32_t* counts, float* scales, float* thresholds,
                                         void* ws, size_t ws_bytes, void* stream_) {
  using namespace qa;
  int rc = check_select_layout(layout);
  if (rc != QA_OK) return rc;
  if (!g || !ind || !sel_codes || !counts || !scales) return QA_ERR_INVALID_ARG;
  if (g_stride < layout->d || (g_stride % 4) != 0 || ind_stride < (layout->d + 31) / 32)
    return QA_ERR_INVALID_ARG;
  if (!aligned(g, 16) || !aligned(ind, 4) || !aligned(sel_codes, 4) || !aligned(counts, 4) ||
      !aligned(scales, 4) || !aligned(thresholds, 4))
    return QA_ERR_ALIGNMENT;
  if (tiles_of(layout->d) > 0x7fffffffLL) return QA_ERR_INVALID_ARG;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  SelArgs a = base_args(layout);
  a.g = g; a.g_stride = g_stride; a.ind_in = ind; a.ind_stride = ind_stride;
  a.sel_codes = sel_codes; a.counts = counts; a.scales = scales; a.thresholds = thresholds;
  const dim3 block(kThreads), tiles((unsigned)tiles_of(layout->d), (unsigned)layout->M);
  const dim3 waves((unsigned)((tiles_of(layout->d) + kWaves - 1) / kWaves), (unsigned)layout->M);   // a tile per wave
  const SelKind kind = sel_kind(layout);
  if (kind == kSelTile) {
    if (tiles_of(layout->d) * layout->M <= kSelFewTiles)
      hipLaunchKernelGGL(quantize_selected_few_kernel, tiles, block, 0, stream, a);
    else
      hipLaunchKernelGGL(quantize_selected_kernel, waves, block, 0, stream, a);
    return launch_status();
  }
  rc = general_args(layout, a, ws, ws_bytes);
  if (rc != QA_OK) return rc;
  if (kind == kSelLocal) {
    hipLaunchKernelGGL(gsel_quantize_local_kernel, tiles, block, 0, stream, a);
    return launch_status();
  }
  const dim3 buckets((unsigned)a.nb, (unsigned)layout->M);
  a.samples = a.tiles_per_bucket / kSelSampleEvery;
  constexpr int kSettled = kThreads / (int)kOpenSlots;   // tiles per work-group
  const dim3 settle_grid((unsigned)((a.ntiles + kSettled - 1) / kSettled), (unsigned)layout->M);
  if (sel_one_read(layout)) {
    hipLaunchKernelGGL(gsel_count_ind_kernel, count_grid(layout), block, 0, stream, a);
    scan_launch<false>(a, layout->M, stream);
    hipLaunchKernelGGL(gsel_sample_kernel, dim3((unsigned)(a.nb * a.samples), (unsigned)layout->M), block, 0, stream, a);
    hipLaunchKernelGGL(gsel_band_kernel, buckets, block, 0, stream, a);
    hipLaunchKernelGGL(gsel_quantize_multi_kernel<true>, waves, block, 0, stream, a);
    hipLaunchKernelGGL(gsel_threshold_kernel, buckets, block, 0, stream, a);
    hipLaunchKernelGGL(gsel_settle_kernel, settle_grid, block, 0, stream, a);
    join_launch(a, layout->M, stream);
  } else {
    hipLaunchKernelGGL(gsel_count_kernel, tiles, block, 0, stream, a);
    scan_launch<true>(a, layout->M, stream);
    hipLaunchKernelGGL(gsel_quantize_multi_kernel<false>, waves, block, 0, stream, a);
    join_launch(a, layout->M, stream);
  }
  hipLaunchKernelGGL(gsel_scale_kernel, buckets, block, 0, stream, a);
  return launch_status();
}

namespace qa {
// S^{-1} for all M messages into dense code words; shared with the steps that take sparse
// messages of other bucket sizes than 4096.  `counts_scratch` (multi-tile buckets only) receives
// the per-bucket counts that the scan produces on the way; it may be the workspace's own.
int decode_selected_launch(const qa_layout* layout, const uint32_t* ind, int64_t ind_stride,
                           const uint32_t* sel_codes, uint32_t* codes_out, int64_t out_stride,
                           void* ws, size_t ws_bytes, hipStream_t stream) {
  SelArgs a = base_args(layout);
  a.ind_in = ind; a.ind_stride = ind_stride; a.sel_in = sel_codes; a.dense = codes_out;
  a.dense_stride = out_stride;
  const dim3 block(kThreads), tiles((unsigned)tiles_of(layout->d), (unsigned)layout->M);
  const SelKind kind = sel_kind(layout);
  const dim3 wave_tiles((unsigned)((tiles_of(layout->d) + kWaves * kDecodeTiles - 1) / (kWaves * kDecodeTiles)),
                        (unsigned)layout->M);
  if (kind == kSelTile) {
    hipLaunchKernelGGL(decode_selected_kernel<kSelTile>, wave_tiles, block, 0, stream, a);
    return launch_status();
  }
  int rc = general_args(layout, a, ws, ws_bytes);
  if (rc != QA_OK) return rc;
  if (kind == kSelLocal) {
    hipLaunchKernelGGL(decode_selected_kernel<kSelLocal>, wave_tiles, block, 0, stream, a);
    return launch_status();
  }
  // the scan also leaves each bucket's count; nobody asked for it here: the kept-count slots of
  // the workspace (unused by a decode) take it, M*nb <= M*ntiles words
  a.counts = a.ws_c2; a.scale_stride = a.nb;
  hipLaunchKernelGGL(gsel_count_ind_kernel, count_grid(layout), block, 0, stream, a);
  scan_launch<false>(a, layout->M, stream);
  hipLaunchKernelGGL(decode_selected_kernel<kSelMulti>, wave_tiles, block, 0, stream, a);
  return launch_status();
}
}  // namespace qa

extern "C" int qa_decode_selected(const qa_layout* layout, const uint32_t* ind, int64_t ind_stride,
                                  const uint32_t* sel_codes, uint32_t* codes_out, void* ws,
                                  size_t ws_bytes, void* stream) {
  using namespace qa;
  int rc = check_select_layout(layout);
  if (rc != QA_OK) return rc;
  if (!ind || !sel_codes || !codes_out) return QA_ERR_INVALID_ARG;
  if (ind_stride != 0 && ind_stride < (layout->d + 31) / 32) return QA_ERR_INVALID_ARG;
  if (!aligned(ind, 4) || !aligned(sel_codes, 4) || !aligned(codes_out, 4)) return QA_ERR_ALIGNMENT;
  if (tiles_of(layout->d) > 0x7fffffffLL) return QA_ERR_INVALID_ARG;
  return decode_selected_launch(layout, ind, ind_stride, sel_codes, codes_out, layout->code_stride, ws,
                                ws_bytes, static_cast<hipStream_t>(stream));
}

extern "C" int qa_select_codes(const qa_layout* layout, const uint32_t* codes, const uint32_t* ind,
                               int64_t ind_stride, uint32_t* sel_codes, uint32_t* counts, void* ws,
                               size_t ws_bytes, void* stream_) {
  using namespace qa;
  int rc = check_select_layout(layout);
  if (rc != QA_OK) return rc;
  if (!codes || !ind || !sel_codes || !counts) return QA_ERR_INVALID_ARG;
  if (ind_stride != 0 && ind_stride < (layout->d + 31) / 32) return QA_ERR_INVALID_ARG;
  if (!aligned(codes, 4) || !aligned(ind, 4) || !aligned(sel_codes, 4) || !aligned(counts, 4))
    return QA_ERR_ALIGNMENT;
  if (codes == sel_codes) return QA_ERR_INVALID_ARG;       // not in place
  if (tiles_of(layout->d) > 0x7fffffffLL) return QA_ERR_INVALID_ARG;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  SelArgs a = base_args(layout);
  a.ind_in = ind; a.ind_stride = ind_stride; a.sel_in = codes; a.sel_codes = sel_codes; a.counts = counts;
  const dim3 block(kThreads), tiles((unsigned)tiles_of(layout->d), (unsigned)layout->M);
  const SelKind kind = sel_kind(layout);
  const dim3 wave_tiles((unsigned)((tiles_of(layout->d) + kWaves - 1) / kWaves), (unsigned)layout->M);
  if (kind == kSelTile) {
    hipLaunchKernelGGL(select_codes_kernel<kSelTile>, wave_tiles, block, 0, stream, a);
    return launch_status();
  }
  rc = general_args(layout, a, ws, ws_bytes);
  if (rc != QA_OK) return rc;
  if (kind == kSelLocal) {
    hipLaunchKernelGGL(select_codes_kernel<kSelLocal>, wave_tiles, block, 0, stream, a);
    return launch_status();
  }
  hipLaunchKernelGGL(gsel_count_ind_kernel, count_grid(layout), block, 0, stream, a);
  scan_launch<false>(a, layout->M, stream);
  hipLaunchKernelGGL(select_codes_kernel<kSelMulti>, wave_tiles, block, 0, stream, a);
  join_launch(a, layout->M, stream);
  return launch_status();
}
