// Warped target rows for sampled verification (gfx950).
//
// Sampled decoding replaces the target p of the acceptance test (the
// Leviathan test of Sec. 2) by a warped p': logits scaled by 1/T, then the
// top-k cut (every token tied with the k-th largest logit kept), then the
// top-p cut (the smallest set {logit >= theta} of the top-k-kept tokens whose
// mass reaches top_p of their total), or, at T = 0, one-hot on the first
// largest logit (greedy).  For each row this kernel finds the cut and the
// normaliser; the acceptance kernels then evaluate
//   p'(v) = [key(v) >= theta] exp(logit(v) / T - lse)   (greedy: [v == argmax]).
//
// One workgroup of 1024 threads per row:
//   1. the largest logit (greedy: and the first index holding it), from one
//      pass, or in a step from the projection's tile maxima (greedy then reads
//      only the tiles that reach it);
//   2. a pass that keeps the few thousand largest entries in LDS and, with no
//      top-k cut, sums the row's mass; for top-k up to 64 with tile maxima only
//      tiles that reach the bound are read;
//   3. the cut among the kept entries: a wave sort for top-k up to 64, else a
//      radix descent on counts (top-k) or masses against ceil(top_p * kept
//      mass).  Rows whose cut lies elsewhere take more passes: flat or tied
//      rows a histogram of the row's mass and the entries of one of its bins,
//      and what is left (large top-k) a radix descent over the row's 32-bit
//      order keys, 11, 11 and 10 bits per level;
//   4. lse = max / T + log(kept mass).
// A pass over 128,256 entries by one workgroup is bound by its instructions (64
// lanes a cycle), so a pass does little per entry: float64 sums per thread
// instead of fixed-point ones, no vote across the wave.  224 rows of 128,256,
// top-p 0.9 in a step: 106 us with three passes of LDS atomics, 40-48 with one.
// Rows off that shape, 224 of 128,256 with the acceptance: within a nat of each
// other 126 -> 96 us, 17 distinct values 203 -> 147, all equal 702 -> 172 (the
// radix descent's atomics meet in few buckets).
// In the radix descent over a long row the second level also gathers the keys
// inside the first level's bucket into LDS; when they fit, the third level
// reads those instead of the row (the same entries, so the same integer
// sums).
// Masses are exp((logit - max) / T) in float32; where atomics add them they are
// scaled by 2^S and truncated to 64-bit integers (S = 62 - ceil(log2 V), so a
// whole row cannot overflow), which makes every histogram and total
// independent of the order of the adds; a row's whole mass is summed in
// float64 in a fixed order.  The cut is deterministic either way.
#include <hip/hip_ext.h>

#include <cmath>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace sdv {

namespace {

constexpr int kWarpThreads = 1024;
constexpr int kWarpWaves = kWarpThreads / kWave;
constexpr int kBuckets = 2048;
constexpr int kCand = 2048;  // candidates the small-k path can hold
// Keys of the entries inside the first level's bucket that a descent's
// second level gathers into LDS, so that its third level histograms them
// instead of passing over the row again (when they fit).
constexpr int kKeep = 16384;
constexpr int kKeepMinV = 65536;
// Key of the lowest float: entries down here are masked.
constexpr uint32_t kMaskedKey = 0x00800000u;
// Largest entries that each thread keeps in LDS (the same space).
constexpr int kKeepEach = 24;
static_assert(kKeepEach * kWarpThreads >= kKeep, "one array serves both");

// trunc(exp((x - m) / T) * 2^S) for x <= m, from the float32 value's bits (the
// value is about 1 at most and S at most 62, so the shifts cover every case;
// values below 2^-126 truncate to 0).
__device__ __forceinline__ unsigned long long fixed_mass(float x, float m, float inv_t, int S) {
  const uint32_t b = __float_as_uint(exp_neg((x - m) * inv_t));
  const int sh = (int)(b >> 23) - 150 + S;
  const uint32_t mant = (b & 0x7fffffu) | 0x800000u;
  const unsigned long long up = (unsigned long long)mant << max(sh, 0);
  const uint32_t down = sh > -24 ? mant >> (max(-sh, 0) & 31) : 0u;
  return (b >> 23) == 0 ? 0ull : (sh >= 0 ? up : (unsigned long long)down);
}

__device__ __forceinline__ unsigned long long shfl_xor_u64(unsigned long long v, int mask) {
  const uint32_t lo = __shfl_xor((uint32_t)v, mask);
  const uint32_t hi = __shfl_xor((uint32_t)(v >> 32), mask);
  return ((unsigned long long)hi << 32) | lo;
}

// Bitonic sort of one 64-bit key per lane across the wave, largest first.
__device__ __forceinline__ unsigned long long wave_sort_desc(unsigned long long v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int size = 2; size <= kWave; size <<= 1) {
#pragma unroll
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      const unsigned long long o = shfl_xor_u64(v, stride);
      const bool desc = (lane & size) == 0 || size == kWave;
      const bool lower = (lane & stride) == 0;
      v = (lower == desc) ? (o > v ? o : v) : (o < v ? o : v);
    }
  }
  return v;
}

// The 64 largest of two lists sorted largest first, sorted largest first: the
// lane-wise maximum of one list and the other reversed is bitonic and holds
// them; a bitonic merge orders it.
__device__ __forceinline__ unsigned long long wave_merge_desc(unsigned long long a, unsigned long long b) {
  const int lane = threadIdx.x & 63;
  const uint32_t lo = __shfl((uint32_t)b, kWave - 1 - lane);
  const uint32_t hi = __shfl((uint32_t)(b >> 32), kWave - 1 - lane);
  const unsigned long long br = ((unsigned long long)hi << 32) | lo;
  unsigned long long v = a > br ? a : br;
#pragma unroll
  for (int stride = kWave >> 1; stride > 0; stride >>= 1) {
    const unsigned long long o = shfl_xor_u64(v, stride);
    v = ((lane & stride) == 0) ? (o > v ? o : v) : (o < v ? o : v);
  }
  return v;
}

__device__ __forceinline__ unsigned long long shfl_u64(unsigned long long v, int src) {
  const uint32_t lo = __shfl((uint32_t)v, src);
  const uint32_t hi = __shfl((uint32_t)(v >> 32), src);
  return ((unsigned long long)hi << 32) | lo;
}

// Rank key of an entry: the float32 order key, then the inverted index, so
// that equal logits rank by increasing index and keys are unique (0: none).
__device__ __forceinline__ unsigned long long entry_key(uint32_t k, int v) {
  return ((unsigned long long)k << 32) | (unsigned long long)(0xffffffffu - (uint32_t)v);
}

// Calls f(v, x[v]) for every element of the row, this thread's share, with
// four 16-byte loads in flight (rows need only their entries' alignment); the
// last V % 4 entries are single loads.  Which entries a thread sees, and in
// which order, depends on V alone, so a float64 sum over them does not depend
// on where the row lies.
template <typename F>
__device__ __forceinline__ void row_pass(const float* __restrict__ x, int V, F&& f) {
  constexpr int U = 4;
  const int tid = threadIdx.x;
  const int V4 = V >> 2;
  auto quad = [&](int i, const f32x4& r) {
#pragma unroll
    for (int e = 0; e < 4; ++e) f(4 * i + e, r[e]);
  };
  int i = tid;
  for (; i + (U - 1) * kWarpThreads < V4; i += U * kWarpThreads) {
    f32x4 r[U];
#pragma unroll
    for (int u = 0; u < U; ++u) r[u] = *reinterpret_cast<const f32x4_u*>(x + 4 * (i + u * kWarpThreads));
#pragma unroll
    for (int u = 0; u < U; ++u) quad(i + u * kWarpThreads, r[u]);
  }
  for (; i < V4; i += kWarpThreads) quad(i, *reinterpret_cast<const f32x4_u*>(x + 4 * i));
  if (tid < (V & 3)) f(4 * V4 + tid, x[4 * V4 + tid]);
}

struct Level {
  int shift, nb;
  uint32_t hmask;  // bits above this level's digit
};

__device__ __forceinline__ Level level_of(int level) {
  Level l;
  l.shift = level == 0 ? 21 : (level == 1 ? 10 : 0);
  l.nb = level == 2 ? 1024 : 2048;
  l.hmask = level == 0 ? 0u : (0xffffffffu << (l.shift + (level == 2 ? 10 : 11)));
  return l;
}

// Wave 0: scanning the buckets from the top, the first bucket at which the
// running total (of counts, or of masses with BY_MASS) reaches `need`, and the
// count and mass of the buckets above it.  need >= 1 and the buckets hold at
// least `need` in total (otherwise the lowest bucket is returned).  Lane l
// totals the l-th group of nb/64 buckets from the top (reading them in a
// lane-rotated order, so the lanes hit different LDS banks); a wave scan and
// a ballot find the group, and the same inside the group finds the bucket.
template <bool BY_MASS>
__device__ void select_bucket(const uint32_t* hcnt, const unsigned long long* hmass, int nb, unsigned long long need,
                              uint32_t* s_bucket, uint32_t* s_cnt_above, unsigned long long* s_mass_above) {
  const int lane = threadIdx.x & 63;
  const int per = nb / kWave;  // 32 or 16: a power of two
  const int top = nb - 1 - lane * per;
  uint64_t c = 0, ms = 0;
  for (int i = 0; i < per; ++i) {
    const int b = top - ((i + lane) & (per - 1));
    c += hcnt[b];
    ms += hmass[b];
  }
  const uint64_t inc_c = wave_inclusive_scan_u64(c), inc_m = wave_inclusive_scan_u64(ms);
  const unsigned long long hit = __ballot((BY_MASS ? inc_m : inc_c) >= need);
  const int L = hit ? __ffsll(hit) - 1 : kWave - 1;
  const uint64_t c_above = lane_u64(inc_c, L) - lane_u64(c, L);
  const uint64_t m_above = lane_u64(inc_m, L) - lane_u64(ms, L);
  // Inside group L: lane i < per takes bucket nb - 1 - L*per - i.
  // Loads clamped rather than predicated, and every lane read taken before
  // the single-lane store: with the reads inside that branch, the compiled
  // selection returned a wrong mass above the bucket.
  const int b = max(nb - 1 - L * per - lane, 0);
  const uint64_t in_group = 0ull - (uint64_t)(lane < per);
  const uint64_t cb = (uint64_t)hcnt[b] & in_group;
  const uint64_t mb = (uint64_t)hmass[b] & in_group;
  const uint64_t ic = wave_inclusive_scan_u64(cb), im = wave_inclusive_scan_u64(mb);
  const unsigned long long hit2 = __ballot(lane < per - 1 && (BY_MASS ? m_above + im : c_above + ic) >= need);
  const int I = hit2 ? __ffsll(hit2) - 1 : per - 1;
  const uint32_t bucket = (uint32_t)(nb - 1 - L * per - I);
  const uint32_t cnt_above = (uint32_t)(c_above + lane_u64(ic, I) - lane_u64(cb, I));
  const uint64_t mass_above = m_above + lane_u64(im, I) - lane_u64(mb, I);
  if (lane == 0) {
    *s_bucket = bucket;
    *s_cnt_above = cnt_above;
    *s_mass_above = mass_above;
  }
}

// Kinds of cut, a kernel each, with tile maxima (TILES) or without: one kernel
// for all took 77 KB of instructions, more than the CU's cache holds.
enum Cut { kGreedy, kSmallK, kLargeK, kNoK };

template <int CUT, bool TILES>
__global__ __launch_bounds__(kWarpThreads)
void warp_kernel(int V, const float* __restrict__ logits, float inv_t, int top_k, float top_p, int scale,
                 const float2* __restrict__ partials, int ntiles, int tile_n, WarpRow* __restrict__ out,
                 float* __restrict__ row_lse, float* __restrict__ row_min_logit) {
  constexpr bool greedy = CUT == kGreedy;
  constexpr bool cut_k = CUT == kSmallK || CUT == kLargeK;
  __shared__ uint32_t hcnt[kBuckets];
  __shared__ unsigned long long hmass[kBuckets];
  __shared__ uint32_t w_key[kWarpWaves];
  __shared__ int w_idx[kWarpWaves];
  __shared__ uint32_t w_low[kWarpWaves];
  __shared__ unsigned long long w_sum[kWarpWaves];
  __shared__ double w_mass[kWarpWaves];
  __shared__ uint32_t s_kmax, s_bucket, s_cnt_above;
  __shared__ int s_amax;
  __shared__ unsigned long long s_mass_above;
  __shared__ unsigned long long s_list[kWarpWaves][kWave];
  __shared__ unsigned long long s_cand[kCand];
  __shared__ uint32_t s_n, s_bound, s_theta, s_pdone;
  __shared__ unsigned long long s_w;


  const int row = blockIdx.x;
  const float* x = logits + (int64_t)row * V;
  float m_row = 0.f;  // the row's largest logit, once known
  __shared__ uint32_t s_keep[kKeepEach * kWarpThreads];
  __shared__ uint32_t s_nkeep;

  // One level of a radix descent over the row: histogram (counts and masses)
  // of the entries whose key is at least `floor` and whose bits above the
  // level's digit equal `prefix`.  Level 1 also gathers those entries' keys;
  // level 2 reads the gathered keys when all of them fit.
  auto histogram = [&](int level, const Level& lv, uint32_t prefix, uint32_t floor) {
    for (int i = threadIdx.x; i < lv.nb; i += kWarpThreads) {
      hcnt[i] = 0;
      hmass[i] = 0;
    }
    if (threadIdx.x == 0 && level == 1) s_nkeep = 0;
    __syncthreads();
    const float* xr = logits + (int64_t)blockIdx.x * V;
    auto add = [&](uint32_t k, float xv) {  // xv = key_value(k)
      const int b = (k >> lv.shift) & (lv.nb - 1);
      atomicAdd(&hcnt[b], 1u);
      atomicAdd(&hmass[b], fixed_mass(xv, m_row, inv_t, scale));
    };
    // Rows short enough to stay in L2 are read again instead: the gathered
    // level measured slower at 32,000 entries, faster at 128,256.
    const bool use_keep = V >= kKeepMinV;
    const bool gather = use_keep && level == 1;
    if (use_keep && level == 2 && s_nkeep <= (uint32_t)kKeep) {
      const int n = (int)s_nkeep;
      for (int i = threadIdx.x; i < n; i += kWarpThreads) {
        const uint32_t k = s_keep[i];
        if (k >= floor && (k & lv.hmask) == prefix) add(k, key_value(k));
      }
    } else {
      row_pass(xr, V, [&](int, float xv) {
        const uint32_t k = order_key(xv);
        if (k >= floor && (k & lv.hmask) == prefix) {
          add(k, xv);
          if (gather) {
            const uint32_t i = atomicAdd(&s_nkeep, 1u);
            if (i < (uint32_t)kKeep) s_keep[i] = k;
          }
        }
      });
    }
    __syncthreads();
  };
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;

  // 1. Largest key; among equal keys the smallest index.
  auto merge = [](uint32_t& k, int& i, uint32_t ok, int oi) {
    if (ok > k || (ok == k && oi < i)) {
      k = ok;
      i = oi;
    }
  };
  // With the projection's tile statistics, from the tile maxima: only greedy
  // needs the entry itself, and then reads the tiles that reach the maximum.
  const float2* tiles = partials + (TILES ? (int64_t)row * ntiles : 0);
  // f(v, x[v]) for every entry of the tiles whose maximum reaches `bound`
  // (tiles w, w + 16, ... on wave w).
  auto tile_pass = [&](float bound, auto&& f) {
    for (int base = 0; base < ntiles; base += kWarpThreads) {
      const int t = base + lane * kWarpWaves + wave;
      const float tm = tiles[min(t, ntiles - 1)].x;
      unsigned long long todo = __ballot(t < ntiles && tm >= bound);
      while (todo) {
        const int v0 = (base + (__ffsll(todo) - 1) * kWarpWaves + wave) * tile_n;
        todo &= todo - 1;
        const int v1 = min(V, v0 + tile_n);
        for (int vb = v0; vb < v1; vb += 8 * kWave) {
          float r[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) r[e] = x[min(vb + e * kWave + lane, v1 - 1)];
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (vb + e * kWave + lane < v1) f(vb + e * kWave + lane, r[e]);
        }
      }
    }
  };
  bool by_tiles = TILES && (CUT != kSmallK || top_k <= ntiles);
  uint32_t bk = 0;
  int bi = 0x7fffffff;
  bool odd = false;  // a tile's sum is no number: NaN or infinite logits, whose order the row itself gives
  if (by_tiles) {
    for (int t = tid; t < ntiles; t += kWarpThreads) {
      const float2 st = tiles[t];
      merge(bk, bi, order_key(st.x), t);
      odd |= st.y != st.y;
    }
    if (__syncthreads_or(odd)) {
      by_tiles = false;
      bk = 0;
      bi = 0x7fffffff;
    }
  }
  if (!by_tiles) row_pass(x, V, [&](int v, float xv) { merge(bk, bi, order_key(xv), v); });
  // This thread's best entry (or tile): a lower bound of one entry of the row.
  const unsigned long long tkey = bi == 0x7fffffff ? 0ull : entry_key(bk, bi);
  for (int off = 32; off >= 1; off >>= 1) merge(bk, bi, __shfl_xor(bk, off), __shfl_xor(bi, off));
  if (greedy && by_tiles) {
    __shared__ float s_top;
    if (lane == 0) w_key[wave] = bk;
    __syncthreads();
    if (tid == 0) {
      uint32_t k = w_key[0];
      for (int w = 1; w < kWarpWaves; ++w) k = max(k, w_key[w]);
      s_top = key_value(k);
    }
    __syncthreads();
    const float top = s_top;
    bk = 0;
    bi = 0x7fffffff;
    tile_pass(top, [&](int v, float xv) { merge(bk, bi, order_key(xv), v); });
    for (int off = 32; off >= 1; off >>= 1) merge(bk, bi, __shfl_xor(bk, off), __shfl_xor(bi, off));
    __syncthreads();
  }
  if (lane == 0) {
    w_key[wave] = bk;
    w_idx[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
    uint32_t k = w_key[0];
    int i = w_idx[0];
    for (int w = 1; w < kWarpWaves; ++w) merge(k, i, w_key[w], w_idx[w]);
    s_kmax = k;
    s_amax = i;
  }
  __syncthreads();
  const int amax = s_amax;
  if (greedy) {
    if (tid == 0) {
      out[row] = WarpRow{0.f, 0xffffffffu, 0.f, amax};
      row_lse[row] = 0.f;
      row_min_logit[row] = INFINITY;
    }
    return;
  }
  const float m = key_value(s_kmax);
  m_row = m;

  // Mass of the whole row (no top-k), or of the top-k set.
  uint32_t theta = 0;
  unsigned long long W = 0;
  bool have_k = false, have_p = false;
  bool few = false;  // fewer unmasked entries than a small top_k
  if (CUT == kSmallK) {
    // Small k: the k-th largest of the threads' best entries bounds the k-th
    // largest logit from below (k threads reach it), so the entries at or
    // above it hold the top-k set and all its ties.  They are collected in
    // LDS and wave 0 sorts them in 64-key batches.
    s_list[wave][lane] = wave_sort_desc(tkey);
    __syncthreads();
    if (wave == 0) {
      unsigned long long acc = s_list[0][lane];
      for (int w = 1; w < kWarpWaves; ++w) acc = wave_merge_desc(acc, s_list[w][lane]);
      const unsigned long long kth = shfl_u64(acc, top_k - 1);
      if (lane == 0) {
        s_bound = (uint32_t)(kth >> 32);
        s_n = 0;
      }
    }
    __syncthreads();
    // As values (-0 equal to +0: a tile maximum may be either); a superset,
    // with every NaN (they rank by their keys).  With fewer threads that hold
    // an unmasked entry than top_k (short rows, or nearly all masked): every
    // unmasked entry.
    const float bound = s_bound <= kMaskedKey ? key_value(kMaskedKey + 1) : key_value(s_bound);
    auto take = [&](int v, float xv) {
      if (!(xv < bound)) {
        const uint32_t i = atomicAdd(&s_n, 1u);
        if (i < (uint32_t)kCand) s_cand[i] = entry_key(order_key(xv), v);
      }
    };
    // A wave's tiles come one after another: only on rows of several rounds of
    // loads (20 rows of 5003, 16-wide tiles: 38 us a step by tiles, 36 without).
    if (by_tiles && V > kWarpThreads * 16) tile_pass(bound, take);
    else row_pass(x, V, take);
    __syncthreads();
    const uint32_t n = s_n;
    few = n < (uint32_t)top_k;
    // Otherwise (masses of ties at the bound, or masked entries in the set) the
    // radix descent below.
    if (!few && n <= (uint32_t)kCand) {
      if (wave == 0) {
        unsigned long long lst = 0;
        for (uint32_t base = 0; base < n; base += kWave)
          lst = wave_merge_desc(lst, wave_sort_desc(base + lane < n ? s_cand[base + lane] : 0ull));
        const uint32_t thk = (uint32_t)(shfl_u64(lst, top_k - 1) >> 32);
        // The kept set: every candidate whose key reaches the k-th (ties kept).
        uint32_t cnt = 0;
        unsigned long long ms = 0;
        for (uint32_t i = lane; i < n; i += kWave) {
          const uint32_t k = (uint32_t)(s_cand[i] >> 32);
          if (k >= thk) {
            ++cnt;
            ms += fixed_mass(key_value(k), m, inv_t, scale);
          }
        }
        for (int off = 32; off >= 1; off >>= 1) {
          cnt += __shfl_xor(cnt, off);
          ms += shfl_xor_u64(ms, off);
        }
        // Equal on every lane; as scalars, the branch below is uniform.
        cnt = (uint32_t)__builtin_amdgcn_readfirstlane((int)cnt);
        ms = lane_u64(ms, 0);
        uint32_t th = thk;
        unsigned long long w = ms;
        bool pdone = false;
        if (top_p < 1.f && cnt <= (uint32_t)kWave) {
          // Lanes [0, cnt) of the sorted list are the kept set, largest first:
          // the cut is the first key whose running mass reaches the target.
          unsigned long long target = (unsigned long long)ceil((double)top_p * (double)ms);
          target = target < 1 ? 1 : (target > ms ? ms : target);
          const uint32_t lk = (uint32_t)(lst >> 32);
          const unsigned long long cum =
              wave_inclusive_scan_u64(lane < (int)cnt ? fixed_mass(key_value(lk), m, inv_t, scale) : 0ull);
          const int i = __ffsll(__ballot(lane < (int)cnt && cum >= target)) - 1;
          th = __shfl(lk, i);
          const int c = __popcll(__ballot(lane < (int)cnt && lk >= th));
          w = shfl_u64(cum, c - 1);
          pdone = true;
        }
        if (lane == 0) {
          s_theta = th;
          s_w = w;
          s_pdone = pdone;
        }
      }
      __syncthreads();
      theta = s_theta;
      W = s_w;
      have_k = true;
      have_p = s_pdone != 0;
    }
  }
  // Other cuts: the largest entries (value at least `bound`, a few thousand)
  // are kept in LDS, each thread its own, and the cut is found among them when
  // they hold it: top_k of them, or top_p of the row's mass (summed in the same
  // pass, per thread in float64).  The bound is the smallest tile maximum where
  // that leaves top_k entries, else 0.15 of the tile maxima's spread below it
  // (3 to 10 % of a normal row), or without tiles a tenth of the spread above the
  // smallest of the threads' maxima (3 % of a 128,256-entry normal row, half of
  // a 1000-entry one); a bound that keeps too many or too few only costs time,
  // the cut is then found from the whole row.  Not tried where it would only
  // cost that time: with more top_k than maxima that it goes by (eight per
  // tile: those of normal rows lie that dense; 40 rows of 32,000, top-k 5000:
  // 50 us tried, 44 not) unless all unmasked entries of a short row fit, and for
  // top_p in rows whose entries lie within a nat, where the largest few hold
  // too little (0.05 normal, top-p 0.95: 50 us, 37).
  bool among = false;  // the cut is among the kept entries
  int mine = 0;        // this thread's, at s_keep[i * kWarpThreads + tid]
  uint32_t kbase = 0;  // a key no kept entry is below
  uint32_t kmax = m == 0.f ? order_key(0.f) : s_kmax;  // and one none is above
  double mass = 0.0;   // of the row, this thread's share
  const bool whole = !have_k && !cut_k;
  float lowest = m;    // the smallest of the threads' (or tiles') unmasked maxima
  const bool few_k = top_k <= (by_tiles ? 8 * ntiles : min(V / 4, kWarpThreads));
  const bool near_k = cut_k && !few && (few_k || V <= 4 * kWarpThreads);
  if (!have_k && (cut_k ? near_k : top_p < 1.f)) {
    // Without the thread that holds a partial last tile.
    const bool part = by_tiles && ntiles > 1 && V % tile_n != 0 && tid == (ntiles - 1) % kWarpThreads;
    const uint32_t own = (uint32_t)(tkey >> 32);
    uint32_t low = own <= kMaskedKey || part ? 0xffffffffu : own;
    for (int off = 32; off >= 1; off >>= 1) low = min(low, (uint32_t)__shfl_xor((int)low, off));
    if (lane == 0) w_low[wave] = low;
    __syncthreads();
    for (int w = 0; w < kWarpWaves; ++w) low = min(low, w_low[w]);
    if (low != 0xffffffffu) lowest = key_value(low);
  }
  const float spread = (m - lowest) * inv_t;
  const bool flat = whole && top_p < 1.f && spread < 1.f && V > 4 * kWarpThreads;
  const bool gather = !have_k && (near_k || (whole && top_p < 1.f && !flat));
  if (gather) {
    const float bound = cut_k && !few_k ? key_value(kMaskedKey + 1)
                        : !by_tiles     ? lowest + 0.1f * (m - lowest)
                                        : (cut_k && top_k <= ntiles ? lowest : lowest - 0.15f * (m - lowest));
    kbase = order_key(bound == 0.f ? -0.f : bound);  // -0 passes as +0 does
    for (int i = tid; i < kBuckets; i += kWarpThreads) hmass[i] = 0;
    auto take = [&](int, float xv) {
      if (xv >= bound) {
        if (mine < kKeepEach) s_keep[mine * kWarpThreads + tid] = __float_as_uint(xv);
        ++mine;
      }
    };
    if (!cut_k)
      row_pass(x, V, [&](int v, float xv) {
        mass += (double)exp_neg((xv - m) * inv_t);
        take(v, xv);
      });
    else
      row_pass(x, V, take);  // nearly every tile reaches the bound
    // Kept values to keys; their count, or their mass.
    unsigned long long near = cut_k ? (unsigned long long)mine : 0ull;
    for (int i = 0; i < min(mine, kKeepEach); ++i) {
      const float xv = __uint_as_float(s_keep[i * kWarpThreads + tid]);
      s_keep[i * kWarpThreads + tid] = order_key(xv);
      if (!cut_k) near += fixed_mass(xv, m, inv_t, scale);
    }
    const bool over = __ballot(mine > kKeepEach) != 0;
    for (int off = 32; off >= 1; off >>= 1) near += shfl_xor_u64(near, off);
    if (lane == 0) {
      w_sum[wave] = near;
      w_key[wave] = over;
    }
  } else if (whole && !flat) {
    row_pass(x, V, [&](int, float xv) { mass += (double)exp_neg((xv - m) * inv_t); });
  }
  if (whole) {
    mass = wave_sum_f64(mass);
    if (lane == 0) w_mass[wave] = mass;
  }
  __syncthreads();
  if (whole) {
    double all = 0.0;
    for (int w = 0; w < kWarpWaves; ++w) all += w_mass[w];
    W = (unsigned long long)ldexp(all, scale);
  }
  if (gather) {
    unsigned long long near = 0;
    uint32_t over = 0;
    for (int w = 0; w < kWarpWaves; ++w) {
      near += w_sum[w];
      over |= w_key[w];
    }
    const unsigned long long target =
        cut_k ? (unsigned long long)top_k : max((unsigned long long)ceil((double)top_p * (double)W), 1ull);
    among = over == 0 && near >= target;
    __syncthreads();
  }
  // Radix descent over the kept entries, on their distance from kbase, in
  // digits of eight bits from the highest bit in use (whole keys share their
  // top bits: few buckets, and atomics that collide): the first key from the
  // top at which the running count (or mass) of the entries at or above
  // `floor` reaches `need`.  A level takes the next of hmass's eight cleared
  // histograms of 256 and one barrier; every wave selects its bucket for
  // itself.  *upto: the count (or mass) down to that key.
  auto near_cut = [&](auto by_mass, int hist0, unsigned long long need, uint32_t floor, unsigned long long* upto) {
    constexpr int kBits = 8, kBins = 1 << kBits;
    int shift = 32 - __clz((int)((kmax - kbase) | 1u));
    uint32_t prefix = 0;
    unsigned long long above = 0;
    for (int level = hist0; shift > 0; ++level) {
      const int top_shift = shift;
      const int width = min(shift, kBits);
      shift -= width;
      unsigned long long* h = hmass + level * kBins;
      for (int i = 0; i < mine; ++i) {
        const uint32_t k = s_keep[i * kWarpThreads + tid];
        const uint32_t d = k - kbase;
        if (k >= floor && (top_shift >= 32 || (d >> top_shift) == prefix))
          atomicAdd(&h[(d >> shift) & ((1u << width) - 1)],
                    decltype(by_mass)::value ? fixed_mass(key_value(k), m, inv_t, scale) : 1ull);
      }
      __syncthreads();
      // Lane l: buckets 255 - 4l .. 252 - 4l, from the top.
      uint64_t c[4], own = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        c[i] = h[kBins - 1 - 4 * lane - i];
        own += c[i];
      }
      const uint64_t inc = wave_inclusive_scan_u64(own);
      const unsigned long long hit = __ballot(above + inc >= need);
      const int at = hit ? __ffsll(hit) - 1 : kWave - 1;
      uint64_t run = above + inc - own;  // of the buckets above this lane's
      int b = kBins - 1 - 4 * lane;
#pragma unroll
      for (int i = 0; i < 3; ++i) {
        const bool on = run + c[i] < need && b == kBins - 1 - 4 * lane - i;
        run += on ? c[i] : 0ull;
        b -= on ? 1 : 0;
      }
      above = lane_u64(run, at);
      b = __builtin_amdgcn_readlane(b, at);
      prefix = (prefix << width) | (uint32_t)b;
      *upto = above + h[b];
    }
    return kbase + prefix;
  };
  if (have_k) {
  } else if (cut_k && among) {
    unsigned long long kept;
    theta = near_cut(std::false_type{}, 0, (unsigned long long)top_k, 0u, &kept);
    unsigned long long sum = 0;
    for (int i = 0; i < mine; ++i) {
      const uint32_t k = s_keep[i * kWarpThreads + tid];
      if (k >= theta) sum += fixed_mass(key_value(k), m, inv_t, scale);
    }
    for (int off = 32; off >= 1; off >>= 1) sum += shfl_xor_u64(sum, off);
    if (lane == 0) w_sum[wave] = sum;
    __syncthreads();
    for (int w = 0; w < kWarpWaves; ++w) W += w_sum[w];
  } else if (cut_k) {
    uint32_t prefix = 0, krem = (uint32_t)top_k;
    unsigned long long above = 0;
    for (int level = 0; level < 3; ++level) {
      const Level lv = level_of(level);
      histogram(level, lv, prefix, 0u);
      if (wave == 0) select_bucket<false>(hcnt, hmass, lv.nb, krem, &s_bucket, &s_cnt_above, &s_mass_above);
      __syncthreads();
      const uint32_t b = s_bucket;
      krem -= s_cnt_above;
      above += s_mass_above;
      prefix |= b << lv.shift;
      if (level == 2) W = above + hmass[b];
      __syncthreads();
    }
    theta = prefix;
  }

  if (top_p < 1.f && !have_p) {
    unsigned long long target = 0;
    auto set_target = [&]() {
      target = (unsigned long long)ceil((double)top_p * (double)W);
      target = target < 1 ? 1 : (target > W ? W : target);
    };
    set_target();
    uint32_t prefix = 0;
    unsigned long long above = 0;
    bool tied = false;
    if (!among && whole) {
      // The cut lies below the kept entries (a flat row), or too many were
      // kept: one pass histograms the row's mass over 2048 bins from the
      // maximum, another keeps the entries of the bin where the running mass
      // reaches the target.  Bins of 1/64 nat; in rows whose maxima lie within
      // two nats, where atomics would meet in few of those and one hold too many
      // entries, 1024 over eight times the maxima's spread and then of 1/32.
      const bool fine = spread > 0.f && spread < 2.f;
      const float per = fine ? fminf(128.f / spread, 1e30f) : 64.f;
      const float far = fine ? 32.f : 0.f, far0 = fine ? 1024.f - 256.f * spread : kBuckets - 1.f;
      auto bin_of = [&](float xv) {
        const float d = (m - xv) * inv_t;
        return (int)fminf(fminf(d * per, fmaf(d, far, far0)), kBuckets - 1.f);
      };
      for (int i = tid; i < kBuckets; i += kWarpThreads) {
        hmass[i] = 0;
        hcnt[i] = 0;
      }
      __syncthreads();
      row_pass(x, V, [&](int, float xv) {
        const unsigned long long w = fixed_mass(xv, m, inv_t, scale);
        if (w != 0) atomicAdd(&hmass[kBuckets - 1 - bin_of(xv)], w);  // far entries would meet in one bin
      });
      __syncthreads();
      if (flat) {  // no pass has summed the row yet
        unsigned long long all = 0;
        for (int i = lane; i < kBuckets; i += kWave) all += hmass[i];
        for (int off = 32; off >= 1; off >>= 1) all += shfl_xor_u64(all, off);
        W = all;
        set_target();
      }
      if (wave == 0) select_bucket<true>(hcnt, hmass, kBuckets, target, &s_bucket, &s_cnt_above, &s_mass_above);
      __syncthreads();
      const int bin = kBuckets - 1 - (int)s_bucket;
      const unsigned long long bin_above = s_mass_above, bin_mass = hmass[s_bucket];
      __syncthreads();
      for (int i = tid; i < kBuckets; i += kWarpThreads) hmass[i] = 0;
      mine = 0;
      uint32_t lo = 0xffffffffu, hi = 0;
      row_pass(x, V, [&](int, float xv) {
        if (bin_of(xv) == bin) {
          const uint32_t k = order_key(xv);
          lo = min(lo, k);
          hi = max(hi, k);
          if (mine < kKeepEach) s_keep[mine * kWarpThreads + tid] = k;
          ++mine;
        }
      });
      const bool over = __ballot(mine > kKeepEach) != 0;
      for (int off = 32; off >= 1; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
      }
      if (lane == 0) {
        w_key[wave] = hi;
        w_low[wave] = lo;
        w_idx[wave] = over;
      }
      __syncthreads();
      kbase = 0xffffffffu;
      kmax = 0;
      int full = 0;
      for (int w = 0; w < kWarpWaves; ++w) {
        kbase = min(kbase, w_low[w]);
        kmax = max(kmax, w_key[w]);
        full |= w_idx[w];
      }
      // Masses summed in 64-bit integers here and in float64 in W may put the
      // target a rounding past the last bin: the radix descent handles that too.
      if (kbase == kmax && target > bin_above && target <= bin_above + bin_mass) {
        tied = true;  // every entry of the bin: the cut is their key
        prefix = kbase;
        W = bin_above + bin_mass;
      } else if (full == 0 && kbase <= kmax && target > bin_above) {
        among = true;
        above = bin_above;
      }
      __syncthreads();
    }
    if (among) {
      prefix = near_cut(std::true_type{}, kBuckets / 512, target - above, theta, &W);
      W += above;
      above = 0;
    }
    for (int level = 0; level < 3 && !among && !tied; ++level) {
      const Level lv = level_of(level);
      histogram(level, lv, prefix, theta);
      if (wave == 0)
        select_bucket<true>(hcnt, hmass, lv.nb, target - above, &s_bucket, &s_cnt_above, &s_mass_above);
      __syncthreads();
      const uint32_t b = s_bucket;
      above += s_mass_above;
      prefix |= b << lv.shift;
      if (level == 2) W = above + hmass[b];
      __syncthreads();
    }
    theta = prefix;
  }

  if (tid == 0) {
    const float lse = (float)((double)m * (double)inv_t + log(ldexp((double)W, -scale)));
    out[row] = WarpRow{inv_t, theta, lse, -1};
    row_lse[row] = lse;
    row_min_logit[row] = theta == 0 ? -INFINITY : key_value(theta);
  }
}

}  // namespace

hipError_t launch_warp(int M, int V, const float* logits, float temperature, int top_k, float top_p, WarpRow* out,
                       float* row_lse, float* row_min_logit, hipStream_t stream, hipEvent_t ev_start, const float2* partials,
                       int ntiles, int tile_n) {
  if (M <= 0) return hipSuccess;
  const bool greedy = temperature == 0.f;
  const float inv_t = greedy ? 0.f : 1.f / temperature;  // float32 division, correctly rounded
  int bits = 0;
  while ((int64_t(1) << bits) < V) ++bits;
  const int scale = 62 - bits;
  const bool cut_k = top_k >= 1 && top_k < V;
  const Cut cut = greedy ? kGreedy : (!cut_k ? kNoK : (top_k <= kWave ? kSmallK : kLargeK));
  const bool tiles = partials != nullptr;
  const auto kern = cut == kGreedy   ? (tiles ? warp_kernel<kGreedy, true> : warp_kernel<kGreedy, false>)
                    : cut == kSmallK ? (tiles ? warp_kernel<kSmallK, true> : warp_kernel<kSmallK, false>)
                    : cut == kLargeK ? (tiles ? warp_kernel<kLargeK, true> : warp_kernel<kLargeK, false>)
                                     : (tiles ? warp_kernel<kNoK, true> : warp_kernel<kNoK, false>);
  hipExtLaunchKernelGGL(kern, dim3(M), dim3(kWarpThreads), 0, stream, ev_start, nullptr, 0, V, logits, inv_t, top_k,
                        top_p, scale, partials, ntiles, tile_n, out, row_lse, row_min_logit);
  return hipGetLastError();
}

}  // namespace sdv
