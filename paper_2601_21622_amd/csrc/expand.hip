// Draft-side tree expansion (Algorithm 2, ExpandLayer), batched over the
// pooled requests of a draft server: every frontier node of every request
// gets as children the top-k tokens of the draft's next-token distribution at
// that node, with their draft probabilities q (which the correction step of
// verification needs).
//
// One workgroup of 1024 threads per frontier row (request b, node f).
// Rank keys are the float32 order key of the logit, then the inverted token
// id, so that equal logits rank by increasing id and every key is unique.
//  1. Each wave scans its share of the row once, 32 steps of 64 entries loaded
//     together (a 32,000-entry row in one round).  It keeps the k best keys
//     seen so far sorted across its lanes (lane i: the i-th best): a ballot
//     against the round's bound (the k-th largest of the lanes' maxima) and the
//     list's k-th finds the few entries that may enter; each is placed by
//     counting the better keys and shifting the rest down one lane.  From the
//     same registers it keeps a running maximum m and, per lane in float64, the
//     sum of exp(logit - m), rescaled when m moves.
//  2. The waves' lists meet in LDS and wave 0 takes the k best of them one by
//     one; the waves' sums, rescaled to the row maximum, are added in wave
//     order, giving lse; q(child) = exp(logit - lse) with the difference kept
//     exact, the logit taken from its key.
// A row is one workgroup's, so a CU's inflow bounds it (128 KB take about 5
// us); a second pass for the sums took as long again: a depth-5 tree of 8 rows of
// 32,000 entries a launch or more takes 61 us against 101.
// Children of node f are numbered first_child + f*k + j in rank order.
#include <hip/hip_ext.h>

#include "common.h"
#include "launch.h"

namespace sdv {

namespace {

constexpr int kExpThreads = 1024;
constexpr int kExpWaves = kExpThreads / kWave;
constexpr int kExpUnroll = 32;  // 64-entry steps whose loads a wave issues together (a 32000-entry row: one round)

__device__ __forceinline__ uint64_t rank_key(float x, int v) {
  return ((uint64_t)order_key(x) << 32) | (uint64_t)(0xffffffffu - (uint32_t)v);
}

// Offer this lane's key to the wave's sorted list (lane i < k holds the i-th
// best key so far, 0 below; thr is the k-th best, 0 while the list is short).
// Keys are unique and never 0 for a real entry.  Every cross-lane move is a
// lane read (uniform source lane) or a one-lane DPP shift, so an insertion
// costs no LDS round trip.
// `may`: the lanes whose key may enter (the others' keys are not above thr).
__device__ __forceinline__ void offer(unsigned long long may, uint64_t key, int k, uint64_t& lst, uint64_t& thr) {
  const int lane = threadIdx.x & 63;
  unsigned long long cand = may;
  while (cand) {
    const int c = __ffsll(cand) - 1;
    cand &= cand - 1;
    const uint64_t kc = lane_u64(key, c);
    if (kc <= thr) continue;
    const int pos = __popcll(__ballot(lane < k && lst > kc));
    const uint64_t up = dpp_u64<kDppWaveShr1>(lst);
    lst = lane == pos ? kc : (lane > pos && lane < k ? up : lst);
    thr = lane_u64(lst, k - 1);
  }
}

__global__ __launch_bounds__(kExpThreads)
void expand_kernel(ExpandArgs e, const float* __restrict__ logits, int32_t* __restrict__ tokens,
                   int32_t* __restrict__ parent, float* __restrict__ q_child) {
  __shared__ uint64_t s_lst[kExpWaves][kExpandMaxK];
  __shared__ float s_m[kExpWaves];
  __shared__ double s_s[kExpWaves];
  const int row = blockIdx.x;  // b * F + f
  const int b = row / e.F;
  const int f = row - b * e.F;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const float* x = logits + (int64_t)row * e.V;

  // 1. Wave lists, running maximum and sum.
  uint64_t lst = 0, thr = 0;
  float m = -INFINITY;
  double acc = 0.0;
  for (int base = wave * kWave; base < e.V; base += kExpThreads * kExpUnroll) {
    float xs[kExpUnroll];
#pragma unroll
    for (int u = 0; u < kExpUnroll; ++u) xs[u] = x[min(base + u * kExpThreads + lane, e.V - 1)];
    float top = -INFINITY;  // this lane's largest entry of the round
#pragma unroll
    for (int u = 0; u < kExpUnroll; ++u) top = base + u * kExpThreads + lane < e.V ? fmaxf(top, xs[u]) : top;
    // The k-th largest of the lanes' largest bounds the round's k-th largest
    // from below (equal ones may fall together, which only lowers it).
    float bound = wave_max(top), rest = top;
    for (int j = 1; j < e.k; ++j) {
      rest = rest == bound ? -INFINITY : rest;
      bound = wave_max(rest);
      if (j == 1 && bound == -INFINITY) break;  // all equal or all masked: 64 x 16 rows of 5000, top-16: 81 -> 72 us
    }
#pragma unroll
    for (int u = 0; u < kExpUnroll; ++u) {
      const int v = base + u * kExpThreads + lane;
      // NaNs pass the bound: they rank by their keys like any other entry.
      const bool in = v < e.V && !(xs[u] < bound);
      const uint64_t key = in ? rank_key(xs[u], v) : 0;
      const unsigned long long may = __ballot(key > thr);
      if (may) offer(may, key, e.k, lst, thr);
    }
    float mx = fmaxf(m, top);
    mx = wave_max(mx);
    if (mx > m) acc *= exp((double)m - (double)mx);
    m = mx;
#pragma unroll
    for (int u = 0; u < kExpUnroll; ++u) {
      const bool in = base + u * kExpThreads + lane < e.V && xs[u] != -INFINITY;
      const float t = xs[u] - m;
      acc += in ? (double)(t != t ? t : exp_neg(t)) : 0.0;
    }
  }
  if (lane < kExpandMaxK) s_lst[wave][lane] = lane < e.k ? lst : 0;
  const double sw = wave_sum_f64(acc);
  if (lane == 0) {
    s_m[wave] = m;
    s_s[wave] = sw;
  }
  __syncthreads();
  if (wave != 0) return;
  float M = s_m[0];
#pragma unroll
  for (int w = 1; w < kExpWaves; ++w) M = fmaxf(M, s_m[w]);
  // Lane w rescales wave w's sum; the sums are added in wave order.
  const double mine = lane < kExpWaves ? s_s[lane] * exp((double)s_m[lane] - (double)M) : 0.0;
  double S = 0.0;
#pragma unroll
  for (int w = 0; w < kExpWaves; ++w) S += lane_f64(mine, w);
  const float lse = (float)((double)M + log(S));

  // 2. Wave 0 takes the k best of the waves' lists, largest first: four
  // candidates per lane, keys unique.
  constexpr int kCand = kExpWaves * kExpandMaxK / kWave;
  uint64_t c[kCand];
#pragma unroll
  for (int i = 0; i < kCand; ++i) {
    const int n = i * kWave + lane;
    c[i] = s_lst[n / kExpandMaxK][n % kExpandMaxK];
  }
  uint64_t best = 0;
  for (int j = 0; j < e.k; ++j) {
    uint64_t own = c[0];
#pragma unroll
    for (int i = 1; i < kCand; ++i) own = c[i] > own ? c[i] : own;
    const uint64_t w = wave_max_u64(own);
    best = lane == j ? w : best;
#pragma unroll
    for (int i = 0; i < kCand; ++i) c[i] = c[i] == w ? 0 : c[i];
  }
  if (lane < e.k) {
    const int v = (int)(0xffffffffu - (uint32_t)(best & 0xffffffffu));
    const int64_t o = (int64_t)b * e.N + e.first_child + f * e.k + lane;
    tokens[o] = v;
    parent[o] = e.frontier0 < 0 ? -1 : e.frontier0 + f;
    q_child[o] = exp_diff(key_value((uint32_t)(best >> 32)), lse);
  }
}

}  // namespace

hipError_t launch_expand(const ExpandArgs& e, const float* logits, int32_t* tokens, int32_t* parent, float* q_child,
                         hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop) {
  const int64_t rows = (int64_t)e.B * e.F;
  if (rows <= 0) return hipSuccess;
  if (rows > 0x7fffffff || e.k < 1 || e.k > kExpandMaxK || e.k > e.V) return hipErrorInvalidValue;
  hipExtLaunchKernelGGL(expand_kernel, dim3((unsigned)rows), dim3(kExpThreads), 0, stream, ev_start, ev_stop, 0, e,
                        logits, tokens, parent, q_child);
  return hipGetLastError();
}

}  // namespace sdv
