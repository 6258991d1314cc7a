// Vocabulary projection, line schedule (gfx950): float32, and bfloat16 with
// at most 64 hidden rows.
//
// One 128-byte line of every row per pipeline step.  A wave owns 16 vocabulary
// rows and DMAs each step's 16 lines of W straight into LDS; the workgroup's
// hidden lines (MB blocks of 16 rows) are shared and DMA'd once.  Every DMA
// instruction moves eight whole lines, where loads in MFMA operand order would
// touch 16 rows x 64 bytes (row-major W at 52 x 1536 x 50021: 56 us with
// those, 40 us with whole lines; 24 x 3712 x 4025, whose K only fitted 32-wide
// chunks before: 85 -> 22 us).  Packed W comes in fragments of 1 KB, two per
// step.  In LDS a 1 KB block holds 8 rows, 16-byte unit u of row r at slot 8r +
// (u + (r & ~1)) mod 8: a fragment read (ds_read_b128) is served 16 lanes at a
// time, lanes {0-3, 12-15, 20-27} of each half wave first and the others next,
// and with this rotation each such group covers all 64 banks once (the
// conflict counter reads 0; with rotation by r + (block & 1) it read 3.4
// cycles per instruction).  Steps run through S stages, S - 1 issued ahead,
// one LDS-only barrier per step (the hidden lines are shared).  Two workgroups
// share a CU where their stages fit: one's start and epilogue run under the
// other's stream (52 x 1536 x 50021: 45.6 us with one, 39.7 with two).
// bfloat16 reads a line's fragments a step ahead, since with one workgroup per
// CU or none a step is a chain of barrier, reads and products (with the lse
// launch, packed: 64 x 4096 x 4000 41.6 -> 29.6 us, 20 x 1024 x 5003 12.9 ->
// 11.3, large vocabularies alike); float32, bound by its products, reads them in
// the step itself (40 x 1024 x 32000: 43.6 us, 54.3 a step ahead).
//
// Bound by HBM (W is read once) at bfloat16: 48 x 4096 x 32000 packed takes 44
// us, 6.1 TB/s.  float32 at 40 x 1024 x 32000 takes 40 us where scalar FMAs on
// LDS tiles took 290: the W stream alone takes 29 us and the float32 matrix
// products 20 (157 TFLOP/s peak), and the two overlap in part.
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "vocab_tile.h"

namespace sdv {

namespace {


// Pipeline stages, at most eight: as many as fit half the CU's 160 KB (the
// epilogue's few bytes aside) if that is three or more, so that two workgroups
// share the CU, else as fit all of it.
constexpr int line_stages(int stage_bytes) {
  const int h = (78 * 1024) / stage_bytes;
  const int n = h >= 3 ? h : (156 * 1024) / stage_bytes;
  return n < 8 ? n : 8;
}

// 16-byte unit of a row's line that lane l of a block's DMA brings.
__device__ __forceinline__ int line_unit(int l) { return ((l & 7) - ((l >> 3) & ~1)) & 7; }
// LDS byte of unit 4*half + lane/16 of row lane%16 of a 16-row (2 KB) block pair.
__device__ __forceinline__ int line_read(int lane, int half) {
  const int q = (lane >> 3) & 1, r = lane & 7;
  return q * 1024 + r * 128 + ((4 * half + (lane >> 4) + (r & ~1)) & 7) * 16;
}

// acc[mb][half] += W hidden^T over one line: w and h hold bytes 16*(lane/16)
// .. +15 of each half of the lane's row.  float32: four 16x16x4 products per
// half, product j taking element j of every lane (the same k order on both
// sides); consecutive products go to different accumulators.
template <int MB>
__device__ __forceinline__ void line_mma(const float*, const u32x4 (&w)[2], const u32x4 (&h)[MB][2],
                                         f32x4 (&acc)[MB][2], int) {
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        acc[mb][half] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w[half][j]), __uint_as_float(h[mb][half][j]),
                                                             acc[mb][half], 0, 0, 0);
}

// bfloat16: one 16x16x32 product per half, in one chain in k order; `halves` 1
// leaves out the second (the last line of a row whose length is an odd number
// of half lines).
template <int MB>
__device__ __forceinline__ void line_mma(const uint16_t*, const u32x4 (&w)[2], const u32x4 (&h)[MB][2],
                                         f32x4 (&acc)[MB][2], int halves) {
#pragma unroll
  for (int half = 0; half < 2; ++half)
    if (half < halves) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        acc[mb][0] = mfma16x16x32(__builtin_bit_cast(bf16x8, w[half]), __builtin_bit_cast(bf16x8, h[mb][half]),
                                  acc[mb][0]);
    }
}

template <typename T, int MB, int NW, bool PACKED>
__device__ __forceinline__ void vocab_lines(int M, int K, int V, int ntiles, int mtiles, const T* __restrict__ hidden,
                                            const T* __restrict__ w, float* __restrict__ logits,
                                            float2* __restrict__ partials) {
  constexpr int kHBlocks = 2 * MB;               // 1 KB blocks of hidden lines per line
  constexpr int kHd = (kHBlocks + NW - 1) / NW;  // of which wave w brings w, w + NW, ...
  constexpr int kStage = (kHBlocks + 2 * NW) * 1024;
  constexpr int S = line_stages(kStage);
  static_assert(S >= 3 && (S - 1) * (2 + kHd) < 64, "vmcnt holds 6 bits");
  __shared__ __align__(1024) unsigned char lds[S * kStage];
  __shared__ float red[NW][16 * MB];

  // The M-tiles of one vocabulary tile share an XCD (ids 8 apart), where the
  // later readers of a W line find it in L2.
  const int grp = 8 * mtiles;
  const int tile = mtiles == 1 ? (int)blockIdx.x : (int)(blockIdx.x / grp) * 8 + (int)(blockIdx.x & 7);
  if (tile >= ntiles) return;
  const int m0 = mtiles == 1 ? 0 : (int)((blockIdx.x % grp) >> 3) * MB * 16;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  constexpr int kHalf = kLineBytes / 2 / (int)sizeof(T);  // elements per half line
  const int nlines = (K + 2 * kHalf - 1) / (2 * kHalf);
  const int tail = K % (2 * kHalf) == 0 ? 2 : 1;  // halves of the last line

  // Rows past V and past M repeat the last row: lines already requested, and
  // results the epilogue does not store.
  const int unit = line_unit(lane);
  // Bytes from a row's line to the last line's unit where that line is a half
  // one: the missing half repeats the first.
  const int tail_shift = tail == 1 ? (unit & 3) * 16 - unit * 16 : 0;
  const int nblk = (V + 15) / 16;
  const char* wsrc[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    if (PACKED) {
      // Fragment (32-wide k-step 2c + q, block): 1 KB in the operand's lane order.
      const int blk = min(tile * NW + wave, nblk - 1);
      wsrc[q] = reinterpret_cast<const char*>(w) + ((int64_t)q * nblk + blk) * 1024 + lane * 16;
    } else {
      const int row = min((tile * NW + wave) * 16 + 8 * q + (lane >> 3), V - 1);
      wsrc[q] = reinterpret_cast<const char*>(w + (int64_t)row * K) + unit * 16;
    }
  }
  const int64_t wline = PACKED ? (int64_t)nblk * 2048 : kLineBytes;
  const char* hsrc[kHd];
#pragma unroll
  for (int i = 0; i < kHd; ++i) {
    const int n = min(wave + NW * i, kHBlocks - 1);
    const int row = min(m0 + 8 * n + (lane >> 3), M - 1);
    hsrc[i] = reinterpret_cast<const char*>(hidden + (int64_t)row * K) + unit * 16;
  }
  // Hidden blocks this wave brings per step: kHd, or one fewer on the last waves.
  const int nh = (kHBlocks - wave + NW - 1) / NW;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  // Rows a multiple of 4 KB apart put one line of every row on few memory
  // channels, and the workgroups move through the lines together: groups of
  // eight tiles then start three lines apart and wrap around (row-major, 16 x
  // 2048 x 60000: 51 -> 41 us; 24 x 8192 x 32000: 107 -> 83; packed weights, which
  // take the same order so that both layouts round alike: within 2 %).  Not with
  // several M-tiles, whose readers of a W line would drift apart.
  const int first = mtiles == 1 && K * (int)sizeof(T) % 4096 == 0 ? (tile >> 3) * 3 % nlines : 0;
  auto issue = [&](int s, int step) {
    const uint32_t dst = lds_base + (uint32_t)s * kStage;
    const int c = step + first < nlines ? step + first : step + first - nlines;
    const bool last = c == nlines - 1;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const char* p = wsrc[q] + (int64_t)c * wline;
      if (PACKED) p -= last && tail == 1 && q == 1 ? (int64_t)nblk * 1024 : 0;  // no such k-step: the one before
      else p += last ? tail_shift : 0;
      line_dma<true>(p, dst + (kHBlocks + 2 * wave + q) * 1024);
    }
#pragma unroll
    for (int i = 0; i < kHd; ++i)
      if (i < nh)
        line_dma<false>(hsrc[i] + (int64_t)c * kLineBytes + (last ? tail_shift : 0), dst + (wave + NW * i) * 1024);
  };

  // float32: two accumulators per block (the halves of a line), added at the
  // end: two shorter chains round less than one.
  f32x4 acc[MB][2];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) acc[mb][0] = acc[mb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int rd0 = line_read(lane, 0), rd1 = line_read(lane, 1);

  struct Frags {
    u32x4 w[2], h[MB][2];
  };
  auto read = [&](int s, Frags& f) {
    const unsigned char* src = lds + s * kStage;
    const unsigned char* wsl = src + (kHBlocks + 2 * wave) * 1024;
    f.w[0] = *reinterpret_cast<const u32x4*>(wsl + (PACKED ? lane * 16 : rd0));
    f.w[1] = *reinterpret_cast<const u32x4*>(wsl + (PACKED ? 1024 + lane * 16 : rd1));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      f.h[mb][0] = *reinterpret_cast<const u32x4*>(src + mb * 2048 + rd0);
      f.h[mb][1] = *reinterpret_cast<const u32x4*>(src + mb * 2048 + rd1);
    }
  };
  // Until all but the newest N steps' lines have landed; `all` of them
  // where fewer are in flight (the last steps of a row).
  auto wait = [&](auto steps, bool all) {
    constexpr int N = decltype(steps)::value;
    if (!all) {
      if (nh == kHd)
        wait_vmcnt<N * (2 + kHd)>();
      else
        wait_vmcnt<N * (1 + kHd)>();
    } else {
      wait_vmcnt<0>();
    }
  };
  auto halves = [&](int c) { return c == nlines - 1 ? tail : 2; };  // tail is 2 where steps wrap around
  if constexpr (sizeof(T) == 2) {
    // A step reads the next line's fragments while it multiplies its own, and
    // then has its stage filled again: the DMAs issue under the reads' latency.
#pragma unroll
    for (int c = 0; c < S; ++c)
      if (c < nlines) issue(c, c);
    wait(std::integral_constant<int, S - 1>{}, nlines < S);
    lds_barrier();
    Frags f0, f1;
    read(0, f0);
    int s = 0;
    auto step = [&](int c, const Frags& now, Frags& next) {
      if (c + 1 < nlines) {
        wait(std::integral_constant<int, S - 2>{}, c + S - 1 >= nlines);
        lds_barrier();  // every wave's lines of step c + 1 are in, and those of step c have been read
        const int sn = s + 1 == S ? 0 : s + 1;
        read(sn, next);
        if (c + S < nlines) issue(s, c + S);
        s = sn;
      }
      line_mma<MB>(hidden, now.w, now.h, acc, halves(c));
    };
    for (int c = 0; c < nlines; c += 2) {
      step(c, f0, f1);
      if (c + 1 < nlines) step(c + 1, f1, f0);
    }
  } else {
#pragma unroll
    for (int c = 0; c < S - 1; ++c)
      if (c < nlines) issue(c, c);
    int s = 0;
    for (int c = 0; c < nlines; ++c) {
      wait(std::integral_constant<int, S - 2>{}, nlines - 1 - c <= S - 2);
      lds_barrier();  // every wave's lines of step c are in, and the stage before has been read
      if (c + S - 1 < nlines) issue(s == 0 ? S - 1 : s - 1, c + S - 1);
      Frags f;
      read(s, f);
      line_mma<MB>(hidden, f.w, f.h, acc, halves(c));
      s = s + 1 == S ? 0 : s + 1;
    }
  }
  f32x4 sum[MB][1];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) sum[mb][0] = sizeof(T) == 4 ? acc[mb][0] + acc[mb][1] : acc[mb][0];
  tile_epilogue<MB, 1, 1, NW>(sum, M, V, ntiles, tile, m0, tile * NW + wave, logits, partials, red);
}

template <int MB, int NW>
__global__ __launch_bounds__(NW * kWave)
void vocab_f32_kernel(int M, int K, int V, int ntiles, int mtiles, const float* __restrict__ hidden,
                      const float* __restrict__ w, float* __restrict__ logits, float2* __restrict__ partials,
                      int* __restrict__ clear, int nclear) {
  clear_counters(clear, nclear);
  vocab_lines<float, MB, NW, false>(M, K, V, ntiles, mtiles, hidden, w, logits, partials);
}

template <int MB, int NW, bool PACKED>
__global__ __launch_bounds__(NW * kWave)
void vocab_bf16_kernel(int M, int K, int V, int ntiles, int mtiles, const uint16_t* __restrict__ hidden,
                            const uint16_t* __restrict__ w, float* __restrict__ logits,
                            float2* __restrict__ partials, int* __restrict__ clear, int nclear) {
  clear_counters(clear, nclear);
  vocab_lines<uint16_t, MB, NW, PACKED>(M, K, V, ntiles, mtiles, hidden, w, logits, partials);
}

// Waves per workgroup (16 vocabulary entries each), one to eight: the least
// cost by the lines that the busiest of 256 CUs pulls, its workgroups' entries
// and hidden rows, with 16 lines for a workgroup's start and end, and one and a
// half times the hidden lines of the average CU on top (every workgroup asks
// for the same ones at the same time).  Ties go to more waves.  Fitted to
// measured kernels: 32 x 5120 x 20000 takes 31 us with five waves (250
// workgroups), 40 with eight (157); 52 x 6400 x 10687 47 with four, 51 with
// three or two; 8 x 1504 x 115716 54 with eight, 60 with six.
// `small`: not fewer than four, whose statistics (8 bytes per row and tile) are
// the least workspace a caller may bring.
constexpr int kLineMaxWaves = 8;
constexpr int kLineSmallWaves = 4;
int line_waves(int V, bool small, int mtiles, int mblocks) {
  int best = kLineMaxWaves;
  double least = 0.0;
  for (int nw = kLineMaxWaves; nw >= (small ? kLineSmallWaves : 1); --nw) {
    const double groups = (double)((V + 16 * nw - 1) / (16 * nw)) * mtiles;
    const double rows = 16.0 * mblocks;
    const double cost = std::ceil(groups / 256.0) * (16 * nw + rows + 16) + 1.5 * rows * groups / 256.0;
    if (nw == kLineMaxWaves || cost < least) {
      least = cost;
      best = nw;
    }
  }
  return best;
}

// Workgroups of a (vocabulary tile, M-tile) grid: one per tile, or groups of
// eight tiles whose M-tiles take ids 8 apart.
int line_grid(const VocabPlan& p) { return p.mtiles == 1 ? p.ntiles : (p.ntiles + 7) / 8 * 8 * p.mtiles; }

struct LineCall {
  const VocabPlan& p;
  const void* hidden;
  const void* w;
  float* logits;
  float2* partials;
  hipStream_t stream;
  hipEvent_t e0, e1;
  int* clear;
  int nclear;
};

template <typename T, typename Kern>
hipError_t line_launch(Kern kern, int nw, const LineCall& a) {
  hipExtLaunchKernelGGL(kern, dim3(line_grid(a.p)), dim3(nw * kWave), 0, a.stream, a.e0, a.e1, 0, a.p.M, a.p.K, a.p.V,
                        a.p.ntiles, a.p.mtiles, static_cast<const T*>(a.hidden), static_cast<const T*>(a.w), a.logits,
                        a.partials, a.clear, a.nclear);
  return hipGetLastError();
}

template <int MB, int NW>
hipError_t line_type(bool f32, const LineCall& a) {
  if (f32) return line_launch<float>(vocab_f32_kernel<MB, NW>, NW, a);
  return a.p.packed ? line_launch<uint16_t>(vocab_bf16_kernel<MB, NW, true>, NW, a)
                    : line_launch<uint16_t>(vocab_bf16_kernel<MB, NW, false>, NW, a);
}

template <int MB>
hipError_t line_waves_of(bool f32, const LineCall& a) {
  switch (a.p.waves) {
    case 1: return line_type<MB, 1>(f32, a);
    case 2: return line_type<MB, 2>(f32, a);
    case 3: return line_type<MB, 3>(f32, a);
    case 4: return line_type<MB, 4>(f32, a);
    case 5: return line_type<MB, 5>(f32, a);
    case 6: return line_type<MB, 6>(f32, a);
    case 7: return line_type<MB, 7>(f32, a);
    case 8: return line_type<MB, 8>(f32, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

void line_plan(int blocks, int V, bool small, VocabPlan* p) {
  p->nbw = 1;
  p->mtiles = (blocks + kLineMaxBlocks - 1) / kLineMaxBlocks;
  p->mblocks = (blocks + p->mtiles - 1) / p->mtiles;
  p->waves = line_waves(V, small, p->mtiles, p->mblocks);
}

hipError_t launch_vocab_lines(bool f32, const VocabPlan& p, const void* hidden, const void* w, float* logits,
                              float2* partials, hipStream_t stream, hipEvent_t e0, hipEvent_t e1, int* clear,
                              int nclear) {
  const LineCall a{p, hidden, w, logits, partials, stream, e0, e1, clear, nclear};
  switch (p.mblocks) {
    case 1: return line_waves_of<1>(f32, a);
    case 2: return line_waves_of<2>(f32, a);
    case 3: return line_waves_of<3>(f32, a);
    case 4: return line_waves_of<4>(f32, a);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace sdv
