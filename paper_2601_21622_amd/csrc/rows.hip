// Vocabulary projection, row schedule (gfx950): bfloat16, more than 64 hidden
// rows, row-major W, 128- or 256-wide vocabulary tiles.
//
// The deep schedule's MFMA operand loads from row-major W touch 32 rows x 32
// bytes per instruction, so each 128-byte line is asked for four times and
// holds a miss slot of the CU four times.  Here a wave DMAs its W rows, and the
// workgroup its hidden rows, as whole lines (eight per instruction, 64 k) into
// LDS, straight from their row-major layouts: no repacking launch.  Of a
// 32-row group (four 1 KB blocks of eight rows), unit u of row r sits at slot
// 8r + (u + r / 2) mod 8: a fragment read takes 32 rows of one unit, 16 lanes
// {0-3, 12-15, 20-27} and then the others at a time, and every such 16 rows
// cover all 64 banks once.
//
// One workgroup of four waves per CU; wave w owns blocks (tile*4 + w)*NB .. +NB
// of 32 vocabulary entries against MB blocks of 32 hidden rows.  A line is four
// 16-wide MFMA steps; the fragments of the next step are read while one is
// multiplied, the last step of a line reading the first of the next line.
// Half-way through line c the wave waits for its DMAs of line c + 1, passes
// the barrier (every wave's lines are in, and the stage of line c - 1 has been
// read by all) and issues line c + S - 1 between the MFMAs of the second half.
#include <hip/hip_ext.h>

#include <algorithm>

#include "common.h"
#include "launch.h"
#include "vocab_tile.h"

namespace sdv {

namespace {

constexpr int kRowWaves = 4;

// Stages that fit the CU's 160 KB next to the epilogue's floats.
constexpr int row_stages(int mb, int nb) {
  const int n = (160 * 1024 - kRowWaves * mb * 32 * 4) / ((4 * mb + 4 * kRowWaves * nb) * 1024);
  return n < 5 ? n : 5;
}

template <int MB, int NB>
__global__ __launch_bounds__(kRowWaves * kWave, 1)
void vocab_bf16_rows_kernel(int M, int K, int V, int ntiles, int mtiles, const uint16_t* __restrict__ hidden,
                            const uint16_t* __restrict__ w, float* __restrict__ logits, float2* __restrict__ partials,
                            int* __restrict__ clear, int nclear) {
  constexpr int NW = kRowWaves;
  constexpr int kHBlocks = 4 * MB;
  constexpr int kStage = (kHBlocks + 4 * NW * NB) * 1024;
  constexpr int S = row_stages(MB, NB);
  constexpr int kOps = MB + 4 * NB;      // DMAs per wave and line
  constexpr int kHalf = 2 * MB * NB;     // MFMAs of half a line
  static_assert(S >= 3 && (S - 2) * kOps < 64, "three stages; vmcnt holds 6 bits");
  clear_counters(clear, nclear);
  __shared__ __align__(1024) unsigned char lds[S * kStage];
  __shared__ float red[NW][MB * 32];

  // The M-tiles of one vocabulary tile share an XCD (ids 8 apart).
  const int grp = 8 * mtiles;
  const int tile = (blockIdx.x / grp) * 8 + (blockIdx.x & 7);
  if (tile >= ntiles) return;
  const int m0 = ((blockIdx.x % grp) >> 3) * MB * 32;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int blk0 = (tile * NW + wave) * NB;
  const int nlines = (K + 63) / 64;
  const bool odd = K % 64 != 0;  // the last line has only its first half

  // Lane l of block q of a group brings unit (l % 8) - r / 2 of row r = 8q + l
  // / 8.  Rows past V and past M repeat the last row (lines already requested;
  // results never stored); the last line's missing half repeats its first.
  auto unit = [&](int q) { return ((lane & 7) - 4 * (q & 1) - (lane >> 4)) & 7; };
  const char* wsrc[NB][4];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = min((blk0 + nb) * 32 + 8 * q + (lane >> 3), V - 1);
      wsrc[nb][q] = reinterpret_cast<const char*>(w + (int64_t)row * K) + unit(q) * 16;
    }
  const char* hsrc[MB];  // block `wave` of every 32-row group
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int row = min(m0 + mb * 32 + 8 * wave + (lane >> 3), M - 1);
    hsrc[mb] = reinterpret_cast<const char*>(hidden + (int64_t)row * K) + unit(wave) * 16;
  }
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
  // DMA j of line c into stage s.
  auto issue_op = [&](int j, int s, int c) {
    const uint32_t dst = lds_base + (uint32_t)s * kStage;
    const bool half = odd && c == nlines - 1;
    const int64_t o = (int64_t)c * kLineBytes;
    if (j < MB) {
      const int u = unit(wave);
      line_dma<false>(hsrc[j] + o + (half ? ((u & 3) - u) * 16 : 0), dst + (4 * j + wave) * 1024);
    } else {
      const int nb = (j - MB) >> 2, q = (j - MB) & 3;
      const int u = unit(q);
      line_dma<true>(wsrc[nb][q] + o + (half ? ((u & 3) - u) * 16 : 0),
                     dst + (kHBlocks + (wave * NB + nb) * 4 + q) * 1024);
    }
  };
  const int r = lane & 31;
  auto read = [&](int s, int ks, bf16x8 (&wf)[NB], bf16x8 (&hf)[MB]) {
    const unsigned char* src = lds + s * kStage + (r >> 3) * 1024 + (r & 7) * 128 +
                               ((2 * ks + (lane >> 5) + (r >> 1)) & 7) * 16;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      wf[nb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + (kHBlocks + (wave * NB + nb) * 4) * 1024));
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
      hf[mb] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(src + 4 * mb * 1024));
  };

  f32x16 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[mb][nb][e] = 0.f;

#pragma unroll
  for (int c = 0; c < S - 1; ++c)
    if (c < nlines) {
#pragma unroll
      for (int j = 0; j < kOps; ++j) issue_op(j, c, c);
    }
  // Line 0: the lines after it may still be in flight.
  if (nlines >= S - 1)
    wait_vmcnt<(S - 2) * kOps>();
  else
    wait_vmcnt<0>();
  lds_barrier();
  bf16x8 wf[2][NB], hf[2][MB];
  read(0, 0, wf[0], hf[0]);
  int s = 0;
  for (int c = 0; c < nlines; ++c) {
    const bool more = c + 1 < nlines;
    const bool fill = c + S - 1 < nlines;
    const int sn = s + 1 == S ? 0 : s + 1;  // stage of line c + 1
    const int sp = s == 0 ? S - 1 : s - 1;  // stage of line c - 1, for line c + S - 1
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      if (ks == 2) {
        if (odd && !more) break;
        if (more) {
          if (c + S - 2 < nlines)
            wait_vmcnt<(S - 3) * kOps>();
          else
            wait_vmcnt<0>();
          lds_barrier();
        }
      }
      if (ks < 3)
        read(s, ks + 1, wf[(ks + 1) & 1], hf[(ks + 1) & 1]);
      else if (more)
        read(sn, 0, wf[0], hf[0]);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          acc[mb][nb] = mfma32x32x16(wf[ks & 1][nb], hf[ks & 1][mb], acc[mb][nb]);
          if (ks >= 2 && fill) {
            const int i = (ks - 2) * MB * NB + mb * NB + nb;
#pragma unroll
            for (int j = i * kOps / kHalf; j < (i + 1) * kOps / kHalf; ++j) issue_op(j, sp, c + S - 1);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    s = sn;
  }
  tile_epilogue32<MB, NB, NW>(acc, M, V, ntiles, tile, m0, blk0, logits, partials, red);
}

template <int MB, int NB>
hipError_t launch_rows(const VocabPlan& p, const void* hidden, const void* w, float* logits, float2* partials,
                       hipStream_t stream, hipEvent_t e0, hipEvent_t e1, int* clear, int nclear) {
  hipExtLaunchKernelGGL((vocab_bf16_rows_kernel<MB, NB>), dim3((p.ntiles + 7) / 8 * 8 * p.mtiles),
                        dim3(kRowWaves * kWave), 0, stream, e0, e1, 0, p.M, p.K, p.V, p.ntiles, p.mtiles,
                        static_cast<const uint16_t*>(hidden), static_cast<const uint16_t*>(w), logits, partials, clear,
                        nclear);
  return hipGetLastError();
}

// Most 32-row blocks per workgroup that leave room for three stages.
constexpr int kRowCap1 = 8, kRowCap2 = 5;
static_assert(row_stages(kRowCap1, 1) >= 3 && row_stages(kRowCap2, 2) >= 3, "three stages");

}  // namespace

bool rows_plan(int blocks32, VocabPlan* p) {
  if (p->waves != kRowWaves || (p->nbw != 2 && p->nbw != 4)) return false;
  const int cap = p->nbw == 2 ? kRowCap1 : kRowCap2;
  p->mtiles = (blocks32 + cap - 1) / cap;
  p->mblocks = (blocks32 + p->mtiles - 1) / p->mtiles;
  return true;
}

hipError_t launch_vocab_rows(const VocabPlan& p, const void* hidden, const void* w, float* logits, float2* partials,
                             hipStream_t stream, hipEvent_t e0, hipEvent_t e1, int* clear, int nclear) {
#define SDV_R(B, N) \
  case B: return launch_rows<B, N>(p, hidden, w, logits, partials, stream, e0, e1, clear, nclear);
  if (p.nbw == 4) {
    switch (p.mblocks) {
      SDV_R(3, 2) SDV_R(4, 2) SDV_R(5, 2)
      default: return hipErrorInvalidValue;
    }
  }
  switch (p.mblocks) {
    SDV_R(3, 1) SDV_R(4, 1) SDV_R(5, 1) SDV_R(6, 1) SDV_R(7, 1) SDV_R(8, 1)
    default: return hipErrorInvalidValue;
  }
#undef SDV_R
}

}  // namespace sdv
