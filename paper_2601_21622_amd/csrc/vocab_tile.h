// Parts shared by the vocabulary projection's schedules (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.h"

namespace sdv {

// Counters a later launch on the stream expects at zero (the acceptance's
// arrival counters): cleared by the first workgroup of a vocabulary launch.
__device__ __forceinline__ void clear_counters(int* __restrict__ clear, int nclear) {
  if (blockIdx.x == 0 && blockIdx.y == 0)
    for (int i = threadIdx.x; i < nclear; i += blockDim.x) clear[i] = 0;
}

// Epilogue of one workgroup of WM x WN waves.  Wave (wm, wn) = (wave / WN,
// wave % WN) holds in acc[mb][nb] hidden row m0 + r0 + mb*16 + (lane & 15),
// with r0 = wm*MBW*16, and vocabulary entries (blk0 + nb)*16 + (lane>>4)*4
// .. +3, where blk0 is the wave's first 16-entry block.  Writes the logits,
// then the tile's per-row maximum and sum of exponentials, combined over the
// WN waves that share the rows through `red` ([WN][WM*MBW*16] floats).
template <int MBW, int NBW, int WM, int WN>
__device__ __forceinline__ void tile_epilogue(const f32x4 (&acc)[MBW][NBW], int M, int V, int ntiles, int tile,
                                              int m0, int blk0, float* __restrict__ logits,
                                              float2* __restrict__ partials, float (*red)[WM * MBW * 16]) {
  const int wave = threadIdx.x >> 6;
  const int wn = wave % WN;
  const int r0 = (wave / WN) * MBW * 16;
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15;
  const int lg = lane >> 4;
  float tmax[MBW];
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) {
    const int m = m0 + r0 + mb * 16 + lr;
    float x = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
      const int v0 = (blk0 + nb) * 16 + lg * 4;
      if (m < M) {
        float* dst = logits + (int64_t)m * V + v0;
        if (v0 + 3 < V) {
          *reinterpret_cast<f32x4_u*>(dst) = acc[mb][nb];
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (v0 + i < V) dst[i] = acc[mb][nb][i];
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) x = (v0 + i < V) ? fmaxf(x, acc[mb][nb][i]) : x;
    }
    x = fmaxf(x, __shfl_xor(x, 16));
    x = fmaxf(x, __shfl_xor(x, 32));
    if (lg == 0) red[wn][r0 + mb * 16 + lr] = x;
  }
  __syncthreads();
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) {
    const int r = r0 + mb * 16 + lr;
    float x = red[0][r];
#pragma unroll
    for (int w = 1; w < WN; ++w) x = fmaxf(x, red[w][r]);
    tmax[mb] = x;
  }
  __syncthreads();
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) {
    float sm = 0.f;
#pragma unroll
    for (int nb = 0; nb < NBW; ++nb) {
      const int v0 = (blk0 + nb) * 16 + lg * 4;
#pragma unroll
      for (int i = 0; i < 4; ++i) sm += (v0 + i < V) ? expf(acc[mb][nb][i] - tmax[mb]) : 0.f;
    }
    sm += __shfl_xor(sm, 16);
    sm += __shfl_xor(sm, 32);
    if (lg == 0) red[wn][r0 + mb * 16 + lr] = sm;
  }
  __syncthreads();
  if (wn == 0 && lg == 0) {
#pragma unroll
    for (int mb = 0; mb < MBW; ++mb) {
      const int r = r0 + mb * 16 + lr;
      const int m = m0 + r;
      if (m < M) {
        // Neighbours first, then the pairs, and so on (a last odd one as it is).
        float part[WN];
#pragma unroll
        for (int w = 0; w < WN; ++w) part[w] = red[w][r];
#pragma unroll
        for (int step = 1; step < WN; step *= 2)
#pragma unroll
          for (int w = 0; w + step < WN; w += 2 * step) part[w] += part[w + step];
        const float sm = part[0];
        partials[(int64_t)m * ntiles + tile] = make_float2(tmax[mb], sm);
      }
    }
  }
}

// Bytes of a row brought per step by the schedules that DMA whole lines.
constexpr int kLineBytes = 128;

// DMA of one 1 KB block: lane l copies 16 bytes from g into LDS bytes lds +
// 16l .. +15 (lds wave-uniform).  From inline assembly, so that the compiler
// inserts no waits of its own between it and reads of other stages; the
// kernel's vmcnt waits order it.  It sets M0 itself, and waits the one state
// that a load into LDS needs after that (the compiler's hazard pass does not
// see into the string).
template <bool NT>
__device__ __forceinline__ void line_dma(const char* g, uint32_t lds) {
  if (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off nt" : : "s"(lds), "v"(g) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds), "v"(g) : "m0", "memory");
}

// Fixed-order combination of the NW per-wave values of row r.
template <int NW, int R>
__device__ __forceinline__ float waves_max(const float (*red)[R], int r) {
  float x = fmaxf(fmaxf(red[0][r], red[1][r]), fmaxf(red[2][r], red[3][r]));
  if (NW == 8) x = fmaxf(x, fmaxf(fmaxf(red[4][r], red[5][r]), fmaxf(red[6][r], red[7][r])));
  return x;
}
template <int NW, int R>
__device__ __forceinline__ float waves_sum(const float (*red)[R], int r) {
  float x = (red[0][r] + red[1][r]) + (red[2][r] + red[3][r]);
  if (NW == 8) x += (red[4][r] + red[5][r]) + (red[6][r] + red[7][r]);
  return x;
}

template <int MB, int NB, int NW>
__device__ __forceinline__ void tile_epilogue32(const f32x16 (&acc)[MB][NB], int M, int V, int ntiles, int tile,
                                                int m0, int blk0, float* __restrict__ logits,
                                                float2* __restrict__ partials, float (*red)[MB * 32]) {
  const int wave = threadIdx.x >> 6;
  const int lane = threadIdx.x & 63;
  const int j = lane & 31;
  const int h = lane >> 5;
  float tmax[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = m0 + mb * 32 + j;
    float x = -INFINITY;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int v0 = (blk0 + nb) * 32 + 8 * g + 4 * h;
        const f32x4 q = {acc[mb][nb][4 * g], acc[mb][nb][4 * g + 1], acc[mb][nb][4 * g + 2], acc[mb][nb][4 * g + 3]};
        if (m < M) {
          float* dst = logits + (int64_t)m * V + v0;
          if (v0 + 3 < V) {
            *reinterpret_cast<f32x4_u*>(dst) = q;
          } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
              if (v0 + i < V) dst[i] = q[i];
          }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) x = (v0 + i < V) ? fmaxf(x, q[i]) : x;
      }
    }
    x = fmaxf(x, __shfl_xor(x, 32));
    if (h == 0) red[wave][mb * 32 + j] = x;
  }
  __syncthreads();
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int r = mb * 32 + j;
    tmax[mb] = waves_max<NW, MB * 32>(red, r);
  }
  __syncthreads();
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    float sm = 0.f;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int v = (blk0 + nb) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        sm += (v < V) ? expf(acc[mb][nb][r] - tmax[mb]) : 0.f;
      }
    sm += __shfl_xor(sm, 32);
    if (h == 0) red[wave][mb * 32 + j] = sm;
  }
  __syncthreads();
  if (wave == 0 && h == 0) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
      const int r = mb * 32 + j;
      const int m = m0 + r;
      if (m < M) {
        const float sm = waves_sum<NW, MB * 32>(red, r);
        partials[(int64_t)m * ntiles + tile] = make_float2(tmax[mb], sm);
      }
    }
  }
}

}  // namespace sdv
