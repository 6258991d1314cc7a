// Repacking of the hidden rows for the deep projection schedules: by a launch
// of its own, or (in a step on the caller's hidden rows) by workgroups that
// follow the attention's in its launch, where it costs the step nothing.
#pragma once

#include "common.h"
#include "launch.h"

namespace sdv {

constexpr int kPackThreads = 256;
// 16-byte pieces per thread, loaded together: four behind the attention, whose
// launch hides them, one in a launch of its own, which is done sooner on more CUs
// (sd_verify_logits, 1000 x 1024 x 4000: 46.2 us, 47.5 with four; 224 x 4096 x
// 8000: 69.6, 70.2).
constexpr int kPackEach = 4;

// Counters a later launch on the stream expects at zero.
__device__ __forceinline__ void clear_ints(int* __restrict__ clear, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) clear[i] = 0;
}

// Hidden rows [M][K] -> fragments [K/16][ceil(M/32)][64 lanes][8]: lane l of
// fragment (k16, mb) holds row mb*32 + l%32, k 16*k16 + 8*(l/32) .. +8; rows
// past M are zero.  Block `block` of kPackThreads threads; writes coalesced.
template <int EACH>
__device__ __forceinline__ void pack_hidden_block(const PackJob& j, int block) {
  if (block == 0) clear_ints(j.clear, j.nclear);
  const int mbt = (j.M + 31) / 32;
  const int64_t pieces = (int64_t)(j.K / 16) * mbt * 64;
  const int64_t i0 = (int64_t)block * (kPackThreads * EACH) + threadIdx.x;
  u32x4 v[EACH];
#pragma unroll
  for (int e = 0; e < EACH; ++e) {
    const int64_t i = i0 + e * kPackThreads;
    const int lane = (int)(i & 63);
    const int64_t f = i >> 6;
    const int mb = (int)(f % mbt);
    const int k16 = (int)(f / mbt);
    const int row = mb * 32 + (lane & 31);
    v[e] = u32x4{0u, 0u, 0u, 0u};
    if (i < pieces && row < j.M)
      v[e] = *reinterpret_cast<const u32x4*>(j.hidden + (int64_t)row * j.K + k16 * 16 + (lane >> 5) * 8);
  }
#pragma unroll
  for (int e = 0; e < EACH; ++e) {
    const int64_t i = i0 + e * kPackThreads;
    if (i < pieces) *reinterpret_cast<u32x4*>(j.out + i * 8) = v[e];
  }
}

}  // namespace sdv
