// Block-wide counting-sort helpers shared by the Alltoall kernels, for gfx950.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "wave.h"

namespace taccl {

// The top `bits` bits of x (0 for bits = 0): one bit-field extract, whose
// width 0 gives 0
__device__ __forceinline__ uint32_t top_bits(uint32_t x, uint32_t bits) {
  return __builtin_amdgcn_ubfe(x, 32u - bits, bits);
}

// Exclusive scan of cnt[0..n) in place with cnt[n] = total (all threads
// call; cnt 16-byte aligned; cnt[n+1..n+3] are overwritten as well). Each
// wavefront takes a contiguous range of 4-word groups and each lane one
// group per round, so a round reads 1 KB of consecutive words: one pass
// for the wavefront totals, one to write the prefixes.
__device__ inline void block_excl_scan4(uint32_t *cnt, int n, uint32_t *wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x >> 6;
  const int ng = (n >> 2) + 1;  // groups up to and including index n
  const int gpw = ((ng + nw - 1) / nw + 63) & ~63;
  const int g0 = wave * gpw;
  uint4 *c4 = (uint4 *)cnt;
  auto group = [&](int g) {  // entries from index n on count as 0
    uint4 x = g < ng ? c4[g] : make_uint4(0u, 0u, 0u, 0u);
    const int e = 4 * g;
    x.x = e < n ? x.x : 0u;
    x.y = e + 1 < n ? x.y : 0u;
    x.z = e + 2 < n ? x.z : 0u;
    x.w = e + 3 < n ? x.w : 0u;
    return x;
  };
  uint32_t sum = 0;
  for (int r = 0; r < gpw; r += 64) {
    const uint4 x = group(g0 + r + lane);
    sum += x.x + x.y + x.z + x.w;
  }
  const uint32_t wt = (uint32_t)__builtin_amdgcn_readlane((int)wave_scan_add(sum), 63);
  if (lane == 0) wsum[wave] = wt;
  __syncthreads();
  const uint32_t ws = row_scan_add(lane < nw ? wsum[lane] : 0u);
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  uint32_t run = w ? (uint32_t)__builtin_amdgcn_readlane((int)ws, w - 1) : 0u;
  for (int r = 0; r < gpw; r += 64) {
    const int g = g0 + r + lane;
    const uint4 x = group(g);
    const uint32_t gs = x.x + x.y + x.z + x.w;
    const uint32_t inc = wave_scan_add(gs);
    const uint32_t e0 = run + inc - gs;
    // the group holding index n receives the total there (later entries
    // count as 0)
    if (g < ng) c4[g] = make_uint4(e0, e0 + x.x, e0 + x.x + x.y, e0 + x.x + x.y + x.z);
    run += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
  }
  __syncthreads();
}

// Rank of entry me among the entries [b, e) of its bucket, four at a time
// (the staging array has three spare entries past its end; entries past the
// bucket never count).
__device__ __forceinline__ uint32_t rank_in_bucket(const uint64_t *e64, uint32_t b, uint32_t e,
                                                   uint64_t me) {
  uint32_t rank = 0;
  for (uint32_t y = b; y < e; y += 4) {
    uint64_t m[4];
#pragma unroll
    for (int t = 0; t < 4; t++) m[t] = e64[y + t];
#pragma unroll
    for (int t = 0; t < 4; t++) rank += (uint32_t)((y + t < e) & (m[t] < me));
  }
  return rank;
}

}  // namespace taccl
