// Launch shapes of kernels whose blocks hold independent wavefronts (host).
#pragma once

#include <algorithm>
#include <cstdint>

namespace taccl {

// LDS of a CU, of the largest block, and the steps a block's LDS comes in
constexpr int32_t kLdsBytes = 160 * 1024, kLdsStep = 1280;

// Wavefronts per block and resident blocks per CU (0: not yet computed).
struct LaunchShape {
  int waves = 0, per_cu = 0;
  int resident() const { return waves * per_cu; }
};

// Blocks of `waves` wavefronts that are resident on a CU of four SIMDs, each
// of which holds per_simd wavefronts of the kernel. From four wavefronts on a
// block puts ceil(waves / 4) of them on some SIMD, and blocks don't interleave
// to fill up what it leaves free on the others: of two blocks of 10 at 5
// wavefronts per SIMD one waits for the other.
inline int blocks_by_waves(int waves, int per_simd) {
  return waves < 4 ? 4 * per_simd / waves : per_simd / ((waves + 3) / 4);
}

inline int blocks_by_lds(int64_t bytes, int64_t lds_per_cu) {
  return (int)(lds_per_cu / std::max<int64_t>((bytes + kLdsStep - 1) / kLdsStep * kLdsStep, kLdsStep));
}

// The block size of 1 to max_waves wavefronts with the most resident
// wavefronts per CU: `shared` bytes of LDS per block and `wave` bytes per
// wavefront, at most max_lds per block. Counting blocks by the bytes asked
// for and by 4 * per_simd / waves took shapes whose last block was not
// resident, so that its candidates came in a round of their own: 11204
// contiguous Allgathers on two 8-rank meshes, 82.3 us with two blocks of 10
// wavefronts, 64.8 us with two of 8; 20000 Allgathers on two nodes of 7
// ranks, 182 us with three blocks of 4 (54528 bytes), 126 us with one of 12.
// whole: a single block is taken before several that hold as many wavefronts
// (the ranked kernel deals candidates out over the blocks then: the same
// Allgathers 125 us with three blocks of 4, 114 us with one of 12).
inline LaunchShape resident_shape(int64_t shared, int64_t wave, int max_waves, int per_simd,
                                  bool whole = false, int64_t max_lds = kLdsBytes,
                                  int64_t lds_per_cu = kLdsBytes) {
  LaunchShape best{1, 1};
  int most = 0;
  for (int w = 1; w <= max_waves; w++) {
    const int64_t bytes = shared + w * wave;
    if (bytes > max_lds) break;
    const int n = std::min(blocks_by_lds(bytes, lds_per_cu), blocks_by_waves(w, per_simd));
    if (n * w > most || (n * w == most && n == 1 && whole)) {
      most = n * w;
      best = LaunchShape{w, n};
    }
  }
  return best;
}

// Blocks for a batch of n candidates, one per wavefront at a time, all of
// them resident. spread: the kernel deals candidates out over the blocks
// before it gives a block a second one, so a small batch takes as many blocks
// as it has candidates; else a block takes as many as it has wavefronts.
inline int wave_grid(const LaunchShape &s, int64_t n, int cus, bool spread) {
  const int64_t w = spread ? 1 : s.waves;
  return (int)std::min<int64_t>((n + w - 1) / w, (int64_t)std::max(cus, 1) * s.per_cu);
}

}  // namespace taccl
