// Rules of launches on sizes, free of device code, so that a host program can
// check them over all sizes.
#pragma once

#include <cstdint>

namespace dplr {

// At most this many chunks: the placement adds up the chunk histograms itself,
// all of a bin's in flight together, instead of k_bin_colscan (a launch of
// 3.4 us at 16,384 particles).
constexpr int kPlaceScanChunks = 16;
constexpr int kPlaceScanBins = 4096;  // and at most this many bins (4 a thread)

// Particles per chunk of the counting sort, for n particles in nbins bins: a
// multiple of align that makes at most max_chunks chunks (what the histograms
// hold), and few of them where that saves the column scan.
constexpr int64_t sort_chunk(int64_t n, int nbins, int max_chunks, int64_t align) {
  constexpr int64_t few = 1024;
  const int most = max_chunks < kPlaceScanChunks ? max_chunks : kPlaceScanChunks;
  return n <= few * most && nbins <= kPlaceScanBins
             ? few
             : ((n + max_chunks - 1) / max_chunks + align - 1) / align * align;
}

// Threads of a block of the fused 2-3-5 kernels for pts points: one radix-10
// butterfly each, a multiple of 64 in [least, most].
constexpr int fused_threads(int64_t pts, int least, int most) {
  const int64_t t = (pts / 10 + 63) / 64 * 64;
  return t < least ? least : t > most ? most : (int)t;
}

// The plane spread: at least 512, because its visits (7,500 a block for 288,768
// particles) take longer than the transforms.  Steps of 288,768 particles on
// 60^3 at order 8: 209 us with a butterfly a thread (384), 203 with 512; 80,000
// on 40^3 at order 5: 74.5 (256) and 70.3; FP64 at 60^3: 96.1 (384) and 94.3;
// 512 particles on 12 x 18 x 12: the same.  (768 for every FP32 plane: 199 and
// 71.0 us.)
constexpr int fused_spread_threads(int64_t pts, int most) { return fused_threads(pts, 512, most); }

// The inverse plane pass: at least 512 from 512 points on, where a stage's small
// radices have work for them (a step on 54^3: 93.1 us with 320 and 90.9; FP64
// 60^3: 96.0 with 384 and 95.4; 24^3: the same), 256 below, where more only wait
// at the barriers (12 x 18 planes in FP64: the pass 6.6 us with 256, 8.7 with 1,024).
constexpr int fused_inverse_threads(int64_t pts, int most) { return fused_threads(pts, pts < 512 ? 256 : 512, most); }

// The z pass for `points` points of one field a block: a thread per point (one
// round of the loads and of the Poisson sums) where the blocks are few, a
// butterfly of both fields a thread where they fill the compute units.  Few:
// 40^3 (100 blocks, 128 threads by butterflies) 74.5 and 71.2 us a step, 54^3 (729
// blocks, 64) 93.1 and 90.2, FP64 30^3 (225 blocks, 64) 83.2 and 80.5; many: FP64
// 90^3 (2,025 blocks, 128) 203 and, with 192, 219; 81^3 (6,561 blocks, 64) 186 and,
// with 128, 197.
constexpr int64_t kFusedZFewBlocks = 1024;
constexpr int fused_z_threads(int64_t points, int64_t blocks, int most) {
  return blocks <= kFusedZFewBlocks ? fused_threads(10 * points, 64, most) : fused_threads(2 * points, 64, most);
}

}  // namespace dplr
