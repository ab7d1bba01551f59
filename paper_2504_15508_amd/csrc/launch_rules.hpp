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

}  // namespace dplr
