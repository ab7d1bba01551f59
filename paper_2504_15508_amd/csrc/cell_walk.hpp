// The index walk of the neighbour scan, free of device code: constexpr
// functions compile for the device and for a host program that checks the
// indices.
#pragma once

namespace dplr {
namespace mlp {

constexpr int kDescLanes = 4;  // lanes per particle
// candidates per lane in flight together (16 per particle and chunk; 8 a lane
// need more registers than four waves a SIMD leave)
constexpr int kScan = 4;
constexpr int kScanChunk = kScan * kDescLanes;
constexpr int kScanPad = kScanChunk;  // spare entries behind the sorted particles
constexpr int kSegments = 18;

// Candidates of a particle in cell (cx, cy, cz): the cells start[] of 9 rows
// of three.  A row's cells cx-1, cx, cx+1 are consecutive; at the ends of the
// row they are two ranges (cells nx-1 | 0, 1 or nx-2, nx-1 | 0).  Segment q of the
// walk: row q / 2 (z outer, y inner), its first or second range.
//
// The 16 particles of a wave walk together, chunk by chunk, until the longest
// of their ranges ends.  A particle whose own range is shorter stays at its end
// (j0 <= j1 throughout), so the last chunk it loads begins at j1 at most: of n
// sorted particles the entries 0 .. n + kScanPad - 1 are read, whatever the
// densities.
struct CellWalk {
  const int* start;
  int nx, ny, nz, cx, cy, cz;
  bool on;         // there is such a particle (its ranges are empty otherwise)
  int j0, j1;      // rest of the present segment
  int j0n, j1n;    // the next one (bounds are loaded one segment ahead)

  static constexpr int third(int k) { return (k * 11) >> 5; }  // k / 3 for k < 9
  constexpr int row_y(int q) const { return cy + (q >> 1) - 3 * third(q >> 1) - 1; }
  constexpr int row_z(int q) const { return cz + third(q >> 1) - 1; }
  constexpr bool at_end() const { return cx == 0 || cx == nx - 1; }  // has second ranges
  constexpr void segment(int q, int& a, int& b) const {
    const int y = row_y(q), z = row_z(q);
    const int* row = start + ((z < 0 ? nz - 1 : z >= nz ? 0 : z) * ny + (y < 0 ? ny - 1 : y >= ny ? 0 : y)) * nx;
    if (q & 1) {
      a = row[0];
      b = row[cx == 0 ? 2 : cx == nx - 1 ? 1 : 0];
    } else {
      a = row[cx == 0 ? nx - 1 : cx - 1];
      b = row[cx == 0 ? nx : cx + 2 < nx ? cx + 2 : nx];
    }
    if (!on) b = a;
  }
  // chunk number `chunk` of segment q (one or two steps, dq, between segments)
  constexpr void begin(int q, int chunk, int dq) {
    segment(q, j0, j1);
    j0 = j1 - j0 > kScanChunk * chunk ? j0 + kScanChunk * chunk : j1;
    segment_ahead(q + dq);
  }
  // candidates of the present chunk (0 .. kScanChunk)
  constexpr int left() const { return j1 - j0 < kScanChunk ? j1 - j0 : kScanChunk; }
  // one chunk on, to the range's end at most; the particle has more of the
  // segment if j0 < j1 then
  constexpr void advance() { j0 = j0 + kScanChunk < j1 ? j0 + kScanChunk : j1; }
  // the next segment becomes the present one; q: its successor
  constexpr void next_segment(int q) {
    j0 = j0n;
    j1 = j1n;
    segment_ahead(q);
  }
  constexpr void segment_ahead(int q) { segment(q < kSegments ? q : kSegments - 1, j0n, j1n); }
};

}  // namespace mlp
}  // namespace dplr
