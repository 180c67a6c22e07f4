// Rules that choose a launch from counts the host knows, in plain C++ so that
// they can be checked without a GPU.
#pragma once

#include <stdint.h>

namespace fmm {
namespace rules {

// Waves that share a segment of the near field (p2p.hip): about four on every
// SIMD (1,024 of them).  One wave takes 150 us over a full segment, so few
// segments left the launch waiting for single waves; with many, more waves per
// segment only add barriers.  Measured, one wave / here: 20,000 uniform points,
// 512 leaves 228 / 88 us (of which the split of the lanes a third), 47,003
// points on a sphere 1,001 / 531, 3,000 points binary32 141 / 35; from 2,048
// segments on within 2 % (issue-bound: 1.42e12 interactions/s on 2^22 Plummer
// points).
// In binary64 the waves share a segment by its entries (`entries` of all
// segments: the leaves' strong lists).  Leaves of more than about 2,000 points
// leave a segment fewer entries than waves, and the idle ones hold LDS that
// other segments' could have.  With eight or four waves whatever the entries /
// here, in ms: 64 leaves, 10^6 uniform points at theta 0.9 (one entry) 638 /
// 192, 200,000 (three) 24.4 / 12.5, 128,000 (four) 6.1 / 4.1; 8 leaves, 20,000
// points (three) 1.00 / 0.61, 12,000 (four) 0.59 / 0.59, with four waves 0.64.
inline int p2p_waves(int64_t nseg, int64_t entries, bool f32) {
  int w = nseg <= 512 ? 8 : nseg <= 2048 ? 4 : 1;
  if (f32) return w;  // the chunks of a segment are dealt to the waves in turn
  if (w == 8 && entries < 4 * nseg) w = 4;
  if (entries < 2 * nseg) w = 1;
  return w;
}

// A bisection round of the tree build (tree.hip) runs chunked, every segment cut
// into chunks of kChunk points that blocks of their own take, or as one block
// of up to 1,024 threads per segment.  A chunked round is 20 launches, bound by
// the host that makes them up to some 10^5 points; one block takes a segment's
// points one 1,024 after the other.  So the largest segment decides, down to
// kChunkedMin points in the smallest (below, most chunks of most segments would
// be empty): chunked from kChunkedMax points in the largest on, up to
// kChunkedSeg segments.  20,000 points (3 levels), rounds chunked from 8,192
// points on / here: the build 477 / 270 us.  Trees off the median, rounds
// chunked only when the smallest segment has kChunkedMax points / here: 10^6
// points of a Gaussian mixture (4 levels, eta 0.9) 4.86 / 4.16 ms, 500,000 of
// which 20,000 lie apart (4 levels, eta 0) 3.73 / 2.40.
constexpr int64_t kChunk = 2048;
constexpr int64_t kChunkedMin = 4 * kChunk, kChunkedMax = 16 * kChunk;
constexpr int64_t kChunkedSeg = 512;
// nseg segments of seg_min to seg_max points
inline bool round_chunked(int64_t nseg, int64_t seg_min, int64_t seg_max) {
  return nseg <= kChunkedSeg && seg_min >= kChunkedMin && seg_max >= kChunkedMax;
}

}  // namespace rules
}  // namespace fmm
