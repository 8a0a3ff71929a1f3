// Which tile shape a merge runs (host).
#pragma once

namespace hmfsr {

// Shapes of launch_merge: the four of kMergeVariants (64 x 32 with 256 and 512
// threads, 64 x 16 with 256 and 128), and the default's smaller forms for
// small outputs, 64 x 8 and 64 x 4 with 256 threads.
constexpr int kDefaultVariant = 2;  // 64 x 16 tile, 256 threads
constexpr int kShape64x8 = 4, kShape64x4 = 5;

inline int tiles_64x16(int OH, int OW) { return ((OW + 63) / 64) * ((OH + 15) / 16); }

// Size class of an output of `tiles` 64 x 16 tiles, and its default shape: 64 x
// 16 (0) where that fills the 256 compute units, else 64 x 8 (1) or 64 x 4
// (2), so that more of them work and a frame's chain (stage, Omega, one to
// four pixels a thread) is shorter. A pixel's arithmetic does not depend on
// the shape: the results are the same bits. Measured with 64 x 16 tiles / 64 x
// 8 / 64 x 4, us per merge: 8 x 256 x 256 (64 tiles) 54.6 / 39.5 / 33.7, 8 x
// 384 x 512 (192) 57.5 / 48.5 / 46.0, 8 x 256 x 256 at scale 2 (256) 51.1 /
// 44.9 / 47.0, 8 x 512 x 512 at 1.5 (576) 75.9 / 75.3 / 82.6, 5 x 750 x 1002
// at 1.5 (1704) 98 / 114 / 139.
constexpr int kSizeClasses = 3;
inline int size_class(int tiles) { return tiles <= 192 ? 2 : (tiles <= 384 ? 1 : 0); }
inline int default_shape(int tiles) {
  const int c = size_class(tiles);
  return c == 2 ? kShape64x4 : (c == 1 ? kShape64x8 : kDefaultVariant);
}

// Shape of a burst's own merge: `forced` (HMFSR_MERGE_VARIANT; -1: not set) as
// it is, else the tuned (or untuned default) index, of which the default one
// stands for the default shape of the output's size.
inline int burst_shape(int forced, int tuned, int tiles) {
  if (forced >= 0) return forced;
  return tuned == kDefaultVariant ? default_shape(tiles) : tuned;
}

}  // namespace hmfsr
