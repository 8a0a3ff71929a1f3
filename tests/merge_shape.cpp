// The choice of a merge's tile shape: a forced shape is run as it is named at
// every size, tuned and default ones as merge_shape.h states.
#include <cstdio>
#include <initializer_list>

#include "../paper_1905_03277_amd/csrc/merge_shape.h"

using namespace hmfsr;

int main() {
  for (int tiles = 1; tiles < 100000; tiles += 1 + tiles / 50) {
    for (int v = 0; v < 4; ++v)
      for (int tuned = 0; tuned < 4; ++tuned)
        if (burst_shape(v, tuned, tiles) != v) return printf("forced %d, %d tiles: %d\n", v, tiles, burst_shape(v, tuned, tiles)), 1;
    for (int tuned : {0, 1, 3})
      if (burst_shape(-1, tuned, tiles) != tuned) return printf("tuned %d, %d tiles\n", tuned, tiles), 1;
  }
  const int edge[][3] = {{1, 2, kShape64x4}, {192, 2, kShape64x4}, {193, 1, kShape64x8}, {384, 1, kShape64x8}, {385, 0, 2}, {1 << 20, 0, 2}};
  for (auto& e : edge)
    if (size_class(e[0]) != e[1] || burst_shape(-1, kDefaultVariant, e[0]) != e[2]) return printf("%d tiles\n", e[0]), 1;
  if (tiles_64x16(16, 64) != 1 || tiles_64x16(17, 64) != 2 || tiles_64x16(16, 65) != 2) return printf("tiles\n"), 1;
  printf("OK\n");
  return 0;
}
