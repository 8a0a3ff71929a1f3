// Every tile of a launch is taken by exactly one workgroup, for launches below,
// at and above a whole number of runs.
#include <cstdio>
#include <vector>

#include "../paper_1905_03277_amd/csrc/device_util.h"

int main() {
  std::vector<int> sizes;
  for (int n = 1; n <= 200; ++n) sizes.push_back(n);
  for (int n : {1023, 1024, 1025, 11907, 36100, 262144, 1048579}) sizes.push_back(n);
  for (int n : sizes) {
    std::vector<char> seen(n, 0);
    for (int b = 0; b < n; ++b) {
      const int t = hmfsr::xcd_tile_runs<8>(b, n);
      if (t < 0 || t >= n || seen[t]) {
        std::printf("n %d, workgroup %d: tile %d\n", n, b, t);
        return 1;
      }
      seen[t] = 1;
    }
  }
  std::printf("OK\n");
  return 0;
}
