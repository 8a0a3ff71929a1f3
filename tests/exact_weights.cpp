// Scales that interpolate R_hat with one rounded weight keep the fraction of
// every output row and column within a cell clear of 1 (see exact_weights).
#include <cstdio>

#include "../paper_1905_03277_amd/csrc/merge_common.h"

using namespace hmfsr;

int main() {
  long long checked = 0;
  for (int m = 64; m <= 512; ++m) {
    const double s = (double)(float)(m / 64.0);
    if (exact_weights(s)) return printf("scale %g takes exact weights\n", s), 1;
    for (int C = 0; C < (int)(32768 * s + 0.5); ++C, ++checked) {
      const double h = out_pos(C, s) * 0.5 - 0.5, f = h - floor(h);
      if (f > 1.0 - 1.0 / 1024 + 1e-9) return printf("scale %g position %d fraction 1 - %g\n", s, C, 1.0 - f), 1;
    }
  }
  for (float s : {1.1f, 1.3f, 2.2f, 3.7f, 7.3f, 1.00001f, 7.99f})
    if (!exact_weights((double)s)) return printf("scale %g takes one weight\n", s), 1;
  printf("OK %lld positions\n", checked);
  return 0;
}
