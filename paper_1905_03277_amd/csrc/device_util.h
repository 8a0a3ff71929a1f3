// Small device helpers shared by the kernels.
#pragma once

#include <hip/hip_runtime.h>

namespace hmfsr {

__host__ __device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// a * b for |a|, |b| < 2^23 (window offsets and widths, LDS indices): the
// full-rate 24-bit multiply instead of the quarter-rate 32-bit one.
__device__ __forceinline__ int mul24(int a, int b) { return __mul24(a, b); }

// Row of flat index k in a row-major window of width w, given inv = 1/w
// rounded to float. (k + 1/2) / w lies at least 1/(2w) from an integer while
// the float product errs by under (k / w) * 2^-22, so the floor is exact for
// every k < 2^16.
__device__ __forceinline__ int split_row(int k, float inv) { return (int)(((float)k + 0.5f) * inv); }

// 1/w for split_row: the hardware reciprocal (1 ulp) instead of the correctly
// rounded division's ten instructions. The product then errs by under
// (k / w) * 2^-21, still less than 1/(2w) for every k < 2^16.
__device__ __forceinline__ float window_inv(int w) { return __builtin_amdgcn_rcpf((float)w); }

// Workgroups of a launch are dispatched round-robin over the XCDs, each with
// its own L2. Tile of linear workgroup id b among n: XCD x = b % XCDS takes a
// contiguous run of tiles (row-major), so neighbouring tiles, which share
// footprint halos, meet in the same L2. A bijection on [0, n).
constexpr int XCDS = 8;
__device__ __forceinline__ int xcd_tile(int b, int n) {
  const int q = n / XCDS, r = n - q * XCDS;
  const int x = b % XCDS, l = b / XCDS;
  return x * q + min(x, r) + l;
}

// The same with several runs per XCD, the eight XCDs' runs interleaved: where
// a tile's cost varies over the image (windows that do not fit, borders), no
// XCD keeps the dear part for itself. A bijection on [0, n): the remainder of
// n / (XCDS * RUNS) comes last, in order. The merge kernels take eight runs,
// measured against one in turn: 15 x 3 MP at scale 2 1271 -> 1258 us, 8 x 3 MP
// with a divergent field 357 -> 352, the forward that keeps its normaliser at
// 8 x 768 x 1024 275 -> 269 (scale 2) and 112 -> 109 (scale 1). At 12 MP x 8
// they give 984 -> 982 (31 rounds), inside the spread of single runs, for 317
// -> 353 MB read from HBM; the adjoint takes 671 us either way, 495 -> 492 and
// 374 -> 380 on divergent fields. The streaming merge and the alignment lose
// 0.8 and 1 % with them, their neighbours' data being worth more in one L2.
template <int RUNS>
__host__ __device__ __forceinline__ int xcd_tile_runs(int b, int n) {
  const int len = n / (XCDS * RUNS), x = b % XCDS, k = b / XCDS;
  if (b >= XCDS * RUNS * len) return b;
  const int r = k / len;
  return (r * XCDS + x) * len + k - r * len;
}

// Persistent work distribution over the XCDs. A launch's items [0, n) are
// split into XCDS contiguous chunks of about equal cost (chunk x = [bounds[x],
// bounds[x + 1])), each with its own counter (zero at launch). A workgroup on
// XCD x (dispatch is round-robin) takes the items of chunk x in turn, then
// what is left of the other chunks, x + 1 first, so that neighbouring items
// (tiles of one burst) meet in one L2 and no XCD idles while another has work.
// `slot` is a workgroup-shared int; `body(item)` runs on the whole workgroup.
struct ItemQueue {
  const int* bounds;  // [XCDS + 1]
  int* counters;      // [XCDS]
};

template <typename F>
__device__ __forceinline__ void for_each_item(const ItemQueue& q, int* slot, F&& body) {
  const int home = blockIdx.x % XCDS;
  for (int k = 0; k < XCDS; ++k) {
    const int c = (home + k) % XCDS;
    const int lo = q.bounds[c], hi = q.bounds[c + 1];
    if (lo >= hi) continue;  // uniform
    while (true) {
      __syncthreads();
      if (threadIdx.x == 0) *slot = lo + atomicAdd(&q.counters[c], 1);
      __syncthreads();
      const int it = __builtin_amdgcn_readfirstlane(*slot);  // uniform: scalar loads follow
      if (it >= hi) break;
      body(it);
    }
  }
}

}  // namespace hmfsr
