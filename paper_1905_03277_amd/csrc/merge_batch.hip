// Persistent batched merge: workgroups of one launch per tile shape and raw
// load batch size pull (burst, tile) items of many bursts from an XCD-chunked
// queue; the tile body is merge_tile.h.
#include "merge_tile.h"

namespace hmfsr {
namespace {

// Persistent form: workgroups pull (burst, tile) items from the XCD-chunked
// queue (for_each_item) until it is exhausted. One launch per tile shape of
// kMergeVariants and raw-load batch size (RB); small outputs take 64 x 16 here,
// the batch's other tiles filling the device. EXACT: some burst of the launch takes exact R_hat weights; the kernel
// then holds both forms of the tile body, and takes each item's. (Both forms in
// every launch spill registers: twelve bursts 1531 -> 1570 us. A launch per
// form ends in one more nearly empty round: three bursts at scales 1, 1.3 and
// 2.2 445 -> 512 us, with both forms in one 448.)
template <int MH, int THREADS, int RB, bool EXACT>
__global__ __launch_bounds__(THREADS, (waves_per_simd<MH, THREADS>())) void k_merge_batch(
    const BurstArgs* __restrict__ bursts, const WorkItem* __restrict__ items, ItemQueue q) {
  __shared__ union {
    MergeSmem<MH, false> plain;
    MergeSmem<MH, EXACT> exact;
  } sm;
  __shared__ int item;
  for_each_item(q, &item, [&](int it) {
    const WorkItem w = items[it];
    const BurstArgs* b = bursts + w.burst;
    const Geometry g = b->g;
    const MergeConsts mc = b->mc;
    const int tx = w.tile % b->merge_tiles_x, ty = w.tile / b->merge_tiles_x;
    const StreamState none{nullptr, nullptr, 0};
    if (EXACT && exact_weights(g.scale))
      merge_tile<MH, THREADS, TILE_PLAIN, RB, EXACT>(b->frames, b->motion, b->rmin, g, mc, b->out, nullptr, none, tx,
                                                     ty, sm.exact);
    else
      merge_tile<MH, THREADS, TILE_PLAIN, RB, false>(b->frames, b->motion, b->rmin, g, mc, b->out, nullptr, none, tx,
                                                     ty, sm.plain);
  });
}

// Calls f(kernel, threads) with the kernel of merge class cls (merge_class).
template <int MH, int THREADS, typename F>
void with_kernel(int cls, bool exact, F f) {
  if (exact) {
    if (cls & 1) f(k_merge_batch<MH, THREADS, 8, true>, THREADS);
    else f(k_merge_batch<MH, THREADS, 4, true>, THREADS);
  } else {
    if (cls & 1) f(k_merge_batch<MH, THREADS, 8, false>, THREADS);
    else f(k_merge_batch<MH, THREADS, 4, false>, THREADS);
  }
}
template <typename F>
void of_class(int cls, bool exact, F f) {
  switch (cls >> 1) {
    case 1: return with_kernel<32, 512>(cls, exact, f);
    case 2: return with_kernel<16, 256>(cls, exact, f);
    case 3: return with_kernel<16, 128>(cls, exact, f);
    default: return with_kernel<32, 256>(cls, exact, f);
  }
}

}  // namespace

hipError_t launch_merge_batch(int cls, bool exact, const BurstArgs* bursts, const WorkItem* items, const int* bounds,
                              int* counters, int n_groups, hipStream_t stream) {
  const ItemQueue q{bounds, counters};
  of_class(cls, exact, [&](auto kernel, int threads) {
    hipLaunchKernelGGL(kernel, dim3(n_groups), dim3(threads), 0, stream, bursts, items, q);
  });
  return hipGetLastError();
}

int merge_batch_blocks_per_cu(int cls, bool exact) {
  int b = 0;
  hipError_t e = hipSuccess;
  of_class(cls, exact, [&](auto kernel, int threads) {
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kernel, threads, 0);
  });
  return e == hipSuccess && b > 0 ? b : 1;
}

}  // namespace hmfsr
