// Per-burst forward merge kernels (one launch over a burst's output tiles),
// the normaliser-keeping forward of the adjoint and the streaming merge; the
// tile body is merge_tile.h.
#include "merge_shape.h"
#include "merge_tile.h"

namespace hmfsr {
namespace {

template <int MH, int THREADS, int RB, bool EXACT>
__global__ __launch_bounds__(THREADS, (waves_per_simd<MH, THREADS>())) void k_merge(
    const uint16_t* __restrict__ frames, const float* __restrict__ motion,
    const float* __restrict__ rmin, Geometry g, MergeConsts mc, float* __restrict__ out) {
  __shared__ MergeSmem<MH, EXACT> sm;
  const int tiles_x = (g.OW + MW - 1) / MW, n = tiles_x * ((g.OH + MH - 1) / MH);
  const int t = xcd_tile_runs<8>(blockIdx.x, n);
  merge_tile<MH, THREADS, TILE_PLAIN, RB, EXACT>(frames, motion, rmin, g, mc, out, nullptr,
                                                 StreamState{nullptr, nullptr, 0}, t % tiles_x, t / tiles_x, sm);
}

// Forward that also keeps the normaliser for the adjoint (float64
// accumulation). Three waves per SIMD, 168 VGPRs; with EXACT, whose second
// weight would take two more, by the launch bound.
template <int MH, int RB, bool EXACT>
__global__ __launch_bounds__(256, EXACT ? 3 : 2) void k_merge_save(
    const uint16_t* __restrict__ frames, const float* __restrict__ motion,
    const float* __restrict__ rmin, Geometry g, MergeConsts mc, float* __restrict__ out,
    float* __restrict__ saved) {
  __shared__ MergeSmem<MH, EXACT> sm;
  const int tiles_x = (g.OW + MW - 1) / MW, n = tiles_x * ((g.OH + MH - 1) / MH);
  const int t = xcd_tile_runs<8>(blockIdx.x, n);
  merge_tile<MH, 256, TILE_SAVE, RB, EXACT>(frames, motion, rmin, g, mc, out, saved, StreamState{nullptr, nullptr, 0},
                                            t % tiles_x, t / tiles_x, sm);
}

// Streaming form: frames from loop index st.first on are added to the state.
template <int MH, int RB, bool EXACT>
__global__ __launch_bounds__(256, 4) void k_merge_stream(
    const uint16_t* __restrict__ frames, const float* __restrict__ motion,
    const float* __restrict__ rmin, Geometry g, MergeConsts mc, StreamState st) {
  __shared__ MergeSmem<MH, EXACT> sm;
  const int tiles_x = (g.OW + MW - 1) / MW, n = tiles_x * ((g.OH + MH - 1) / MH);
  const int t = xcd_tile(blockIdx.x, n);
  merge_tile<MH, 256, TILE_STREAM, RB, EXACT>(frames, motion, rmin, g, mc, nullptr, nullptr, st, t % tiles_x,
                                              t / tiles_x, sm);
}

// eq. (1) on a streaming state: C = num / den per channel, mapped to [0, 1].
__global__ void k_stream_finish(const float* __restrict__ state, size_t plane, float black, float inv_range,
                                float* __restrict__ out) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= plane) return;
#pragma unroll
  for (int c = 0; c < 3; ++c)
    out[i + c * plane] = (state[i + c * plane] / state[i + (3 + c) * plane] - black) * inv_range;
}

dim3 tile_grid(const Geometry& g, int rows) { return dim3(((g.OW + MW - 1) / MW) * ((g.OH + rows - 1) / rows)); }

// Calls launch(RB, EXACT), two compile-time constants, with the raw-load batch
// size and the weights' form that a tile shape takes at the burst's scale.
template <typename F>
hipError_t with_form(const Geometry& g, int rows, int threads, F launch) {
  using W = std::integral_constant<int, 8>;
  using N = std::integral_constant<int, 4>;
  const bool wide = wide_raw_window(rows, threads, g.scale);
  if (exact_weights(g.scale)) {
    if (wide) launch(W{}, std::true_type{});
    else launch(N{}, std::true_type{});
  } else {
    if (wide) launch(W{}, std::false_type{});
    else launch(N{}, std::false_type{});
  }
  return hipGetLastError();
}

template <int MH, int THREADS>
hipError_t launch_variant(const Geometry& g, const MergeConsts& mc, const uint16_t* frames,
                          const float* motion, const float* rmin, float* out, hipStream_t stream) {
  return with_form(g, MH, THREADS, [&](auto rb, auto exact) {
    hipLaunchKernelGGL((k_merge<MH, THREADS, decltype(rb)::value, decltype(exact)::value>), tile_grid(g, MH),
                       dim3(THREADS), 0, stream, frames, motion, rmin, g, mc, out);
  });
}

template <int MH>
hipError_t launch_save(const Geometry& g, const MergeConsts& mc, const uint16_t* frames, const float* motion,
                       const float* rmin, float* out, float* saved, hipStream_t stream) {
  return with_form(g, MH, 256, [&](auto rb, auto exact) {
    hipLaunchKernelGGL((k_merge_save<MH, decltype(rb)::value, decltype(exact)::value>), tile_grid(g, MH), dim3(256), 0,
                       stream, frames, motion, rmin, g, mc, out, saved);
  });
}

template <int MH>
hipError_t launch_stream(const Geometry& g, const MergeConsts& mc, const uint16_t* frames, const float* motion,
                         const float* rmin, StreamState st, hipStream_t stream) {
  return with_form(g, MH, 256, [&](auto rb, auto exact) {
    hipLaunchKernelGGL((k_merge_stream<MH, decltype(rb)::value, decltype(exact)::value>), tile_grid(g, MH), dim3(256),
                       0, stream, frames, motion, rmin, g, mc, st);
  });
}

}  // namespace

const MergeVariant kMergeVariants[] = {
    {"64x32/256", 32, 256}, {"64x32/512", 32, 512}, {"64x16/256", 16, 256}, {"64x16/128", 16, 128},
};
const int kNumMergeVariants = sizeof(kMergeVariants) / sizeof(kMergeVariants[0]);

hipError_t launch_merge(int shape, const Geometry& g, const MergeConsts& mc, const uint16_t* frames,
                        const float* motion, const float* rmin, float* out, float* saved,
                        hipStream_t stream) {
  if (saved) switch (default_shape(tiles_64x16(g.OH, g.OW))) {  // 64 columns, 256 threads keep the normaliser
      case kShape64x4: return launch_save<4>(g, mc, frames, motion, rmin, out, saved, stream);
      case kShape64x8: return launch_save<8>(g, mc, frames, motion, rmin, out, saved, stream);
      default: return launch_save<16>(g, mc, frames, motion, rmin, out, saved, stream);
    }
  switch (shape) {
    case 1: return launch_variant<32, 512>(g, mc, frames, motion, rmin, out, stream);
    case 2: return launch_variant<16, 256>(g, mc, frames, motion, rmin, out, stream);
    case 3: return launch_variant<16, 128>(g, mc, frames, motion, rmin, out, stream);
    case kShape64x8: return launch_variant<8, 256>(g, mc, frames, motion, rmin, out, stream);
    case kShape64x4: return launch_variant<4, 256>(g, mc, frames, motion, rmin, out, stream);
    default: return launch_variant<32, 256>(g, mc, frames, motion, rmin, out, stream);
  }
}

int merge_class(int variant, double scale) {
  return 2 * variant + (wide_raw_window(kMergeVariants[variant].rows, kMergeVariants[variant].threads, scale) ? 1 : 0);
}

int merge_tile_rows(int variant) { return kMergeVariants[variant].rows; }

hipError_t launch_merge_stream(const Geometry& g, const MergeConsts& mc, const uint16_t* frames,
                               const float* motion, const float* rmin, const float* state_in, float* state_out,
                               int first, hipStream_t stream) {
  const StreamState st{state_in, state_out, first};
  switch (default_shape(tiles_64x16(g.OH, g.OW))) {
    case kShape64x4: return launch_stream<4>(g, mc, frames, motion, rmin, st, stream);
    case kShape64x8: return launch_stream<8>(g, mc, frames, motion, rmin, st, stream);
    default: return launch_stream<16>(g, mc, frames, motion, rmin, st, stream);
  }
}

hipError_t launch_stream_finish(const Geometry& g, const MergeConsts& mc, const float* state, float* out,
                                hipStream_t stream) {
  const size_t plane = (size_t)g.OH * g.OW;
  hipLaunchKernelGGL(k_stream_finish, dim3((unsigned)((plane + 255) / 256)), dim3(256), 0, stream, state, plane,
                     mc.black, mc.inv_range, out);
  return hipGetLastError();
}

}  // namespace hmfsr
