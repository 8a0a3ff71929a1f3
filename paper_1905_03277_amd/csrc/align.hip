// Tile alignment of a burst against its base frame (Sec. 3.2): a pyramid of
// integer 2x2 sums of the half-resolution luma, coarse-to-fine block matching
// by integer sum of squared differences, and Lucas-Kanade refinement of the
// finest level's vectors.
//
// Every integer step (pyramid, costs, the argmin and its tie rules) is exact,
// and the noise gate that keeps a block at its guess when the winner's gain
// is within the noise (the noise model of Sec. 5.2.2) compares float64 values
// rounded in a fixed order, so the block-matching vectors are fully
// determined by the frames and the descriptor. The
// Lucas-Kanade normal matrix is an exact integer sum as well; its solve and
// the error image run in float64.
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "device_util.h"
#include "hmfsr_internal.h"

namespace hmfsr {
namespace {

constexpr int kPyrEdge = 64;       // level-0 pixels per pyramid workgroup edge
constexpr int kAlignThreads = 256;   // pyramid workgroup

// ---- pyramid ------------------------------------------------------------------
// Workgroup = a 64 x 64 region of level 0 (128 x 128 raw pixels) of one frame;
// level l of the region (64 >> l pixels square) is summed in LDS from level
// l - 1. A level-l pixel inside the level's size has all four children inside
// level l - 1 and inside the same region, since regions are aligned to 64.
__global__ __launch_bounds__(kAlignThreads) void k_align_pyramid(const uint16_t* __restrict__ frames, int H,
                                                                 int W, int32_t* __restrict__ pyr,
                                                                 AlignGeom ag) {
  __shared__ int32_t sa[kPyrEdge * kPyrEdge];
  __shared__ int32_t sb[(kPyrEdge / 2) * (kPyrEdge / 2)];
  const int f = blockIdx.z;
  const uint16_t* fr = frames + (size_t)f * H * W;
  int32_t* P = pyr + f * ag.fstride;
  const int lane = threadIdx.x & 63, wrow = threadIdx.x >> 6;
  const int h0 = ag.lh[0], w0 = ag.lw[0];
  const int X0 = blockIdx.x * kPyrEdge, Y0 = blockIdx.y * kPyrEdge;
  for (int r = wrow; r < kPyrEdge; r += kAlignThreads / 64) {
    const int y = Y0 + r, x = X0 + lane;
    int v = 0;
    if (y < h0 && x < w0) {
      const uint32_t a = *(const uint32_t*)(fr + (size_t)(2 * y) * W + 2 * x);
      const uint32_t b = *(const uint32_t*)(fr + (size_t)(2 * y + 1) * W + 2 * x);
      v = (int)((a & 0xffffu) + (a >> 16) + (b & 0xffffu) + (b >> 16));
      P[ag.loff[0] + (long long)y * w0 + x] = v;
    }
    sa[r * kPyrEdge + lane] = v;
  }
  int32_t* src = sa;
  int32_t* dst = sb;
  int e = kPyrEdge;  // region edge on the source level
  for (int l = 1; l < ag.L; ++l) {
    __syncthreads();  // the source level is complete and the destination is free
    const int ne = e >> 1;
    const int sh = 31 - __clz(ne);
    const int oy = blockIdx.y * ne, ox = blockIdx.x * ne;
    for (int i = threadIdx.x; i < ne * ne; i += kAlignThreads) {
      const int r = i >> sh, c = i & (ne - 1);
      const int* s0 = src + (2 * r) * e + 2 * c;
      const int v = s0[0] + s0[1] + s0[e] + s0[e + 1];
      dst[i] = v;
      const int y = oy + r, x = ox + c;
      if (y < ag.lh[l] && x < ag.lw[l]) P[ag.loff[l] + (long long)y * ag.lw[l] + x] = v;
    }
    int32_t* t = src;
    src = dst;
    dst = t;
    e = ne;
  }
}

// ---- block matching ---------------------------------------------------------------
struct MatchLevel {
  int B, R;                 // block edge, search radius
  int h, w;                 // level size
  int gby, gbx;             // block grid
  long long loff, voff;     // level offset in a frame's pyramid; its vectors in a frame's set
  int parent;               // 1 when the coarser level supplies the guess
  int pB, pgby, pgbx;       // the coarser level's block edge and grid
  long long pvoff;
  int level;                // pyramid level (a pixel sums 4^(level+1) raw values)
  double k12, na, nb, black, rng;  // noise gate: (12 kappa) kappa (0: off) and the noise model
};

// Noise gate of block matching: does a winner that lowers the cost by `gain`
// below the guess's cost move the block? N pixels with integer sum S on a
// level whose pixels sum m raw values. The operations are rounded one by one
// in this order (no contraction), so that every caller takes the same
// decision for the same integers.
__device__ __forceinline__ bool gate_moves(const MatchLevel& ml, int npx, long long S, double g) {
  const double n = (double)npx;
  const double nm = __dmul_rn(n, (double)(1ll << (2 * ml.level + 2)));
  double e = __dsub_rn((double)S, __dmul_rn(nm, ml.black));
  e = fmin(fmax(e, 0.0), __dmul_rn(nm, ml.rng));
  const double u = __dadd_rn(__dmul_rn(__dmul_rn(ml.na, ml.rng), e), __dmul_rn(__dmul_rn(__dmul_rn(nm, ml.nb), ml.rng), ml.rng));
  return __dmul_rn(__dmul_rn(n, g), g) > __dmul_rn(__dmul_rn(ml.k12, u), u);
}

// Persistent launches: kWaves independent waves per workgroup. Wave w of
// workgroup b (XCD-aware order) takes the contiguous item range
// [(4b + w) * chunk, (4b + w + 1) * chunk), so neighbouring items share an L2.
// A wave synchronises only with itself: its LDS region is private.
constexpr int kWaves = 4;
constexpr int kGroupsPerCU = 8;

// Cross-lane visibility of a wave's own LDS writes: the LDS executes one
// wave's operations in order, so only compiler reordering must be fenced.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Raw buffer resource over n 32-bit words (word 3 as for gfx9 raw buffers).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t words_rsrc(const int32_t* p, long long n) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)(n * 4), 0x00020000);
}

__device__ __forceinline__ int32_t ld_word(__amdgpu_buffer_rsrc_t r, int idx) {
  return __builtin_amdgcn_raw_buffer_load_b32(r, idx * 4, 0, 0);
}

// Copy a block's base window (rows x cols from the base frame's buffer
// resource) and its search region (E x E from the frame, per-lane pointer)
// into LDS, by the LPG lanes of its group; all loads of a round before its
// stores.
template <int LPG, int U>
__device__ __forceinline__ void stage_block(int32_t* tpl, int ldt, int rows, int cols, __amdgpu_buffer_rsrc_t rs_base,
                                            int ty0, int tx0, int32_t* reg, int E, const int32_t* img, int ry0,
                                            int rx0, int h, int w, int l) {
  const int ta = rows * cols, tb = E * E;
  const float ia = 1.0f / (float)cols, ib = 1.0f / (float)E;
  for (int i0 = 0; i0 < ta || i0 < tb; i0 += LPG * U) {
    int va[U], vb[U], aa[U], ab[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * LPG + l;
      aa[u] = -1;
      ab[u] = -1;
      va[u] = 0;
      vb[u] = 0;
      if (i < ta) {
        const int r = split_row(i, ia), c = i - r * cols;
        aa[u] = r * ldt + c;
        va[u] = ld_word(rs_base, clampi(ty0 + r, 0, h - 1) * w + clampi(tx0 + c, 0, w - 1));
      }
      if (i < tb) {
        const int r = split_row(i, ib), c = i - r * E;
        ab[u] = i;
        vb[u] = img[clampi(ry0 + r, 0, h - 1) * w + clampi(rx0 + c, 0, w - 1)];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (aa[u] >= 0) tpl[aa[u]] = va[u];
      if (ab[u] >= 0) reg[ab[u]] = vb[u];
    }
  }
}

// Sum of squared differences of one block row of W pixels, every LDS read of
// the row issued before the arithmetic. Values are integers: with float64
// sums below 2^53 (or 64-bit integers) the order does not matter.
template <int W, bool EXACT_F64>
__device__ __forceinline__ void row_ssd(const int32_t* tr, const int32_t* rr, double& acc, unsigned long long& ssd) {
  int tv[W], rv[W];
#pragma unroll
  for (int c = 0; c < W; ++c) {
    tv[c] = tr[c];
    rv[c] = rr[c];
  }
#pragma unroll
  for (int c = 0; c < W; ++c) {
    if (EXACT_F64) {
      const double d = (double)(rv[c] - tv[c]);
      acc = fma(d, d, acc);
    } else {
      const long long d = (long long)(rv[c] - tv[c]);
      ssd += (unsigned long long)(d * d);
    }
  }
}

// Candidate key packed for lane exchanges: cost, then (squared offset from
// the guess) * 2^16 + scan index; the lexicographic minimum wins.
struct PKey {
  unsigned long long ssd;
  int tie;
};

template <int CTRL>
__device__ __forceinline__ PKey dpp_key(const PKey& a) {
  PKey o;
  o.ssd = ((unsigned long long)(unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(a.ssd >> 32), CTRL, 0xF, 0xF,
                                                                      true)
           << 32) |
          (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(a.ssd & 0xffffffffull), CTRL, 0xF, 0xF, true);
  o.tie = __builtin_amdgcn_update_dpp(0, a.tie, CTRL, 0xF, 0xF, true);
  return o;
}

__device__ __forceinline__ void key_min(PKey& a, const PKey& b) {
  if (b.ssd < a.ssd || (b.ssd == a.ssd && b.tie < a.tie)) a = b;
}

// Block matching of one level, four blocks per wave: the 16 lanes of group g
// take block q0 + g of the wave's chunk and split its candidates (lane l takes
// l, l + 16, ...); the group minimum of the keys is then exchanged over DPP
// (row mirror, half mirror, quad permutations: disjoint orbits, so four steps
// cover the 16 lanes). LDS per group: the base block (B x B) and the frame's
// search region ((B + 2R)^2, edge-replicated).
// EXACT_F64: every level value is below 2^22 (levels 0-2 of 16-bit frames), so
// squared differences and their sums stay below 2^53 and float64 adds them
// exactly; coarser levels add in 64-bit integers.
template <bool EXACT_F64>
__global__ __launch_bounds__(256) void k_align_match(const int32_t* __restrict__ pyr, int2* __restrict__ vecs,
                                                     MatchLevel ml, int ref, long long fstride, long long vstride,
                                                     int items, int chunk) {
  constexpr int LPG = 16, GPW = 4;
  extern __shared__ int32_t smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane >> 4, l = lane & 15;
  const int B = ml.B, R = ml.R, E = B + 2 * R, D = 2 * R + 1, K = D * D;
  int32_t* tpl = smem + (wave * GPW + g) * (B * B + E * E);
  int32_t* reg = tpl + B * B;
  const int per = ml.gby * ml.gbx;
  const int gw = xcd_tile(blockIdx.x, gridDim.x) * (blockDim.x >> 6) + wave;
  const int c0 = gw * chunk, c1 = min(items, c0 + chunk);
  const long long lvl_words = (long long)ml.h * ml.w;
  const __amdgpu_buffer_rsrc_t rs_base = words_rsrc(pyr + (long long)ref * fstride + ml.loff, lvl_words);
  for (int q0 = c0; q0 < c1; q0 += GPW) {
    const int item = q0 + g;
    const bool valid = item < c1;
    const int fi = valid ? item / per : 0;
    const int t = valid ? item - fi * per : 0;
    const int by = t / ml.gbx, bx = t - (t / ml.gbx) * ml.gbx;
    const int f = fi < ref ? fi : fi + 1;
    int gx = 0, gy = 0;
    if (valid && ml.parent) {
      const int cy = min(((2 * by + 1) * B) / (4 * ml.pB), ml.pgby - 1);
      const int cx = min(((2 * bx + 1) * B) / (4 * ml.pB), ml.pgbx - 1);
      const int2 pv = vecs[(long long)f * vstride + ml.pvoff + cy * ml.pgbx + cx];
      gx = 2 * pv.x;
      gy = 2 * pv.y;
    }
    const int nby = min(B, ml.h - by * B), nbx = min(B, ml.w - bx * B);
    if (valid)
      stage_block<LPG, 9>(tpl, B, nby, nbx, rs_base, by * B, bx * B, reg, E, pyr + (long long)f * fstride + ml.loff,
                          by * B + gy - R, bx * B + gx - R, ml.h, ml.w, l);
    wave_sync();
    PKey best{~0ull, 0x7fffffff};
    const int kc = R * D + R;  // the candidate at the guess
    unsigned long long ssd_c = 0;
    if (valid) {
      for (int k = l; k < K; k += LPG) {
        const int dyi = k / D, dxi = k - (k / D) * D;
        unsigned long long ssd = 0;
        if (nbx == 4 || nbx == 8 || nbx == 16 || nbx == 32) {  // full-width rows, unrolled
          double acc = 0.0;
          for (int r = 0; r < nby; ++r) {
            const int32_t* tr = tpl + r * B;
            const int32_t* rr = reg + (r + dyi) * E + dxi;
            if (nbx == 8) {
              row_ssd<8, EXACT_F64>(tr, rr, acc, ssd);
            } else if (nbx == 4) {
              row_ssd<4, EXACT_F64>(tr, rr, acc, ssd);
            } else {
              for (int c0 = 0; c0 < nbx; c0 += 8) row_ssd<8, EXACT_F64>(tr + c0, rr + c0, acc, ssd);
            }
          }
          if (EXACT_F64) ssd = (unsigned long long)acc;
        } else if (EXACT_F64) {
          double acc = 0.0;
          for (int r = 0; r < nby; ++r) {
            const int32_t* tr = tpl + r * B;
            const int32_t* rr = reg + (r + dyi) * E + dxi;
            for (int c = 0; c < nbx; ++c) {
              const double d = (double)(rr[c] - tr[c]);
              acc = fma(d, d, acc);
            }
          }
          ssd = (unsigned long long)acc;
        } else {
          for (int r = 0; r < nby; ++r) {
            const int32_t* tr = tpl + r * B;
            const int32_t* rr = reg + (r + dyi) * E + dxi;
            for (int c = 0; c < nbx; ++c) {
              const long long d = (long long)(rr[c] - tr[c]);
              ssd += (unsigned long long)(d * d);
            }
          }
        }
        const int dx = dxi - R, dy = dyi - R;
        if (k == kc) ssd_c = ssd;
        key_min(best, PKey{ssd, ((dx * dx + dy * dy) << 16) | k});
      }
    }
    key_min(best, dpp_key<0x140>(best));
    key_min(best, dpp_key<0x141>(best));
    key_min(best, dpp_key<0x4E>(best));
    key_min(best, dpp_key<0xB1>(best));
    bool keep = false;
    if (ml.k12 > 0.0) {
      // the guess's cost (one lane of the group holds it) and the block's sum
      long long S = 0;
      if (valid)
        for (int r = 0; r < nby; ++r)
          for (int c = l; c < nbx; c += LPG) S += tpl[r * B + c];
      for (int m = 8; m >= 1; m >>= 1) {
        S += __shfl_xor(S, m, LPG);
        ssd_c += __shfl_xor(ssd_c, m, LPG);
      }
      keep = !gate_moves(ml, nby * nbx, S, (double)(ssd_c - best.ssd));
    }
    if (valid && l == 0) {
      const int k = keep ? kc : best.tie & 0xffff;
      const int dyi = k / D, dxi = k - (k / D) * D;
      vecs[(long long)f * vstride + ml.voff + t] = make_int2(gx + dxi - R, gy + dyi - R);
    }
    wave_sync();  // the next blocks restage this wave's LDS
  }
}

// ---- block matching by rows --------------------------------------------------------
// Blocks of 8, 16 or 32 pixels on levels 0-3 with radius 2 or 4 (the defaults
// for every usual tile size). A lane owns an 8-pixel piece of a block row:
// its template piece stays in registers, and for each vertical offset it reads
// the 8 + 2R pixels of the frame that the 2R + 1 horizontal offsets share
// (three or four 16-byte loads) straight from the level, so no index is
// computed and no LDS read per candidate and pixel. The lane's partial sums
// go to LDS, and the block's lanes then add one candidate each over the
// pieces. B = 8: eight blocks per wave, 16: two, 32: one (two pieces a lane).
//
// A piece's sum of eight squared differences stays below 2^53 while a level's
// values are below 2^25 (levels 0-3 of 16-bit frames), so float64 holds it
// exactly; over the block it does below 2^22 (levels 0-2), and WIDE (level 3)
// adds the pieces as 64-bit integers.
//
// Bound by the VALU (25 candidates x 8 pixels x a float64 difference and a
// fused multiply-add per lane and pass, 4.4 cycles each) and, with three waves
// per SIMD (13 KB of LDS a wave), the loads' latency. With a candidate per
// lane and the block and its search region in LDS (two reads, a conversion and
// index arithmetic per candidate and pixel) 12 MP x 8 took 245 us on level 0,
// now 107; 5 x 510 x 766 with 32-pixel tiles took 38 us on the coarsest level
// and 26 on each other one, now 11 and 7.5.
template <int B>
struct RowBlocks {
  static constexpr int PPR = B / 8;                             // pieces per block row
  static constexpr int LPB = B * PPR < 64 ? B * PPR : 64;       // lanes per block
  static constexpr int SEG = B * PPR / LPB;                     // pieces per lane
  static constexpr int BPW = 64 / LPB;                          // blocks per wave
  // Lane of piece q of block b: the wave's blocks side by side within a row,
  // so that lanes next to each other read memory next to each other.
  __host__ __device__ static constexpr int lane_of(int b, int q) {
    return q / PPR * (BPW * PPR) + b * PPR + q % PPR;
  }
  // Place of a lane's partial sum of candidate k: permuted by k, so that lanes
  // adding different candidates read different banks.
  __device__ static int slot(int k, int lane) { return k * 64 + (lane ^ (B == 8 ? (k & 3) << 3 : k & 31)); }
};

// 4 x NV consecutive words at byte offset voff + soff (four-byte aligned).
template <int NV>
__device__ __forceinline__ void ld_words(__amdgpu_buffer_rsrc_t rs, int voff, int soff, int32_t (&v)[4 * NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 16 * i, soff, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) v[4 * i + j] = (int32_t)q[j];
  }
}

// WPP: waves that share one group of blocks (they split the vertical offsets;
// wave 0 then adds the candidates up).
template <int B, int R, bool WIDE, int WPP>
__global__ __launch_bounds__(256) void k_align_match_rows(const int32_t* __restrict__ pyr, int2* __restrict__ vecs,
                                                          MatchLevel ml, int ref, long long fstride,
                                                          long long vstride, int per_frame, int passes) {
  using RB = RowBlocks<B>;
  constexpr int LPB = RB::LPB, SEG = RB::SEG, BPW = RB::BPW, PPR = RB::PPR;
  constexpr int D = 2 * R + 1, K = D * D, NV = (8 + 2 * R) / 4;
  extern __shared__ double part[];  // per pass: [K][64] partial sums
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  double* pw = part + wave / WPP * (K * 64);
  const int dy0 = wave % WPP;
  const int blk = lane / PPR % BPW, lb = lane / (BPW * PPR) * PPR + lane % PPR;  // lane = lane_of(blk, lb)
  const int h = ml.h, w = ml.w, per = ml.gby * ml.gbx;
  const int p = xcd_tile(blockIdx.x, gridDim.x) * ((blockDim.x >> 6) / WPP) + wave / WPP;
  const __amdgpu_buffer_rsrc_t rs_base = words_rsrc(pyr + (long long)ref * fstride + ml.loff, (long long)h * w);
  if (p >= passes) return;  // the waves of a pass share p
  const int fi = p / per_frame, f = fi < ref ? fi : fi + 1;  // one frame per pass: uniform
  const int t0 = (p - fi * per_frame) * BPW + blk;
  const bool valid = t0 < per;
  const int t = valid ? t0 : per - 1;
  const int by = t / ml.gbx, bx = t - by * ml.gbx;
  const __amdgpu_buffer_rsrc_t rs = words_rsrc(pyr + (long long)f * fstride + ml.loff, (long long)h * w);
  int gx = 0, gy = 0;
  if (ml.parent) {
    const int cy = min(((2 * by + 1) * B) / (4 * ml.pB), ml.pgby - 1);
    const int cx = min(((2 * bx + 1) * B) / (4 * ml.pB), ml.pgbx - 1);
    const int2 pv = vecs[(long long)f * vstride + ml.pvoff + cy * ml.pgbx + cx];
    gx = 2 * pv.x;
    gy = 2 * pv.y;
  }
  const int y0 = by * B, x0 = bx * B;
  const int nby = min(B, h - y0), nbx = min(B, w - x0);
  // every block of the wave whole, its search region inside the level: vector
  // loads without clamps
  const bool inside = nby == B && nbx == B && y0 + gy >= R && y0 + gy + B + R <= h && x0 + gx >= R &&
                      x0 + gx + B + R <= w;
  const bool fast = __all(inside);
  // the frame's row under each of the lane's pieces at vertical offset dy
  // (edge-replicated), the base frame's piece, all loads before any use
  int32_t cur[SEG][4 * NV];
  auto load_region = [&](int dy) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < SEG; ++s) {
      const int q = lb + s * LPB, row = y0 + gy - R + q / PPR, col = x0 + gx - R + 8 * (q % PPR);
      if (fast) {
        ld_words<NV>(rs, (row * w + col) * 4, dy * w * 4, cur[s]);
      } else {
        const int yy = clampi(row + dy, 0, h - 1) * w;
#pragma unroll
        for (int c = 0; c < 4 * NV; ++c) cur[s][c] = ld_word(rs, yy + clampi(col + c, 0, w - 1));
      }
    }
  };
  load_region(dy0);
  double tp[SEG][8];
  unsigned in = 0;  // pixels of the piece that lie in the block
  int tsum = 0;
  {
    int32_t tv[SEG][8];
#pragma unroll
    for (int s = 0; s < SEG; ++s) {
      const int q = lb + s * LPB, row = q / PPR, col = 8 * (q % PPR);
      if (fast) {
        ld_words<2>(rs_base, ((y0 + row) * w + x0 + col) * 4, 0, tv[s]);
      } else {
#pragma unroll
        for (int c = 0; c < 8; ++c) tv[s][c] = ld_word(rs_base, min(y0 + row, h - 1) * w + min(x0 + col + c, w - 1));
      }
    }
#pragma unroll
    for (int s = 0; s < SEG; ++s) {
      const int q = lb + s * LPB, row = q / PPR, col = 8 * (q % PPR);
#pragma unroll
      for (int c = 0; c < 8; ++c) {
        const bool ok = row < nby && col + c < nbx;
        in |= (unsigned)ok << (8 * s + c);
        tsum += ok ? tv[s][c] : 0;
        tp[s][c] = (double)tv[s][c];
      }
    }
  }
#pragma unroll 1
  for (int dy = dy0; dy < D; dy += WPP) {
    double rg[SEG][4 * NV];
#pragma unroll
    for (int s = 0; s < SEG; ++s)
#pragma unroll
      for (int c = 0; c < 4 * NV; ++c) rg[s][c] = (double)cur[s][c];
    if (dy + WPP < D) load_region(dy + WPP);  // the next offset's row, under this one's sums
    auto costs = [&](auto masked) __attribute__((always_inline)) {
#pragma unroll
      for (int dx = 0; dx < D; ++dx) {
        double acc = 0.0;
#pragma unroll
        for (int s = 0; s < SEG; ++s)
#pragma unroll
          for (int c = 0; c < 8; ++c) {
            double d = rg[s][dx + c] - tp[s][c];
            if (decltype(masked)::value && !((in >> (8 * s + c)) & 1)) d = 0.0;
            acc = fma(d, d, acc);
          }
        pw[RB::slot(dy * D + dx, lane)] = acc;
      }
    };
    if (fast) costs(std::false_type{});
    else costs(std::true_type{});
  }
  if (WPP > 1) {
    __syncthreads();  // a workgroup is one pass
    if (wave) return;
  } else {
    wave_sync();
  }
  // One candidate per lane of the block: its cost as 64 bits that order as
  // the costs do (a non-negative float64's pattern, or the integer itself).
  PKey best{~0ull, 0x7fffffff};
  constexpr int kc = R * D + R;  // the candidate at the guess
  unsigned long long cost_c = 0;
  for (int k = lb; k < K; k += LPB) {
    unsigned long long cost;
    if (WIDE) {
      cost = 0;
#pragma unroll
      for (int i = 0; i < LPB; ++i) cost += (unsigned long long)pw[RB::slot(k, RB::lane_of(blk, i))];
    } else {
      double sum = 0.0;
#pragma unroll
      for (int i = 0; i < LPB; ++i) sum += pw[RB::slot(k, RB::lane_of(blk, i))];
      cost = (unsigned long long)__double_as_longlong(sum);
    }
    const int dyi = k / D, dxi = k - dyi * D;
    const int dx = dxi - R, dy = dyi - R;
    if (k == kc) cost_c = cost;
    key_min(best, PKey{cost, ((dx * dx + dy * dy) << 16) | k});
  }
  const int from = RB::lane_of(blk, kc % LPB);
  cost_c = ((unsigned long long)(unsigned)__shfl((int)(cost_c >> 32), from, 64) << 32) |
           (unsigned)__shfl((int)(unsigned)(cost_c & 0xffffffffull), from, 64);
  // minimum key and block sum over the block's lanes: every bit of the lane
  // index but those that name the block
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) {
    if (m >= PPR && m < BPW * PPR) continue;
    PKey o;
    o.ssd = ((unsigned long long)(unsigned)__shfl_xor((int)(best.ssd >> 32), m, 64) << 32) |
            (unsigned)__shfl_xor((int)(unsigned)(best.ssd & 0xffffffffull), m, 64);
    o.tie = __shfl_xor(best.tie, m, 64);
    key_min(best, o);
    tsum += __shfl_xor(tsum, m, 64);
  }
  bool keep = false;
  if (ml.k12 > 0.0) {
    const double gain = WIDE ? (double)(cost_c - best.ssd)
                             : __longlong_as_double((long long)cost_c) - __longlong_as_double((long long)best.ssd);
    keep = !gate_moves(ml, nby * nbx, tsum, gain);
  }
  if (valid && lb == 0) {
    const int k = keep ? kc : best.tie & 0xffff;
    const int dyi = k / D, dxi = k - dyi * D;
    vecs[(long long)f * vstride + ml.voff + t] = make_int2(gx + dxi - R, gy + dyi - R);
  }
}

// ---- Lucas-Kanade ----------------------------------------------------------------
struct LkArgs {
  int B, m;         // tile edge on level 0, window margin
  int h, w;         // level-0 size
  int TY, TX;       // tile grid
  int iters;
  int ref;
  long long fstride, vstride, voff0;
};

// Lane exchanges with the partner whose lane index differs in bit BIT (and,
// for BIT <= 3, possibly in lower bits too): bits 5 and 4 through the LDS
// crossbar, bits 3..0 through DPP (row_mirror: i <-> 15 - i, row_half_mirror:
// i <-> 7 - i, quad permutations [2,3,0,1] and [1,0,3,2]; gfx9 encodings).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const unsigned long long u = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u & 0xffffffffull), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

template <int BIT>
__device__ __forceinline__ double partner(double v) {
  if constexpr (BIT == 5) return __shfl_xor(v, 32, 64);
  else if constexpr (BIT == 4) return __shfl_xor(v, 16, 64);
  else if constexpr (BIT == 3) return dpp_move<0x140>(v);
  else if constexpr (BIT == 2) return dpp_move<0x141>(v);
  else if constexpr (BIT == 1) return dpp_move<0x4E>(v);
  else return dpp_move<0xB1>(v);
}

// Halving step: of N values a lane keeps the half its bit BIT selects, added
// to the partner's copy of that half; the partner keeps the other half.
template <int BIT, int N>
__device__ __forceinline__ void halve(const double* in, double* out, int lane) {
  const bool up = (lane >> BIT) & 1;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const double keep = up ? in[i + N / 2] : in[i], send = up ? in[i] : in[i + N / 2];
    out[i] = keep + partner<BIT>(send);
  }
}

// Sums of 24 per-lane values over each group of LPG (16, 32 or 64) lanes, written
// to tbl[0..24) of the group by one lane per value. Each partner step pairs
// lanes of disjoint orbits, so after log2(LPG) steps every sum covers the
// whole group. Every value is an integer below 2^53: the sums are exact in any
// order.
template <int LPG>
__device__ __forceinline__ void group_sum24(const double* v, double* tbl, int lane, bool write) {
  constexpr int TOP = LPG == 16 ? 3 : (LPG == 32 ? 4 : 5);
  double a[12], b[6], c[3];
  halve<TOP, 24>(v, a, lane);
  halve<TOP - 1, 12>(a, b, lane);
  halve<TOP - 2, 6>(b, c, lane);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if constexpr (TOP - 3 >= 2) c[j] += partner<2>(c[j]);
    if constexpr (TOP - 3 >= 1) c[j] += partner<1>(c[j]);
    c[j] += partner<0>(c[j]);
  }
  if (write && (lane & ((1 << (TOP - 2)) - 1)) == 0) {
    const int i0 = 12 * ((lane >> TOP) & 1) + 6 * ((lane >> (TOP - 1)) & 1) + 3 * ((lane >> (TOP - 2)) & 1);
#pragma unroll
    for (int j = 0; j < 3; ++j) tbl[i0 + j] = c[j];
  }
}

// Copy the bordered base window and the frame's bordered patch of one tile
// into LDS, by the LPG lanes of its group (l = lane within the group). Base
// loads go through the base frame's buffer resource, frame loads through a
// per-lane pointer (the groups of a wave may hold different frames).
template <int LPG, int U>
__device__ __forceinline__ void stage_tile(int32_t* SB, int32_t* SM, int SWW, int rows, __amdgpu_buffer_rsrc_t rs_base,
                                           const int32_t* img, int h, int w, int by0, int bx0, int my0, int mx0,
                                           bool base_too, int l) {
  const int total = rows * SWW;
  const float inv = 1.0f / (float)SWW;
  for (int i0 = 0; i0 < total; i0 += LPG * U) {
    int vb[U], vm[U], at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      at[u] = -1;
      vb[u] = 0;
      vm[u] = 0;
      const int i = i0 + u * LPG + l;
      if (i < total) {
        const int r = split_row(i, inv), c = i - r * SWW;
        at[u] = r * SWW + c;
        if (base_too) vb[u] = ld_word(rs_base, clampi(by0 + r, 0, h - 1) * w + clampi(bx0 + c, 0, w - 1));
        vm[u] = img[clampi(my0 + r, 0, h - 1) * w + clampi(mx0 + c, 0, w - 1)];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (at[u] >= 0) {
        if (base_too) SB[at[u]] = vb[u];
        SM[at[u]] = vm[u];
      }
  }
}

// Per-lane partial sums of one tile over the columns l, l + LPG, ... of its
// window, each walked top to bottom with the 3 x 3 frame neighbourhood and
// the base column kept in registers: [0, 9) sum D_x I(o), [9, 18) sum D_y I(o),
// o = (oy + 1) * 3 + ox + 1; with BASE also 18, 19: sum D_x T, sum D_y T and
// 20, 21, 22: sum D_x^2, D_x D_y, D_y^2. Products are below 2^37 and sums below
// 2^49, so float64 keeps them exact.
template <int LPG, bool BASE>
__device__ __forceinline__ void tile_sums(const int32_t* SB, const int32_t* SM, int SWW, int WH, int WW, int l,
                                          double* acc) {
#pragma unroll
  for (int i = 0; i < 24; ++i) acc[i] = 0.0;
  for (int c = l; c < WW; c += LPG) {
    const int32_t* b = SB + c + 1;
    const int32_t* m = SM + c;
    double m0[3], m1[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      m0[k] = (double)m[k];
      m1[k] = (double)m[SWW + k];
    }
    int bu = b[0], bc = b[SWW];
    double m2[3];
    // window row r: the frame rows r .. r + 2 in ra, rb, rc (rc loaded here),
    // the base column's rows r, r + 1 in bu, bc (r + 2 loaded here)
    auto step = [&](int r, const double (&ra)[3], const double (&rb)[3], double (&rc)[3]) {
      const int32_t* mp = m + (r + 2) * SWW;
#pragma unroll
      for (int k = 0; k < 3; ++k) rc[k] = (double)mp[k];
      const int32_t* brow = b + (r + 1) * SWW;
      const int bd = b[(r + 2) * SWW];
      const double dx = (double)(brow[1] - brow[-1]), dy = (double)(bd - bu);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        acc[k] = fma(dx, ra[k], acc[k]);
        acc[3 + k] = fma(dx, rb[k], acc[3 + k]);
        acc[6 + k] = fma(dx, rc[k], acc[6 + k]);
        acc[9 + k] = fma(dy, ra[k], acc[9 + k]);
        acc[12 + k] = fma(dy, rb[k], acc[12 + k]);
        acc[15 + k] = fma(dy, rc[k], acc[15 + k]);
      }
      if (BASE) {
        const double tv = (double)bc;
        acc[18] = fma(dx, tv, acc[18]);
        acc[19] = fma(dy, tv, acc[19]);
        acc[20] = fma(dx, dx, acc[20]);
        acc[21] = fma(dx, dy, acc[21]);
        acc[22] = fma(dy, dy, acc[22]);
      }
      bu = bc;
      bc = bd;
    };
    if constexpr (LPG == 16) {
      // three rows per pass: the three row registers rotate by name, not by
      // copies (the wider groups keep the plain loop, whose registers allow a
      // fourth wave per SIMD)
      int r = 0;
      for (; r + 3 <= WH; r += 3) {
        step(r, m0, m1, m2);
        step(r + 1, m1, m2, m0);
        step(r + 2, m2, m0, m1);
      }
      if (r < WH) step(r++, m0, m1, m2);
      if (r < WH) step(r, m1, m2, m0);
    } else {
      for (int r = 0; r < WH; ++r) {
        step(r, m0, m1, m2);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          m0[k] = m1[k];
          m1[k] = m2[k];
        }
      }
    }
  }
}

// Lucas-Kanade, LPG lanes per (frame, tile): 16 (four tiles per wave) for
// tiles of up to 8 half-res pixels, else 64. The displacement is uniform over
// the tile, so with D = 2 g the integer central differences of the base
// window, the normal equations need only integer correlations:
//   sum_p D(p) e(p) = sum_corners w_c sum_p D(p) I(p + o_c) - sum_p D(p) T(p),
// o_c the four integer corners of the bilinear sample and w_c their weights.
// The correlations at the 3 x 3 integer offsets around a centre (first the
// block-matching vector) serve every iteration whose sample cell stays within
// them; a step that leaves them re-centres that tile and recomputes. LDS per
// group: the bordered base window and frame patch, and the 24 sums.
template <int LPG>
__global__ __launch_bounds__(256) void k_align_lk(const int32_t* __restrict__ pyr, const int2* __restrict__ vecs,
                                                  LkArgs a, float2* __restrict__ motion, int2* __restrict__ bm_out,
                                                  int items, int chunk, int sw) {
  constexpr int GPW = 64 / LPG;  // tiles per wave
  extern __shared__ int32_t smem[];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int g = lane / LPG, l = lane % LPG;
  const int grp_words = 2 * sw * sw + 48;  // two windows, then 24 doubles (sw even keeps them aligned)
  int32_t* SB = smem + (wave * GPW + g) * grp_words;
  int32_t* SM = SB + sw * sw;
  double* tbl = (double*)(SM + sw * sw);
  const int per = a.TY * a.TX;
  const int gw = xcd_tile(blockIdx.x, gridDim.x) * (blockDim.x >> 6) + wave;
  const int c0 = gw * chunk, c1 = min(items, c0 + chunk);
  const long long lvl_words = (long long)a.h * a.w;
  const __amdgpu_buffer_rsrc_t rs_base = words_rsrc(pyr + (long long)a.ref * a.fstride, lvl_words);
  for (int q0 = c0; q0 < c1; q0 += GPW) {
    const int item = q0 + g;
    const int f = item / per;
    const bool valid = item < c1;
    const bool work = valid && f != a.ref;
    const int t = item - f * per;
    const int ty = t / a.TX, tx = t - (t / a.TX) * a.TX;
    const int wy0 = max(0, ty * a.B - a.m), wy1 = min(ty * a.B + a.B + a.m, a.h);
    const int wx0 = max(0, tx * a.B - a.m), wx1 = min(tx * a.B + a.B + a.m, a.w);
    const int WH = wy1 - wy0, WW = wx1 - wx0, SWW = WW + 2;
    const int32_t* img = pyr + (long long)(work ? f : a.ref) * a.fstride;
    int2 bm = make_int2(0, 0);
    if (work) bm = vecs[(long long)f * a.vstride + a.voff0 + t];
    int ccx = bm.x, ccy = bm.y;  // centre of the 3 x 3 correlation offsets
    if (work)
      stage_tile<LPG, LPG == 16 ? 11 : 8>(SB, SM, SWW, WH + 2, rs_base, img, a.h, a.w, wy0 - 1, wx0 - 1,
                                           wy0 - 1 + ccy, wx0 - 1 + ccx, true, l);
    wave_sync();
    double acc[24];
    if (work) tile_sums<LPG, true>(SB, SM, SWW, WH, WW, l, acc);
    else {
#pragma unroll
      for (int i = 0; i < 24; ++i) acc[i] = 0.0;
    }
    group_sum24<LPG>(acc, tbl, lane, true);
    wave_sync();
    const double Hxx = tbl[20], Hxy = tbl[21], Hyy = tbl[22], STx = tbl[18], STy = tbl[19];
    // Singular-window test on the exact sums, rounded step by step as written
    // (no fused multiply-add), so that it is decided identically everywhere.
    const double tr = __dadd_rn(Hxx, Hyy);
    const double det = __dsub_rn(__dmul_rn(Hxx, Hyy), __dmul_rn(Hxy, Hxy));
    const double thr = __dmul_rn(__dmul_rn(1e-9, tr), tr);
    const bool ok = work && tr > 0.0 && det > thr;
    const double k2 = ok ? 2.0 / det : 0.0;  // H and b here are 4x and 2x the half-gradient ones
    double vx = bm.x, vy = bm.y;
    for (int it = 0; it < a.iters; ++it) {
      const double fxf = floor(vx), fyf = floor(vy);
      const bool need = ok && (fxf < ccx - 1 || fxf > ccx || fyf < ccy - 1 || fyf > ccy);
      if (__any(need)) {
        // the sample cell left the correlated offsets: re-centre those tiles
        wave_sync();
        if (need) {
          ccx = (int)fmax(fmin(fxf, 1e9), -1e9);
          ccy = (int)fmax(fmin(fyf, 1e9), -1e9);
          stage_tile<LPG, LPG == 16 ? 11 : 8>(SB, SM, SWW, WH + 2, rs_base, img, a.h, a.w, 0, 0, wy0 - 1 + ccy,
                                               wx0 - 1 + ccx, false, l);
        }
        wave_sync();
        double acc2[24];
        if (need) tile_sums<LPG, false>(SB, SM, SWW, WH, WW, l, acc2);
        else {
#pragma unroll
          for (int i = 0; i < 24; ++i) acc2[i] = 0.0;
        }
        // every lane takes part in the exchanges; only re-centred groups
        // overwrite their table
        group_sum24<LPG>(acc2, tbl, lane, need);
        wave_sync();
      }
      if (ok) {
        const double fx = vx - fxf, fy = vy - fyf;
        const int o00 = ((int)(fyf - ccy) + 1) * 3 + (int)(fxf - ccx) + 1;
        const double w00 = (1.0 - fx) * (1.0 - fy), w01 = fx * (1.0 - fy), w10 = (1.0 - fx) * fy, w11 = fx * fy;
        const double sx = w00 * tbl[o00] + w01 * tbl[o00 + 1] + w10 * tbl[o00 + 3] + w11 * tbl[o00 + 4] - STx;
        const double sy =
            w00 * tbl[9 + o00] + w01 * tbl[9 + o00 + 1] + w10 * tbl[9 + o00 + 3] + w11 * tbl[9 + o00 + 4] - STy;
        vx -= k2 * (Hyy * sx - Hxy * sy);
        vy -= k2 * (Hxx * sy - Hxy * sx);
      }
    }
    if (valid && l == 0) {
      motion[item] = make_float2((float)(2.0 * vx), (float)(2.0 * vy));
      if (bm_out) bm_out[item] = bm;
    }
    wave_sync();  // the next tiles restage this wave's LDS
  }
}

// Lucas-Kanade by columns, for tiles of 8, 16 or 32 half-res pixels (window
// WIN = 16, 32 or 64): WIN lanes per tile, a lane walks down one window column
// and reads the 3 x 3 frame neighbourhood and the base frame's row around it
// straight from the level (one 12-byte load per row and frame, at a per-lane
// offset plus a uniform row offset: no index arithmetic, no LDS copy), two
// rows ahead of the sums. A wave's tiles belong to one frame. Where a window
// or its displaced patch leaves the level, rows and columns are clamped (edge
// replication) and lanes and rows past a clipped window add nothing.
//
// The sums, their order-free exactness and the iterations are those of
// k_align_lk above, which stays for other tile sizes.
//
// Bound by the VALU (23 float64 multiply-adds and six conversions per row) and
// the loads' latency at three waves per SIMD (152 VGPRs). Windows copied to
// LDS by flat index took 2100 VALU instructions per wave and pass of four
// tiles, 381 us at 12 MP x 8 and 28 us at 5 x 510 x 766 (32-pixel tiles); this
// takes 1090, 208 and 21 us (260 at 12 MP x 8 while the base frame had passes
// of its own). Three one-word loads instead of one 12-byte load
// per row, or neighbour columns from the adjacent lanes: 3 and 8 % slower
// alignment; four rows ahead: registers spill (0.48 -> 0.67 ms).
template <int WIN>
__global__ __launch_bounds__(256, 3) void k_align_lk_cols(const int32_t* __restrict__ pyr,
                                                          const int2* __restrict__ vecs, LkArgs a,
                                                          float2* __restrict__ motion, int2* __restrict__ bm_out,
                                                          int n_aligned, int per_frame, int passes, int chunk) {
  constexpr int TPW = 64 / WIN, RC = 2;  // tiles per wave; rows loaded together
  __shared__ double tables[kWaves][TPW * 24];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane / WIN, l = lane % WIN;
  double* tbl = tables[wave] + g * 24;
  const int h = a.h, w = a.w, per = a.TY * a.TX;
  const int gw = xcd_tile(blockIdx.x, gridDim.x) * (blockDim.x >> 6) + wave;
  const int p0 = gw * chunk, p1 = min(passes, p0 + chunk);
  const __amdgpu_buffer_rsrc_t rs_base = words_rsrc(pyr + (long long)a.ref * a.fstride, (long long)h * w);
  // passes run over the aligned frames (over the base frame of a burst of one)
  auto frame_of = [&](int m) { return n_aligned == 0 ? a.ref : m < a.ref ? m : m + 1; };
  // a pass's block-matching vectors are loaded one pass ahead
  auto load_bm = [&](int p) {
    const int m = p / per_frame, t = min((p - m * per_frame) * TPW + g, per - 1);
    return n_aligned == 0 ? make_int2(0, 0) : vecs[(long long)frame_of(m) * a.vstride + a.voff0 + t];
  };
  int2 next_bm = make_int2(0, 0);
  if (p0 < p1) next_bm = load_bm(p0);
  for (int p = p0; p < p1; ++p) {
    const int m = p / per_frame, f = frame_of(m);  // uniform
    const int t0 = (p - m * per_frame) * TPW + g;
    const bool valid = t0 < per;
    const int t = valid ? t0 : per - 1;
    const long long item = (long long)f * per + t;
    const int2 bm = next_bm;
    if (p + 1 < p1) next_bm = load_bm(p + 1);
    if (m == 0 && valid && l == 0) {  // the base frame's vector of the same tile
      const long long base = (long long)a.ref * per + t;
      motion[base] = make_float2(0.f, 0.f);
      if (bm_out) bm_out[base] = make_int2(0, 0);
    }
    if (n_aligned == 0) continue;
    const __amdgpu_buffer_rsrc_t rs = words_rsrc(pyr + (long long)f * a.fstride, (long long)h * w);
    const int ty = t / a.TX, tx = t - ty * a.TX;
    const int wy0 = max(0, ty * a.B - a.m), WH = min(ty * a.B + a.B + a.m, h) - wy0;
    const int wx0 = max(0, tx * a.B - a.m), WW = min(tx * a.B + a.B + a.m, w) - wx0;
    int ccx = bm.x, ccy = bm.y;  // centre of the 3 x 3 correlation offsets
    const bool base_in = WH == WIN && WW == WIN && wy0 >= 1 && wx0 >= 1 && wy0 + WIN < h && wx0 + WIN < w;
    double acc[24];
    // partial sums of this lane's column, as tile_sums states them
    auto sums = [&]() __attribute__((always_inline)) {
      const int my = wy0 - 1 + ccy, mx = wx0 - 1 + ccx;  // the patch's first row and column
      const bool in = base_in && my >= 0 && mx >= 0 && my + WIN + 1 < h && mx + WIN + 1 < w;
      const bool fast = __all(in);
      const int vb = ((wy0 - 1) * w + wx0 - 1 + l) * 4, vm = (my * w + mx + l) * 4;
      int cb[3], cm[3];
      if (!fast) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          cb[k] = clampi(wx0 - 1 + l + k, 0, w - 1);
          cm[k] = clampi(mx + l + k, 0, w - 1);
        }
      }
      // patch and base rows i .. i + N - 1 (0: the row above the window)
      auto rows = [&](int i, auto& m, auto& b) __attribute__((always_inline)) {
        constexpr int N = sizeof(m) / sizeof(m[0]);
        if (fast) {
#pragma unroll
          for (int q = 0; q < N; ++q) {
            const auto u = __builtin_amdgcn_raw_buffer_load_b96(rs, vm, (i + q) * w * 4, 0);
            const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs_base, vb, (i + q) * w * 4, 0);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              m[q][k] = (int)u[k];
              b[q][k] = (int)v[k];
            }
          }
        } else {
#pragma unroll
          for (int q = 0; q < N; ++q) {
            const int ym = clampi(my + i + q, 0, h - 1) * w, yb = clampi(wy0 - 1 + i + q, 0, h - 1) * w;
#pragma unroll
            for (int k = 0; k < 3; ++k) {
              m[q][k] = ld_word(rs, ym + cm[k]);
              b[q][k] = ld_word(rs_base, yb + cb[k]);
            }
          }
        }
      };
#pragma unroll
      for (int i = 0; i < 24; ++i) acc[i] = 0.0;
      int m01[2][3], b01[2][3], mn[RC][3], bn[RC][3];
      rows(0, m01, b01);
      rows(2, mn, bn);
      double ra[3], rb[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        ra[k] = (double)m01[0][k];
        rb[k] = (double)m01[1][k];
      }
      int bu = b01[0][1], bc[3] = {b01[1][0], b01[1][1], b01[1][2]};
#pragma unroll 1
      for (int r0 = 0; r0 < WIN; r0 += 2 * RC) {
        // window rows r0 .. r0 + RC - 1 from mn, bn; the rows after them in flight
        int m2[RC][3], b2[RC][3];
        auto step = [&](int r, const int (&m)[3], const int (&b)[3]) __attribute__((always_inline)) {
          double rc[3];
#pragma unroll
          for (int k = 0; k < 3; ++k) rc[k] = (double)m[k];
          int dxi = bc[2] - bc[0], dyi = b[1] - bu;
          if (!fast && (l >= WW || r >= WH)) dxi = dyi = 0;
          const double dx = (double)dxi, dy = (double)dyi, tv = (double)bc[1];
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            acc[k] = fma(dx, ra[k], acc[k]);
            acc[3 + k] = fma(dx, rb[k], acc[3 + k]);
            acc[6 + k] = fma(dx, rc[k], acc[6 + k]);
            acc[9 + k] = fma(dy, ra[k], acc[9 + k]);
            acc[12 + k] = fma(dy, rb[k], acc[12 + k]);
            acc[15 + k] = fma(dy, rc[k], acc[15 + k]);
          }
          acc[18] = fma(dx, tv, acc[18]);
          acc[19] = fma(dy, tv, acc[19]);
          acc[20] = fma(dx, dx, acc[20]);
          acc[21] = fma(dx, dy, acc[21]);
          acc[22] = fma(dy, dy, acc[22]);
#pragma unroll
          for (int k = 0; k < 3; ++k) {
            ra[k] = rb[k];
            rb[k] = rc[k];
          }
          bu = bc[1];
#pragma unroll
          for (int k = 0; k < 3; ++k) bc[k] = b[k];
        };
        rows(r0 + RC + 2, m2, b2);
#pragma unroll
        for (int q = 0; q < RC; ++q) step(r0 + q, mn[q], bn[q]);
        if (r0 + 2 * RC < WIN) rows(r0 + 2 * RC + 2, mn, bn);
#pragma unroll
        for (int q = 0; q < RC; ++q) step(r0 + RC + q, m2[q], b2[q]);
      }
    };
    double k2 = 0.0;
    bool ok = false;
    double vx = bm.x, vy = bm.y;
#pragma unroll 1
    for (int it = 0; it < a.iters; ++it) {
      const double fxf = floor(vx), fyf = floor(vy);
      // the first sums, or the sample cell left the correlated offsets:
      // re-centre those tiles (the others' sums are formed again and dropped)
      const bool need = it == 0 || (ok && (fxf < ccx - 1 || fxf > ccx || fyf < ccy - 1 || fyf > ccy));
      if (__any(need)) {
        if (need) {
          ccx = (int)fmax(fmin(fxf, 1e9), -1e9);
          ccy = (int)fmax(fmin(fyf, 1e9), -1e9);
        }
        wave_sync();
        sums();
        group_sum24<WIN>(acc, tbl, lane, need);
        wave_sync();
      }
      // (every round of sums writes the same base-frame sums)
      const double Hxx = tbl[20], Hxy = tbl[21], Hyy = tbl[22], STx = tbl[18], STy = tbl[19];
      if (it == 0) {
        // Singular-window test on the exact sums, rounded step by step as
        // written (no fused multiply-add), so that it is decided identically
        // everywhere.
        const double tr = __dadd_rn(Hxx, Hyy);
        const double det = __dsub_rn(__dmul_rn(Hxx, Hyy), __dmul_rn(Hxy, Hxy));
        const double thr = __dmul_rn(__dmul_rn(1e-9, tr), tr);
        ok = valid && tr > 0.0 && det > thr;
        k2 = ok ? 2.0 / det : 0.0;  // H and b here are 4x and 2x the half-gradient ones
      }
      if (ok) {
        const double fx = vx - fxf, fy = vy - fyf;
        const int o00 = ((int)(fyf - ccy) + 1) * 3 + (int)(fxf - ccx) + 1;
        const double w00 = (1.0 - fx) * (1.0 - fy), w01 = fx * (1.0 - fy), w10 = (1.0 - fx) * fy, w11 = fx * fy;
        const double sx = w00 * tbl[o00] + w01 * tbl[o00 + 1] + w10 * tbl[o00 + 3] + w11 * tbl[o00 + 4] - STx;
        const double sy =
            w00 * tbl[9 + o00] + w01 * tbl[9 + o00 + 1] + w10 * tbl[9 + o00 + 3] + w11 * tbl[9 + o00 + 4] - STy;
        vx -= k2 * (Hyy * sx - Hxy * sy);
        vy -= k2 * (Hxx * sy - Hxy * sx);
      }
    }
    if (valid && l == 0) {
      motion[item] = make_float2((float)(2.0 * vx), (float)(2.0 * vy));
      if (bm_out) bm_out[item] = bm;
    }
    wave_sync();  // the next tiles overwrite this wave's tables
  }
}

template <int WIN>
hipError_t lk_cols(const int32_t* pyr, const int2* vecs, const LkArgs& a, int n, int cus, float* motion,
                   int* block_match, hipStream_t stream) {
  constexpr int TPW = 64 / WIN;
  const int per_frame = (a.TY * a.TX + TPW - 1) / TPW;
  // The aligned frames only: as passes of their own, the base frame's left the
  // XCD whose run they were without work (12 MP x 8 alignment 0.485 -> 0.450
  // ms, this kernel at 3 MP x 8 93 -> 82 us).
  const long long passes = (long long)std::max(n - 1, 1) * per_frame;
  // about twelve rounds of the resident waves (three per SIMD), so that runs of
  // tiles with far-apart vectors, whose loads miss the caches, even out (12 MP
  // x 8 alignment with four / six / eight / twelve rounds and one pass per
  // wave: 0.454 / 0.450 / 0.450 / 0.445 / 0.453 ms)
  const long long waves_wanted = (long long)cus * 12 * 12;
  const long long chunk = (passes + waves_wanted - 1) / waves_wanted;
  const int waves = passes >= 4ll * cus ? kWaves : 1;  // few passes spread over more compute units
  const unsigned groups = (unsigned)(((passes + chunk - 1) / chunk + waves - 1) / waves);
  hipLaunchKernelGGL(k_align_lk_cols<WIN>, dim3(groups), dim3(64 * waves), 0, stream, pyr, vecs, a, (float2*)motion,
                     (int2*)block_match, n - 1, per_frame, (int)passes, (int)chunk);
  return hipGetLastError();
}

unsigned cdiv(long long a, long long b) { return (unsigned)((a + b - 1) / b); }

template <int B, int R, bool WIDE>
hipError_t match_rows(const int32_t* pyr, int2* vecs, const MatchLevel& ml, const AlignGeom& ag, int cus,
                      hipStream_t stream) {
  constexpr int K = (2 * R + 1) * (2 * R + 1), BPW = RowBlocks<B>::BPW;
  const int per_frame = (ml.gby * ml.gbx + BPW - 1) / BPW;
  const long long passes = (long long)(ag.n - 1) * per_frame;
  // Radius 2: a wave takes one pass (kept persistent, each wave's share of
  // consecutive passes ran up to twice as long as another's: 12 MP x 8 level 0
  // 129 us instead of 100); four per workgroup where that still fills the
  // device, else one, so that few passes spread over more compute units.
  // Radius 4 is the coarsest level's, which has few blocks: four waves share a
  // pass (one wave each took 16-22 us at 510 x 766 x 5 and at 12 MP x 8).
  constexpr int WPP = R == 2 ? 1 : 4;
  const int waves = WPP > 1 ? WPP : (passes >= 4ll * cus ? 4 : 1), per_group = waves / WPP;
  const unsigned groups = (unsigned)((passes + per_group - 1) / per_group);
  hipLaunchKernelGGL((k_align_match_rows<B, R, WIDE, WPP>), dim3(groups), dim3(64 * waves),
                     (size_t)per_group * K * 64 * 8, stream, pyr, vecs, ml, ag.ref, ag.fstride, ag.vstride, per_frame,
                     (int)passes);
  return hipGetLastError();
}

// Block matching of one level by rows where that form exists (see
// k_align_match_rows); false: the general kernel takes the level. (A level has
// at most 2^28 pixels, so byte offsets are int, and blocks of 8 above level 0.)
bool launch_match_rows(const int32_t* pyr, int2* vecs, const MatchLevel& ml, const AlignGeom& ag, int cus,
                       hipStream_t stream, hipError_t* err) {
  if (ml.level > 3) return false;
  const bool wide = ml.level == 3;
  if (ml.R == 2 && ml.B == 8 && !wide) *err = match_rows<8, 2, false>(pyr, vecs, ml, ag, cus, stream);
  else if (ml.R == 2 && ml.B == 8) *err = match_rows<8, 2, true>(pyr, vecs, ml, ag, cus, stream);
  else if (ml.R == 2 && ml.B == 16) *err = match_rows<16, 2, false>(pyr, vecs, ml, ag, cus, stream);
  else if (ml.R == 2 && ml.B == 32) *err = match_rows<32, 2, false>(pyr, vecs, ml, ag, cus, stream);
  else if (ml.R == 4 && ml.B == 8 && !wide) *err = match_rows<8, 4, false>(pyr, vecs, ml, ag, cus, stream);
  else if (ml.R == 4 && ml.B == 8) *err = match_rows<8, 4, true>(pyr, vecs, ml, ag, cus, stream);
  else return false;
  return true;
}

}  // namespace

size_t align_bytes(const AlignGeom& ag) {
  return (size_t)ag.n * (size_t)ag.fstride * 4 + (size_t)ag.n * (size_t)ag.vstride * 8 + 256;
}

hipError_t launch_align(const AlignGeom& ag, const uint16_t* frames, int H, int W, void* ws, float* motion,
                        int* block_match, hipStream_t stream) {
  int32_t* pyr = (int32_t*)ws;
  size_t vbyte = ((size_t)ag.n * (size_t)ag.fstride * 4 + 255) & ~(size_t)255;
  int2* vecs = (int2*)((char*)ws + vbyte);
  const dim3 pg(cdiv(ag.lw[0], kPyrEdge), cdiv(ag.lh[0], kPyrEdge), ag.n);
  hipLaunchKernelGGL(k_align_pyramid, pg, dim3(kAlignThreads), 0, stream, frames, H, W, pyr, ag);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  int cus = 0, dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    cus = 256;
  if (ag.n > 1) {
    for (int l = ag.L - 1; l >= 0; --l) {
      MatchLevel ml;
      ml.B = ag.blk[l];
      ml.R = l == ag.L - 1 ? ag.radius_coarse : ag.radius_fine;
      ml.h = ag.lh[l];
      ml.w = ag.lw[l];
      ml.gby = ag.gby[l];
      ml.gbx = ag.gbx[l];
      ml.loff = ag.loff[l];
      ml.voff = ag.voff[l];
      ml.parent = l < ag.L - 1;
      ml.pB = ml.parent ? ag.blk[l + 1] : 1;
      ml.pgby = ml.parent ? ag.gby[l + 1] : 1;
      ml.pgbx = ml.parent ? ag.gbx[l + 1] : 1;
      ml.pvoff = ml.parent ? ag.voff[l + 1] : 0;
      ml.level = l;
      ml.k12 = ag.gate_k12;
      ml.na = ag.na;
      ml.nb = ag.nb;
      ml.black = ag.black;
      ml.rng = ag.rng;
      if (launch_match_rows(pyr, vecs, ml, ag, cus, stream, &err)) {
        if (err != hipSuccess) return err;
        continue;
      }
      const int E = ml.B + 2 * ml.R;
      const int waves = ml.B <= 8 ? kWaves : 1;  // keeps LDS within 64 KiB per workgroup
      const size_t lds = (size_t)waves * 4 * (ml.B * ml.B + E * E) * 4;
      const long long items = (long long)(ag.n - 1) * ml.gby * ml.gbx;
      const long long total_waves = std::min<long long>((items + 3) / 4, (long long)cus * kGroupsPerCU * kWaves);
      long long chunk = (items + total_waves - 1) / total_waves;
      chunk = (chunk + 3) / 4 * 4;
      const unsigned groups = (unsigned)(((items + chunk - 1) / chunk + waves - 1) / waves);
      // levels 0-2 of 16-bit frames stay below 2^22 (sums of 4^(l+1) values)
      if (l <= 2)
        hipLaunchKernelGGL(k_align_match<true>, dim3(groups), dim3(64 * waves), lds, stream, pyr, vecs, ml, ag.ref,
                           ag.fstride, ag.vstride, (int)items, (int)chunk);
      else
        hipLaunchKernelGGL(k_align_match<false>, dim3(groups), dim3(64 * waves), lds, stream, pyr, vecs, ml, ag.ref,
                           ag.fstride, ag.vstride, (int)items, (int)chunk);
      if ((err = hipGetLastError()) != hipSuccess) return err;
    }
  }
  LkArgs a;
  a.B = ag.blk[0];
  a.m = a.B / 2;
  a.h = ag.lh[0];
  a.w = ag.lw[0];
  a.TY = ag.gby[0];
  a.TX = ag.gbx[0];
  a.iters = ag.lk_iterations;
  a.ref = ag.ref;
  a.fstride = ag.fstride;
  a.vstride = ag.vstride;
  a.voff0 = ag.voff[0];
  if (a.B == 8) return lk_cols<16>(pyr, vecs, a, ag.n, cus, motion, block_match, stream);
  if (a.B == 16) return lk_cols<32>(pyr, vecs, a, ag.n, cus, motion, block_match, stream);
  if (a.B == 32) return lk_cols<64>(pyr, vecs, a, ag.n, cus, motion, block_match, stream);
  const int sw = ((a.B + 2 * a.m + 2) + 1) & ~1;  // window edge with its border, at most; even
  const long long items = (long long)ag.n * a.TY * a.TX;
  const int lpg = a.B <= 8 ? 16 : 64;
  const int gpw = 64 / lpg;
  const int waves = a.B <= 16 ? kWaves : 1;  // keeps LDS within 64 KiB per workgroup
  const size_t lds = (size_t)waves * gpw * (2 * sw * sw + 48) * 4;
  const long long total_waves =
      std::min<long long>((items + gpw - 1) / gpw, (long long)cus * kGroupsPerCU * kWaves);
  long long chunk = (items + total_waves - 1) / total_waves;
  chunk = (chunk + gpw - 1) / gpw * gpw;
  const unsigned groups = (unsigned)(((items + chunk - 1) / chunk + waves - 1) / waves);
  if (lpg == 16)
    hipLaunchKernelGGL(k_align_lk<16>, dim3(groups), dim3(64 * waves), lds, stream, pyr, vecs, a, (float2*)motion,
                       (int2*)block_match, (int)items, (int)chunk, sw);
  else
    hipLaunchKernelGGL(k_align_lk<64>, dim3(groups), dim3(64 * waves), lds, stream, pyr, vecs, a, (float2*)motion,
                       (int2*)block_match, (int)items, (int)chunk, sw);
  return hipGetLastError();
}

}  // namespace hmfsr
