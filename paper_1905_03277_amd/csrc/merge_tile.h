// The fused output-tile merge body (Sec. 5.1, eq. 1-2 with the kernel
// covariance of Sec. 5.1.2 / S.1 and the robustness of Sec. 5.2), shared by
// the per-burst kernels (merge.hip) and the persistent batched kernels
// (merge_batch.hip), which live in translation units of their own so that
// neither's code generation depends on the other's instantiations.
//
// One workgroup owns a 64 x MH output tile: lane = column, wave w = a band of
// PX rows, so every thread keeps the per-channel accumulators of PX pixels in
// registers for the whole burst (the paper's online merge: memory does not
// grow with the frame count). The displacements of up to FCH frames, and the
// footprint of every alignment tile derived from its displacement and the
// tile's extreme pixel positions, are staged at once; then, for each frame,
// base frame first:
//   1. the raw Bayer footprint (zero outside the frame) and its 2x2-quad sums
//      (luma) go to LDS, quad by quad: a quad is two 32-bit loads, which give
//      four raw floats and the luma value; beside them the tile's R_hat
//      window. The loads were issued before the previous frame's pixels;
//   2. the kernel covariance Omega (float64, edge values repeated outside the
//      grid) is computed over the footprint;
//   3. every pixel interpolates Omega and R_hat bilinearly, inverts Omega in
//      float64, forms the nine exponents and accumulates exp2-weighted raw values per
//      channel against a per-channel reference exponent that is raised only
//      when a frame would exceed it by more than 2^64 (online normalisation).
// If a frame's footprint does not fit the LDS buffers (a strongly divergent
// motion field), every alignment tile of the output tile gets its own
// windows, laid out side by side in as few groups as the buffers allow.
//
// What bounds it: VALU issue and the latency of the steps above at four waves
// per SIMD (128 VGPRs, 40 KB of LDS per workgroup). Measured on this kernel's
// instruction mix, a float32 add, multiply or FMA of registers takes 2.2
// cycles of a SIMD, a float64 or three-operand integer one, a conversion, a
// min/max or an operand from a scalar register 4.3, exp2 8.3 and a float64
// reciprocal 16; so the index and conversion work around a sample cost more
// than its arithmetic. Loading the window by single samples (index, bounds
// and conversion per sample, then a pass over LDS for the quad sums) and
// recomputing a column's position, fractions and offsets for each of its
// pixels took 1.285 ms for the 12 MP x 8 merge; with quads, columns, colours
// from two parities, staged footprints and one barrier fewer per frame (three
// instead of four and a load round trip) 1.009 ms; with Omega free of
// branches, rows addressed from a vector register and the windows first in
// LDS 0.985 ms (15 x 1512 x 2016 at scale 2: 1.642, 1.337, 1.287 ms; 8 x 256 x
// 256: 82.8, 64.3, 62.3 us). Slower, by 1-4 %: Omega's three values
// interleaved per entry, the interior flag as an integer, the staging's
// threads rotated over the waves.
#pragma once

#include <math.h>

#include <type_traits>

#include "device_util.h"
#include "hmfsr_internal.h"
#include "merge_common.h"
#include "omega.h"

namespace hmfsr {
namespace {

constexpr float SLACK = 64.f;   // log2 headroom above the reference exponent

// R_hat window row of a pixel row (its offset in the window) and its weights.
// The gap keeps the two apart: read as one 64-bit word, the batch of twelve
// bursts took 1540 instead of 1521 us, single merges the same.
template <bool EXACT>
struct RowInfo {
  int ya, gap;
  CellWeights<EXACT> y;
};

template <int MH, bool EXACT>
struct MergeSmem {
  using CP = Caps<MH>;
  static constexpr int NV = 2 * CP::VT;  // displacements staged at once (at least two frames')
  // the windows first: their addresses then fit the instructions' offsets
  float2 sRaw[CP::RAW / 2];
  double sOm[3][CP::OM];
  float sLum[CP::LUMA];
  float sRh[CP::RH];
  double sX[MW], sY[MH];
  int sTyRow[MH], sTxCol[MW];
  int sRlo[CP::TY], sRhi[CP::TY], sClo[CP::TX], sChi[CP::TX];
  RowInfo<EXACT> sRow[MH];
  float2 sV[NV];    // displacement per frame slot and alignment tile (slot * ntiles + tile)
  int sBox[FCH][8];  // footprint of the whole tile per frame slot: Bounds, upper ends negated
  Win sWin[CP::VT];    // per alignment tile, when the whole tile's window does not fit
  int sGrp[CP::VT + 1];  // groups of alignment tiles whose windows fit side by side
  int sNGrp;
};

// What a tile keeps besides the output:
//   TILE_PLAIN   nothing;
//   TILE_SAVE    the normaliser of eq. (1), accumulated in float64, for the adjoint;
//   TILE_STREAM  the accumulators themselves, loaded from and stored to a
//                caller's state, so that frames can be added one call at a time.
enum { TILE_PLAIN = 0, TILE_SAVE = 1, TILE_STREAM = 2 };

// Accumulator state of a streaming merge: [9][OH][OW] floats, per channel the
// numerator and denominator of eq. (1) (raw units, scaled by 2^-m) and the
// reference exponent m; `first` is the first frame (loop index) to add.
struct StreamState {
  const float* in;  // nullable: start from empty accumulators
  float* out;
  int first;
};

// One 64 x MH output tile (tile_x, tile_y) of one burst. RB: raw-footprint
// samples a thread loads at once (quads of four; see wide_raw_window). EXACT:
// see exact_weights.
template <int MH, int THREADS, int MODE, int RB, bool EXACT>
__device__ __forceinline__ void merge_tile(const uint16_t* __restrict__ frames,
                                           const float* __restrict__ motion,
                                           const float* __restrict__ rmin, const Geometry& g,
                                           const MergeConsts& mc, float* __restrict__ out,
                                           float* __restrict__ saved, StreamState st, int tile_x,
                                           int tile_y, MergeSmem<MH, EXACT>& sm) {
  constexpr bool SAVE = MODE == TILE_SAVE;
  constexpr int WAVES = THREADS / 64;
  constexpr int PX = MH / WAVES;
  constexpr int QB = RB / 4;  // quads a thread loads at once
  // Rows of one quad load per thread lie close (scale 1.5 and more): a pixel
  // then often shares its Omega corner rows with the row before and keeps
  // their horizontal interpolation (15 x 3 MP at scale 2 1.292 -> 1.270 ms, 10
  // x 384 x 512 at scale 3 159 -> 156 us). The forward that keeps its
  // normaliser would fall from three to two waves per SIMD (180 VGPRs).
  constexpr bool KEEP = RB == 4 && !SAVE;
  static_assert(PX * WAVES == MH, "tile rows must split evenly over the waves");
  static_assert(PX <= 8 && Caps<MH>::TY <= 16, "a row's alignment tile row is kept in four bits");
  using CP = Caps<MH>;
  static_assert(CP::RAW == 4 * CP::LUMA, "the raw window is the luma window's quads");
  using SM = MergeSmem<MH, EXACT>;
  double* sX = sm.sX;
  double* sY = sm.sY;
  int* sTyRow = sm.sTyRow;
  int* sTxCol = sm.sTxCol;
  int* sRlo = sm.sRlo;
  int* sRhi = sm.sRhi;
  int* sClo = sm.sClo;
  int* sChi = sm.sChi;
  RowInfo<EXACT>* sRow = sm.sRow;
  float2* sV = sm.sV;
  const float* sRaw = (const float*)sm.sRaw;
  float* sLum = sm.sLum;
  double(*sOm)[CP::OM] = sm.sOm;
  float* sRh = sm.sRh;
  Win* sWin = sm.sWin;
  int* sGrp = sm.sGrp;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int C0 = tile_x * MW, R0 = tile_y * MH;
  const int ncol = min(MW, g.OW - C0), nrow = min(MH, g.OH - R0);

  // ---- per-tile geometry ------------------------------------------------
  const int C = C0 + lane;
  const bool col_ok = lane < ncol;
  const double X = out_pos(C, g.scale);  // base-frame position of the column
  if (tid < MW) {
    sX[tid] = X;
    sTxCol[tid] = col_ok ? min((int)floor(X) / g.T, g.TX - 1) : 0;
  }
  for (int r = tid; r < MH; r += THREADS) {
    const double Y = out_pos(R0 + r, g.scale);
    sY[r] = Y;
    sTyRow[r] = r < nrow ? min((int)floor(Y) / g.T, g.TY - 1) : 0;
  }
  __syncthreads();
  const int txA = __builtin_amdgcn_readfirstlane(sTxCol[0]), txB = __builtin_amdgcn_readfirstlane(sTxCol[ncol - 1]);
  const int tyA = __builtin_amdgcn_readfirstlane(sTyRow[0]), tyB = __builtin_amdgcn_readfirstlane(sTyRow[nrow - 1]);
  const int ntx = txB - txA + 1, nty = tyB - tyA + 1, ntiles = ntx * nty;
  // first / last pixel row and column of every alignment tile in the output tile
  if (tid < ncol) {
    const int t = sTxCol[tid] - txA;
    if (tid == 0 || sTxCol[tid - 1] != sTxCol[tid]) sClo[t] = tid;
    if (tid == ncol - 1 || sTxCol[tid + 1] != sTxCol[tid]) sChi[t] = tid;
  }
  for (int r = tid; r < nrow; r += THREADS) {
    const int t = sTyRow[r] - tyA;
    if (r == 0 || sTyRow[r - 1] != sTyRow[r]) sRlo[t] = r;
    if (r == nrow - 1 || sTyRow[r + 1] != sTyRow[r]) sRhi[t] = r;
  }
  // R_hat window on the base half-res grid: the bilinear corners of X/2 - 1/2,
  // edge values repeated outside the grid (so that a pixel's corners are
  // always neighbours).
  const int rhc0 = (int)floor(out_pos(C0, g.scale) * 0.5 - 0.5);
  const int rhr0 = (int)floor(out_pos(R0, g.scale) * 0.5 - 0.5);
  const int rhw = (int)floor(out_pos(C0 + ncol - 1, g.scale) * 0.5 - 0.5) + 2 - rhc0;
  const int rhh = (int)floor(out_pos(R0 + nrow - 1, g.scale) * 0.5 - 0.5) + 2 - rhr0;
  for (int r = tid; r < MH; r += THREADS) {
    const double hy = sY[r] * 0.5 - 0.5;
    const double fhy = floor(hy);
    RowInfo<EXACT> ri;
    ri.ya = ((int)fhy - rhr0) * rhw;
    ri.y.set(hy - fhy);
    sRow[r] = ri;
  }
  int rxa;
  CellWeights<EXACT> rx;
  {
    const double hx = X * 0.5 - 0.5;
    const double fhx = floor(hx);
    rxa = (int)fhx - rhc0;
    rx.set(hx - fhx);
  }
  const int txl = sTxCol[lane] - txA;
  // alignment tile row of each of this wave's pixel rows, four bits each
  unsigned typack = 0;
#pragma unroll
  for (int p = 0; p < PX; ++p) {
    const int r = wave * PX + p;
    const int t = __builtin_amdgcn_readfirstlane(sTyRow[r]) - tyA;
    typack |= (unsigned)(r < nrow ? t : 0) << (4 * p);
  }
  // displacements beyond this put every sample outside the frame
  const float vlim = (float)(max(g.W, g.H) + 16);
  // colour of Bayer position (r, c): green where r + c has parity gpar, and
  // the other colour of a row is red where the row has parity rpar
  const int rpar = g.red_pos >> 1, gpar = (rpar ^ g.red_pos ^ 1) & 1;
  // this wave's rows, addressed from a vector register (as scalars they were
  // spilled and read back for every pixel)
  const RowInfo<EXACT>* rowv = sRow + (tid >> 6) * PX;
  const double* yv = sY + (tid >> 6) * PX;

  // ---- accumulators -----------------------------------------------------
  using Acc = typename std::conditional<SAVE, double, float>::type;
  using EF = typename std::conditional<SAVE, double, float>::type;  // exponent arithmetic
  Acc num[PX][3], den[PX][3];
  float M[PX][3];
#pragma unroll
  for (int p = 0; p < PX; ++p)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      num[p][c] = 0;
      den[p][c] = 0;
      M[p][c] = -INFINITY;
    }
  if (MODE == TILE_STREAM && st.in && col_ok) {
    const size_t plane = (size_t)g.OH * g.OW;
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      const int r = wave * PX + p;
      if (r >= nrow) continue;
      const size_t o = (size_t)(R0 + r) * g.OW + C;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        num[p][c] = st.in[o + c * plane];
        den[p][c] = st.in[o + (3 + c) * plane];
        M[p][c] = st.in[o + (6 + c) * plane];
      }
    }
  }

  // The R_hat window's entries of this thread: byte offsets in a frame's map,
  // the same for every frame (entries past the window re-read its last one
  // and are not stored).
  constexpr int RHT = (CP::RH + THREADS - 1) / THREADS;
  int rho_off[RHT];
  {
    const float inv = window_inv(rhw);
    const int nrh = rhw * rhh;
#pragma unroll
    for (int i = 0; i < RHT; ++i) {
      const int k = min(tid + i * THREADS, nrh - 1);
      const int r = split_row(k, inv), c = k - mul24(r, rhw);
      rho_off[i] = (clampi(rhr0 + r, 0, g.h - 1) * g.w + clampi(rhc0 + c, 0, g.w - 1)) * 4;  // below 2^30
    }
  }
  auto frame_of = [&](int fi) { return fi == 0 ? g.ref : (fi <= g.ref ? fi - 1 : fi); };

  // ---- what one frame stages ----------------------------------------------
  struct Frame {
    Win w;
    bool whole;  // the tile's footprint fits the buffers
    bool inner;  // every sample window lies inside the frame
  };
  auto head = [&](int slot) {
    Bounds bd;
    const int* b = sm.sBox[slot];
    bd.jc0 = __builtin_amdgcn_readfirstlane(b[0]);
    bd.jc1 = -__builtin_amdgcn_readfirstlane(b[1]);
    bd.ic0 = __builtin_amdgcn_readfirstlane(b[2]);
    bd.ic1 = -__builtin_amdgcn_readfirstlane(b[3]);
    bd.hj0 = __builtin_amdgcn_readfirstlane(b[4]);
    bd.hj1 = -__builtin_amdgcn_readfirstlane(b[5]);
    bd.hi0 = __builtin_amdgcn_readfirstlane(b[6]);
    bd.hi1 = -__builtin_amdgcn_readfirstlane(b[7]);
    Frame F;
    F.w = make_win(bd, g);
    F.whole = F.w.ow * F.w.oh <= CP::OM && F.w.lw * F.w.lh <= CP::LUMA;
    F.inner = bd.jc0 >= 1 && bd.jc1 <= g.W - 2 && bd.ic0 >= 1 && bd.ic1 <= g.H - 2;
    return F;
  };
  struct Quads {
    uint32_t top[QB], bot[QB];
    float rh[RHT];
  };
  // Quads k0 .. of the whole window in flight: each reads the clamped quad
  // (whose sum is the luma outside the grid); entries past the window re-read
  // its last one and are not stored.
  auto quad_load = [&](const Win& w, const uint16_t* f, int k0, uint32_t (&top)[QB], uint32_t (&bot)[QB]) {
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(f, (size_t)g.H * g.W * 2);
    const float inv = window_inv(w.lw);
    const int nq = w.lw * w.lh;
#pragma unroll
    for (int i = 0; i < QB; ++i) {
      const int k = min(k0 + i * THREADS, nq - 1);
      const int r = split_row(k, inv), c = k - mul24(r, w.lw);
      const int I = min(max(w.lr0 + r, 0), g.h - 1), J = min(max(w.lc0 + c, 0), g.w - 1);
      const int o = (int)((unsigned)I * (unsigned)(4 * g.W)) + 4 * J;  // bytes, below 2^31
      top[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0);
      bot[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, o, 2 * g.W, 0);
    }
  };
  // One quad into the raw window (zero outside the frame) and its sum into
  // the luma window.
  auto quad_put = [&](uint32_t top, uint32_t bot, bool in, int at, int rw2, int lum) {
    const float a0 = (float)(top & 0xffffu), a1 = (float)(top >> 16);
    const float b0 = (float)(bot & 0xffffu), b1 = (float)(bot >> 16);
    sLum[lum] = (a0 + a1) + (b0 + b1);  // exact
    sm.sRaw[at] = in ? make_float2(a0, a1) : make_float2(0.f, 0.f);
    sm.sRaw[at + rw2] = in ? make_float2(b0, b1) : make_float2(0.f, 0.f);
  };
  auto quad_store = [&](const Win& w, int k0, const uint32_t (&top)[QB], const uint32_t (&bot)[QB]) {
    const float inv = window_inv(w.lw);
    const int nq = w.lw * w.lh;
    // uniform: no quad of the window lies outside the grid
    const bool all_in = w.lr0 >= 0 && w.lc0 >= 0 && w.lr0 + w.lh <= g.h && w.lc0 + w.lw <= g.w;
#pragma unroll
    for (int i = 0; i < QB; ++i) {
      const int k = k0 + i * THREADS;
      if (k >= nq) continue;
      const int r = split_row(k, inv), c = k - mul24(r, w.lw);
      bool in = true;
      if (!all_in) in = (unsigned)(w.lr0 + r) < (unsigned)g.h && (unsigned)(w.lc0 + c) < (unsigned)g.w;
      quad_put(top[i], bot[i], in, 2 * k - c, w.lw, k);  // raw rows 2r, 2r + 1 of lw quads each, in pairs
    }
  };
  auto rh_load = [&](int n, float (&rhv)[RHT]) {
    const size_t plane = (size_t)g.h * g.w;
    const __amdgpu_buffer_rsrc_t rs = tile_rsrc(rmin + (size_t)n * plane, plane * 4);
#pragma unroll
    for (int i = 0; i < RHT; ++i) {
      const uint32_t u = __builtin_amdgcn_raw_buffer_load_b32(rs, rho_off[i], 0, 0);
      rhv[i] = __uint_as_float(u);
    }
  };
  auto rh_store = [&](const float (&rhv)[RHT]) {
    const int t = here(tid);
#pragma unroll
    for (int i = 0; i < RHT; ++i)
      if (t + i * THREADS < rhw * rhh) sRh[t + i * THREADS] = rhv[i];
  };
  // Omega at entry (r, c) of window w, stored at flat entry e
  auto omega_at = [&](int e, const Win& w, int r, int c) {
    const int I = min(max(w.or0 + r, 0), g.h - 1), J = min(max(w.oc0 + c, 0), g.w - 1);  // one v_med3 each
    // the window's outer ring repeats the edge quads: no clamps here
    const int base = w.lum + mul24(I - 1 - w.lr0, w.lw) + (J - 1 - w.lc0);
    float l[3][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int bb = 0; bb < 3; ++bb) l[a][bb] = sLum[base + a * w.lw + bb];
    double oxx, oxy, oyy;
    omega_from_quads(l, mc.om, oxx, oxy, oyy);
    sOm[0][e] = oxx;
    sOm[1][e] = oxy;
    sOm[2][e] = oyy;
  };

  // What the pixels of one column in one alignment tile row share.
  struct Column {
    float vy;
    int jc;           // Bayer column of the window centre
    int raw, rw;      // raw index of a window's first sample: raw + row centre * rw
    int om, ow;       // Omega index of a pixel's first corner: om + corner row * ow
    EF dx[3];
    double fx;        // Omega's bilinear fraction
    // Omega at fx along the corner rows hi, hi + 1 of the row before (KEEP)
    int hi;
    double top[3], bot[3];
  };
  auto column = [&](int slot, int tyl, const Win& w, bool inner, Column& cl) __attribute__((always_inline)) {
    const float2 v = sV[mul24(slot, ntiles) + mul24(tyl, ntx) + txl];
    cl.vy = v.y;
    cl.hi = -2;  // no corner row of a pixel that is not skipped (they start at -1)
    const double px = X + (double)v.x;
    const double fjc = floor(px);
    cl.jc = (int)fjc;
    // sample offsets d = q + 1/2 - p; far away where the sample is outside
    // the frame (far enough that its weight is 0, near enough that no product
    // overflows: the row distance dominates)
    const EF fx0 = (EF)(px - fjc);  // exact
#pragma unroll
    for (int j = 0; j < 3; ++j) cl.dx[j] = ((EF)j - (EF)0.5) - fx0;
    if (!inner) {
#pragma unroll
      for (int j = 0; j < 3; ++j)
        if ((unsigned)(cl.jc + j - 1) >= (unsigned)g.W) cl.dx[j] = SAVE ? (EF)FAR_X : (EF)FAR_X32;
    }
    // Omega at p / 2 - 1/2 (bilinear; the window repeats edge values)
    const double hx = px * 0.5 - 0.5;
    const double fhj = floor(hx);
    cl.fx = hx - fhj;
    cl.ow = w.ow;
    cl.rw = w.rw;
    cl.om = w.om + (int)fhj - w.oc0 - mul24(w.or0, w.ow);
    cl.raw = w.raw + cl.jc - 1 - w.rc0 - mul24(w.rr0 + 1, w.rw);
  };

  // R_hat at the thread's pixel row p
  auto rho_at = [&](int p) __attribute__((always_inline)) {
    const RowInfo<EXACT> ri = rowv[p];
    const float* h = sRh + ri.ya + rxa;
    return ri.y.lerp(rx.lerp(h[0], h[1]), rx.lerp(h[rhw], h[rhw + 1]));
  };

  // accumulate: one pixel of column cl
  auto pixel = [&](const int p, const float rho, bool inner, Column& cl)
                   __attribute__((always_inline)) {
    if (!(rho > 0.f)) return;
    const double py = yv[p] + (double)cl.vy;
    const double fic = floor(py);
    const double fry = py - fic;  // exact
    const int ic = (int)fic;
    if (!inner && samples_outside(cl.jc, ic, g)) return;  // no in-frame sample: no term
    const double hy = py * 0.5 - 0.5;
    const double fhi = floor(hy);
    const double fy = hy - fhi;
    const int ow = cl.ow;
    const int ob = mul24((int)fhi, ow) + cl.om;
    double O[3];
    if (!KEEP || cl.hi != (int)fhi) {
      cl.hi = (int)fhi;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const double o00 = sOm[e][ob], o01 = sOm[e][ob + 1];
        const double o10 = sOm[e][ob + ow], o11 = sOm[e][ob + ow + 1];
        cl.top[e] = fma(cl.fx, o01 - o00, o00);
        cl.bot[e] = fma(cl.fx, o11 - o10, o10);
      }
    }
#pragma unroll
    for (int e = 0; e < 3; ++e) O[e] = fma(fy, cl.bot[e] - cl.top[e], cl.top[e]);
    // eq. (2): log2 w = -1/2 log2(e) d^T Omega^-1 d. Omega_bar, its
    // determinant and inverse in float64 (Omega is ill-conditioned,
    // k1/k2 up to ~10^3); the inverse's entries, the offsets and the
    // nine exponents then in EF: float where the normaliser is not
    // kept (the exponents' terms are products of well-scaled values,
    // so each exponent carries a float rounding of its largest term,
    // a relative weight error of ~10^-5 where it matters), float64 in
    // the forward that keeps its normaliser, whose weights the adjoint
    // recomputes in float64 and must reproduce.
    const double sc = NEG_HALF_LOG2E * recip64_1(O[0] * O[2] - O[1] * O[1]);
    const EF qa = (EF)(O[2] * sc), qb2 = (EF)-2 * (EF)(O[1] * sc), qc = (EF)(O[0] * sc);
    EF dy[3];
    {
      const EF fy0 = (EF)fry;
#pragma unroll
      for (int i = 0; i < 3; ++i) dy[i] = ((EF)i - (EF)0.5) - fy0;
    }
    if (!inner) {
#pragma unroll
      for (int i = 0; i < 3; ++i)
        if ((unsigned)(ic + i - 1) >= (unsigned)g.H) dy[i] = SAVE ? (EF)FAR_Y : (EF)FAR_Y32;
    }
    // exponent of sample (i, j): (qa dx[j] + by[i]) dx[j] + cy[i]
    EF cy[3], by[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      by[i] = qb2 * dy[i];
      cy[i] = qc * (dy[i] * dy[i]);
    }
    auto E = [&](int i, int j, EF row) { return fma(fma(qa, cl.dx[j], by[i]), cl.dx[j], row); };
    // Colour groups of the 3x3 window: centre (0), left/right (1), up/down (2), corners (3).
    const bool isG = ((ic ^ cl.jc ^ gpar) & 1) == 0;
    const bool xIsR = ((ic ^ rpar) & 1) == 0;  // group "X" (centre or left/right) is red
    float d[3][3];
    auto exponents = [&]() __attribute__((always_inline)) {
      const float MX = xIsR ? M[p][0] : M[p][2], MY = xIsR ? M[p][2] : M[p][0], MG = M[p][1];
      const EF g0 = (EF)(isG ? MG : MX), g1 = (EF)(isG ? MX : MG);
      const EF g2 = (EF)(isG ? MY : MG), g3 = (EF)(isG ? MG : MY);
      // the group's reference joins the row term
      const EF r1c = cy[1] - g0, r1s = cy[1] - g1;
      const EF r0m = cy[0] - g2, r0c = cy[0] - g3, r2m = cy[2] - g2, r2c = cy[2] - g3;
      d[1][1] = (float)E(1, 1, r1c);
      d[1][0] = (float)E(1, 0, r1s);
      d[1][2] = (float)E(1, 2, r1s);
      d[0][1] = (float)E(0, 1, r0m);
      d[2][1] = (float)E(2, 1, r2m);
      d[0][0] = (float)E(0, 0, r0c);
      d[0][2] = (float)E(0, 2, r0c);
      d[2][0] = (float)E(2, 0, r2c);
      d[2][2] = (float)E(2, 2, r2c);
    };
    exponents();
    const float dmax = fmaxf(fmaxf(fmaxf(d[0][0], d[0][1]), fmaxf(d[0][2], d[1][0])),
                             fmaxf(fmaxf(d[1][1], d[1][2]), fmaxf(fmaxf(d[2][0], d[2][1]), d[2][2])));
    if (dmax > SLACK) {
      // raise the reference of every channel this frame would overflow
      const float m0 = (float)E(1, 1, cy[1]);
      const float m1 = (float)fmax(E(1, 0, cy[1]), E(1, 2, cy[1]));
      const float m2 = (float)fmax(E(0, 1, cy[0]), E(2, 1, cy[2]));
      const float m3 = (float)fmax(fmax(E(0, 0, cy[0]), E(0, 2, cy[0])), fmax(E(2, 0, cy[2]), E(2, 2, cy[2])));
      const float fG = isG ? fmaxf(m0, m3) : fmaxf(m1, m2);
      const float fX = isG ? m1 : m0, fY = isG ? m2 : m3;
      const float fm[3] = {xIsR ? fX : fY, fG, xIsR ? fY : fX};
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        if (fm[c] > M[p][c] + SLACK) {
          const float s = __builtin_amdgcn_exp2f(M[p][c] - fm[c]);
          num[p][c] *= s;
          den[p][c] *= s;
          M[p][c] = fm[c];
        }
      }
      exponents();
    }
    const int rw = cl.rw;
    const float* rp = sRaw + mul24(ic, rw) + cl.raw;
    float wt[3][3], val[3][3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        wt[i][j] = __builtin_amdgcn_exp2f(d[i][j]);
        val[i][j] = rp[i * rw + j];
      }
    const float S0n = wt[1][1] * val[1][1], S0d = wt[1][1];
    const float S1n = fmaf(wt[1][0], val[1][0], wt[1][2] * val[1][2]), S1d = wt[1][0] + wt[1][2];
    const float S2n = fmaf(wt[0][1], val[0][1], wt[2][1] * val[2][1]), S2d = wt[0][1] + wt[2][1];
    const float S3n = fmaf(wt[0][0], val[0][0], wt[0][2] * val[0][2]) +
                      fmaf(wt[2][0], val[2][0], wt[2][2] * val[2][2]);
    const float S3d = (wt[0][0] + wt[0][2]) + (wt[2][0] + wt[2][2]);
    const float Gn = isG ? S0n + S3n : S1n + S2n, Gd = isG ? S0d + S3d : S1d + S2d;
    const float Xn = isG ? S1n : S0n, Xd = isG ? S1d : S0d;
    const float Yn = isG ? S2n : S3n, Yd = isG ? S2d : S3d;
    const Acc ra = rho;
    num[p][0] = fma(ra, (Acc)(xIsR ? Xn : Yn), num[p][0]);
    den[p][0] = fma(ra, (Acc)(xIsR ? Xd : Yd), den[p][0]);
    num[p][1] = fma(ra, (Acc)Gn, num[p][1]);
    den[p][1] = fma(ra, (Acc)Gd, den[p][1]);
    num[p][2] = fma(ra, (Acc)(xIsR ? Yn : Xn), num[p][2]);
    den[p][2] = fma(ra, (Acc)(xIsR ? Yd : Xd), den[p][2]);
  };

  // ---- the frames, base frame first ------------------------------------------
  const int first = MODE == TILE_STREAM ? st.first : 0;
  const int per_chunk = min(FCH, SM::NV / ntiles);
  for (int f0 = first; f0 < g.n; f0 += per_chunk) {
    const int nf = min(per_chunk, g.n - f0);
    // Displacements and footprints of the next nf frames: per frame and
    // alignment tile the clamped displacement, and the tile's footprint
    // (positions are monotonic in X and Y, so the tile's extreme pixels give
    // its extreme window centres), reduced over the output tile.
    for (int k = here(tid); k < nf * 8; k += THREADS) (&sm.sBox[0][0])[k] = 0x7fffffff;
    __syncthreads();
    for (int k = here(tid); k < nf * ntiles; k += THREADS) {
      const int slot = k / ntiles, t = k - slot * ntiles, ky = t / ntx, kx = t - ky * ntx;
      const int n = frame_of(f0 + slot);
      float2 v = make_float2(0.f, 0.f);
      if (n != g.ref) {
        const float* q = motion + (((size_t)n * g.TY + tyA + ky) * g.TX + txA + kx) * 2;
        v = make_float2(q[0], q[1]);
      }
      // clamping keeps non-finite or huge vectors finite and changes no result
      v = make_float2(fminf(fmaxf(v.x, -vlim), vlim), fminf(fmaxf(v.y, -vlim), vlim));
      sV[k] = v;
      const Bounds b = footprint(sX[sClo[kx]] + (double)v.x, sX[sChi[kx]] + (double)v.x,
                                 sY[sRlo[ky]] + (double)v.y, sY[sRhi[ky]] + (double)v.y, g);
      int* red = sm.sBox[slot];
      atomicMin(&red[0], b.jc0); atomicMin(&red[1], -b.jc1);
      atomicMin(&red[2], b.ic0); atomicMin(&red[3], -b.ic1);
      atomicMin(&red[4], b.hj0); atomicMin(&red[5], -b.hj1);
      atomicMin(&red[6], b.hi0); atomicMin(&red[7], -b.hi1);
    }
    __syncthreads();

    // A frame's first loads are issued before the pixels of the frame before
    // it, so that their latency lies under those pixels.
    Quads q;
    auto prefetch = [&](int slot) __attribute__((always_inline)) {
      const int n = frame_of(f0 + slot);
      const Frame nx = head(slot);
      if (n != g.ref) rh_load(n, q.rh);
      if (nx.whole) quad_load(nx.w, frames + n * g.fstride, here(tid), q.top, q.bot);
    };
    prefetch(0);
    for (int slot = 0; slot < nf; ++slot) {
      const int n = frame_of(f0 + slot);
      const bool is_ref = n == g.ref;
      const uint16_t* f = frames + n * g.fstride;
      const Frame F = head(slot);
      if (slot) __syncthreads();  // the previous frame's windows are no longer read
      if (!is_ref) rh_store(q.rh);
      // Windows: the whole tile's footprint in one window when it fits the
      // buffers; otherwise every alignment tile's own window, laid out side by
      // side in groups that fit (one alignment tile always does: its pixels
      // share one displacement, and its footprint stops at the frame's ring,
      // so its windows span at most its own pixels plus the rings; the caps
      // check of the test suite replays this arithmetic for extreme vectors).
      int ngroups = 1;
      if (!F.whole) {
        for (int k = here(tid); k < ntiles; k += THREADS) {
          const int ky = k / ntx, kx = k - ky * ntx;
          const float2 v = sV[slot * ntiles + k];
          sWin[k] = make_win(footprint(sX[sClo[kx]] + (double)v.x, sX[sChi[kx]] + (double)v.x,
                                       sY[sRlo[ky]] + (double)v.y, sY[sRhi[ky]] + (double)v.y, g), g);
        }
        __syncthreads();
        if (tid == 0) {
          int ng = 0, n_lum = 0, n_om = 0;
          sGrp[0] = 0;
          for (int k = 0; k < ntiles; ++k) {
            Win& w = sWin[k];
            const int a_lum = w.lw * w.lh, a_om = w.ow * w.oh;
            if (k > sGrp[ng] && (n_lum + a_lum > CP::LUMA || n_om + a_om > CP::OM)) {
              sGrp[++ng] = k;
              n_lum = n_om = 0;
            }
            w.raw = 4 * n_lum;
            w.lum = n_lum;
            w.om = n_om;
            n_lum += a_lum;
            n_om += a_om;
          }
          sGrp[++ng] = ntiles;
          sm.sNGrp = ng;
        }
        __syncthreads();
        ngroups = __builtin_amdgcn_readfirstlane(sm.sNGrp);
      }
      for (int gi = 0; gi < ngroups; ++gi) {
        if (gi) __syncthreads();  // the previous group's windows are no longer read
        int s0 = 0, s1 = ntiles;
        // stage the raw footprint and the quad sums, then Omega
        if (F.whole) {
          const int t = here(tid);
          quad_store(F.w, t, q.top, q.bot);
          const int nq = F.w.lw * F.w.lh;
          for (int k0 = QB * THREADS; k0 < nq; k0 += QB * THREADS) {
            quad_load(F.w, f, k0 + t, q.top, q.bot);
            quad_store(F.w, k0 + t, q.top, q.bot);
          }
          __syncthreads();
          const float inv = window_inv(F.w.ow);
          for (int k = here(tid); k < F.w.ow * F.w.oh; k += THREADS) {
            const int r = split_row(k, inv);
            omega_at(k, F.w, r, k - mul24(r, F.w.ow));
          }
        } else {
          s0 = __builtin_amdgcn_readfirstlane(sGrp[gi]);
          s1 = __builtin_amdgcn_readfirstlane(sGrp[gi + 1]);
          // window of flat quad (Omega) entry e of this group
          auto find = [&](int e, bool om) -> int {
            int k = s0;
            while (k + 1 < s1 && (om ? sWin[k + 1].om : sWin[k + 1].lum) <= e) ++k;
            return k;
          };
          const __amdgpu_buffer_rsrc_t rs = tile_rsrc(f, (size_t)g.H * g.W * 2);
          const int nq = sWin[s1 - 1].lum + sWin[s1 - 1].lw * sWin[s1 - 1].lh;
          const int no = sWin[s1 - 1].om + sWin[s1 - 1].ow * sWin[s1 - 1].oh;
          for (int e0 = here(tid); e0 < nq; e0 += 2 * THREADS) {
            uint32_t top[2], bot[2];
            int at[2], lw[2];
            bool in[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int e = min(e0 + i * THREADS, nq - 1);
              const Win& w = sWin[find(e, false)];
              const int k = e - w.lum, r = k / w.lw, c = k - mul24(r, w.lw);
              const int I = w.lr0 + r, J = w.lc0 + c;
              in[i] = (unsigned)I < (unsigned)g.h && (unsigned)J < (unsigned)g.w;
              at[i] = 2 * e - c;  // pairs: the window's raw offset is 4 lum
              lw[i] = w.lw;
              const int o = (int)((unsigned)clampi(I, 0, g.h - 1) * (unsigned)(4 * g.W)) + 4 * clampi(J, 0, g.w - 1);
              top[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0);
              bot[i] = __builtin_amdgcn_raw_buffer_load_b32(rs, o, 2 * g.W, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
              if (e0 + i * THREADS < nq) quad_put(top[i], bot[i], in[i], at[i], lw[i], e0 + i * THREADS);
          }
          __syncthreads();
          for (int e = here(tid); e < no; e += THREADS) {
            const Win& w = sWin[find(e, true)];
            const int k = e - w.om, r = k / w.ow;
            omega_at(e, w, r, k - mul24(r, w.ow));
          }
        }
        __syncthreads();
        // the next frame's first loads, under this frame's (last) pixels
        if (gi + 1 == ngroups && slot + 1 < nf) prefetch(slot + 1);
        if (col_ok) {
          const bool inner = F.whole && F.inner;
          // every row's R_hat at once, so that their LDS round trips overlap
          // (15 x 3 MP at scale 2: 1.305 -> 1.295 ms); the forward that keeps
          // its normaliser has no registers to spare for them (1.20 -> 1.26
          // ms for the training burst) and takes them one by one
          float rho[PX];
          if (!SAVE) {
#pragma unroll
            for (int p = 0; p < PX; ++p) rho[p] = is_ref ? 1.f : rho_at(p);
          }
          Column cl;
          int had = -1;
          bool active = true;
#pragma unroll
          for (int p = 0; p < PX; ++p) {
            const int r = wave * PX + p;
            if (r >= nrow) break;
            const int tyl = (int)(typack >> (4 * p)) & 15;
            if (tyl != had) {  // uniform
              if (F.whole) {
                column(slot, tyl, F.w, inner, cl);
              } else {
                const int k = here(mul24(tyl, ntx) + txl);
                active = k >= s0 && k < s1;
                if (active) column(slot, tyl, sWin[k], false, cl);
              }
              had = tyl;
            }
            if (active) pixel(p, SAVE ? (is_ref ? 1.f : rho_at(p)) : rho[p], inner, cl);
          }
        }
      }
    }
    __syncthreads();  // the chunk's displacements and footprints are no longer read
  }

  // eq. (1): normalise and map raw units to [0, 1]
  if (col_ok) {
    const size_t plane = (size_t)g.OH * g.OW;
#pragma unroll
    for (int p = 0; p < PX; ++p) {
      const int r = wave * PX + p;
      if (r >= nrow) continue;
      const size_t o = (size_t)(R0 + r) * g.OW + C;
      if (out) {
#pragma unroll
        for (int c = 0; c < 3; ++c)
          out[o + c * plane] = (float)((num[p][c] / den[p][c] - (Acc)mc.black) * (Acc)mc.inv_range);
      }
      if (SAVE) {  // the normaliser of eq. (1), for the adjoint
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          ((double*)saved)[o + c * plane] = (double)(num[p][c] / den[p][c]);
          saved[o + (6 + c) * plane] = (float)den[p][c];
          saved[o + (9 + c) * plane] = M[p][c];
        }
      }
      if (MODE == TILE_STREAM && st.out) {
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          st.out[o + c * plane] = (float)num[p][c];
          st.out[o + (3 + c) * plane] = (float)den[p][c];
          st.out[o + (6 + c) * plane] = M[p][c];
        }
      }
    }
  }
}

// Minimum resident waves per SIMD (the second launch bound), i.e. the VGPR
// budget: 4 (128 VGPRs) when a thread keeps at most four pixel rows of
// accumulators, 2 (256) otherwise.
template <int MH, int THREADS>
constexpr int waves_per_simd() {
  return (MH / (THREADS / 64) <= 4) ? 4 : 2;
}

// Whether a 64 x MH tile's raw footprint (64/s + 8 by MH/s + 8 samples with
// its rings) exceeds one quad of four samples per thread: then a thread loads
// two quads (eight samples) at once, else one (entries past the window still
// issue a load).
inline bool wide_raw_window(int MH, int THREADS, double scale) {
  return (64.0 / scale + 8.0) * (MH / scale + 8.0) > 4.0 * THREADS;
}

}  // namespace
}  // namespace hmfsr
