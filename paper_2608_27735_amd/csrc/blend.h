// blend.h -- pieces shared by the forward and backward tile blend kernels:
// the launch constants, the tile schedule lookup, list-entry loads, the
// tile's pixel-centre box and the block-wide compaction of staged entries.
//
// One 256-thread workgroup (4 wave64) per 16x16 tile, one thread per pixel.
// Gaussians of the tile's depth-sorted list are staged through LDS in batches
// of 256; an entry is kept only if its alpha >= alpha_min ellipse reaches the
// tile's pixel-centre box.
#pragma once

#include "abcd_internal.h"

namespace abcd {
namespace {


struct BlendConsts {
  int width, height, ntx, ntiles, per_xcd;
  float alpha_min, alpha_max, t_min;
};

// Tile of this workgroup: the given schedule (heaviest tiles first), or, with
// none, raster order with each of the 8 XCDs (which take workgroups round
// robin) given a contiguous band of tiles, so that neighbouring tiles (which
// share Gaussians) share an L2.
__device__ __forceinline__ int tile_of_block(const BlendConsts& k, const uint32_t* order) {
  const int b = blockIdx.x;
  if (order) return (int)order[b];
  return (b & 7) * k.per_xcd + (b >> 3);
}

// One list entry as loaded from global memory by one thread.
struct Rec {
  float2 m;
  float4 co;
  float r, g, b;
  uint32_t gid;
  bool valid;
};

// The gathers of one entry, for a Gaussian index read earlier. The loads are
// unconditional (an invalid entry reads a valid index, see the callers):
// loads under a divergent branch would make the compiler wait for them at the
// branch's end instead of where the values are first used, which serialised
// the staging of every batch.
__device__ __forceinline__ Rec gather_rec(uint32_t gid, bool valid,
                                          const float2* __restrict__ means2d,
                                          const float4* __restrict__ conic_opacity,
                                          const float* __restrict__ rgb) {
  Rec r;
  r.valid = valid;
  r.gid = gid;
  r.m = means2d[gid];
  r.co = conic_opacity[gid];
  r.r = rgb[3 * gid];
  r.g = rgb[3 * gid + 1];
  r.b = rgb[3 * gid + 2];
  return r;
}

// Pixel-centre box of a tile, clipped to the image.
struct TileBox {
  float x0, x1, y0, y1;
};

__device__ __forceinline__ TileBox tile_box(const BlendConsts& k, int tile) {
  const int tx = tile % k.ntx, ty = tile / k.ntx;
  TileBox b;
  b.x0 = (float)(tx * kTile) + 0.5f;
  b.y0 = (float)(ty * kTile) + 0.5f;
  b.x1 = (float)(min(tx * kTile + kTile, k.width) - 1) + 0.5f;
  b.y1 = (float)(min(ty * kTile + kTile, k.height) - 1) + 0.5f;
  return b;
}

// The general kernels give each wave an 8x8 quadrant of the tile (wave w the
// columns 8 (w & 1) .., rows 8 (w >> 1) ..), lane l pixel (l & 7, l >> 3) of it: a
// splat of radius r meets a square of 64 pixels less often than a strip of
// 16x4 ((8 + 2r)^2 against (16 + 2r)(4 + 2r)). Forward, 16x4 strips -> quadrants:
// 1M Gaussians at 1297x840 151 -> 141 us, 300K 138 -> 129, 4M tiny ones at
// 2560x1440 390 -> 287 (the strips of its longest walks split worse than its
// average), the 64K ring scene at 512x512 87 -> 77.
__device__ __forceinline__ int quad_x(int tid) { return 8 * ((tid >> 6) & 1) + (tid & 7); }
__device__ __forceinline__ int quad_y(int tid) { return 8 * (tid >> 7) + ((tid >> 3) & 7); }

// Box (x0, x1, y0, y1) of the centres of the wave's pixels that can still blend,
// from the lanes' flags; out of every splat's reach when none can. Uniform. At
// the rim of a dense cluster a few pixels walk lists of 100,000 entries whose
// splats lie where all others have stopped: tested against the whole quadrant,
// nearly all of them were walked. Forward / backward in us, quadrant -> box:
// 900K tiny Gaussians on 161x141 9,989 / 20,184 -> 4,625 / 5,031, 857K on 161x141
// 3,220 / 10,564 -> 1,765 / 1,588, 30K on 80x60 544 / 1,224 -> 261 / 538, 300K on
// 400x300 359 / 106 -> 260 / 106. On large frames it pays for itself (1M block
// step 912 -> 901, 300K 530 -> 519, 4M at 2560x1440 1,787 -> 1,714).
__device__ __forceinline__ float4 live_box(const BlendConsts& k, int tile, bool live) {
  const uint64_t m = __ballot(live);
  if (m == 0ull) return make_float4(1e18f, 1e18f, 1e18f, 1e18f);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int x = (tile % k.ntx) * kTile + 8 * (w & 1), y = (tile / k.ntx) * kTile + 8 * (w >> 1);
  uint32_t cols = (uint32_t)m | (uint32_t)(m >> 32);
  cols |= cols >> 16;
  cols = (cols | (cols >> 8)) & 255u;
  return make_float4((float)(x + __builtin_ctz(cols)) + 0.5f, (float)(x + 31 - __builtin_clz(cols)) + 0.5f,
                     (float)(y + (__builtin_ctzll(m) >> 3)) + 0.5f,
                     (float)(y + ((63 - __builtin_clzll(m)) >> 3)) + 0.5f);
}

// Tile test and quadrants mask of an entry in one: bit w set when some point of
// box[w] (live_box of wave w) can see the Gaussian with alpha >= alpha_min, i.e.
// d^T Q d <= tau = 2 ln(o / alpha_min), Q = [[a, b], [b, c]]; 0: the entry is
// dropped. With the columns fixed, the minimum of the convex quadratic over dx
// is a convex function of dy whose minimiser y* is 0 when the mean's column
// lies among them, else -b dx_e / c on the nearer edge dx_e; the minimum over
// the box is at y* clamped to its rows, with dx = -b dy / a clamped to its
// columns. The margin keeps every entry whose per-pixel decision could go
// either way in fp32 (no pixel that blends is ever dropped, so the outputs do
// not depend on this test); it also covers the 1 ulp reciprocals, which move the
// minimiser and so the minimum in second order only.
__device__ __forceinline__ uint32_t splat_quads(float2 m, float4 co, float alpha_min,
                                                const float4 (&box)[4]) {
  if (!(co.w >= alpha_min)) return 0u;
  const float tau = 2.0f * (__logf(co.w) - __logf(alpha_min));
  const float lim = tau * 1.001f + 1e-3f;
  const float c = co.y * co.y + co.z * co.z;
  const float mia = co.x > 0.0f ? -co.y * __builtin_amdgcn_rcpf(co.x) : 0.0f;
  const float mic = c > 0.0f ? -co.x * co.y * __builtin_amdgcn_rcpf(c) : 0.0f;
  uint32_t quads = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float4 q4 = box[w];
    const float dx0 = q4.x - m.x, dx1 = q4.y - m.x;
    const float ys = mic * __builtin_amdgcn_fmed3f(0.0f, dx0, dx1);
    const float dy = __builtin_amdgcn_fmed3f(ys, q4.z - m.y, q4.w - m.y);
    const float dx = __builtin_amdgcn_fmed3f(mia * dy, dx0, dx1);
    const float e1 = co.x * dx + co.y * dy, e2 = co.z * dy;
    if (e1 * e1 + e2 * e2 <= lim) quads |= 1u << w;
  }
  return quads;
}

// The same test for single pixel rows of the tile: bit w set when pixel row row0 + w of
// the tile (clipped to the image) can see the Gaussian. With the row fixed,
// the minimum over the columns is at dx = -b dy / a clamped to the columns.
__device__ __forceinline__ uint32_t splat_rows_single(float u, float v, float a, float b, float c,
                                                      float o, float alpha_min, const TileBox& box,
                                                      int row0) {
  if (!(o >= alpha_min)) return 0u;
  const float tau = 2.0f * (__logf(o) - __logf(alpha_min));
  const float lim = tau * 1.001f + 1e-3f;
  const float ia = a > 0.0f ? 1.0f / a : 0.0f;
  const float dx0 = box.x0 - u, dx1 = box.x1 - u;
  uint32_t rows = 0;
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float yb = box.y0 + (float)(row0 + w);
    const float dy = yb - v;
    const float dx = fminf(fmaxf(-b * dy * ia, dx0), dx1);
    const float q = a * dx * dx + 2.0f * b * dx * dy + c * dy * dy;
    if (yb <= box.y1 && q <= lim) rows |= 1u << w;
  }
  return rows;
}

// Block-wide compaction of the staged entries into slots `pos` and, for
// each wave w, the list of the staged slots whose rows mask has bit w, in
// list order, into s_idx[w]. s_cnt holds 5 x 4 wave counts. Returns the
// number kept; wcnt is the length of the calling wave's list (both uniform).
__device__ __forceinline__ int compact_rows(bool keep, uint32_t rows, int (*s_cnt)[4],
                                            uint8_t (*s_idx)[256], int& pos, int& wcnt) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const uint64_t below = (1ull << l) - 1ull;
  const uint64_t bal = __ballot(keep);
  uint64_t rb[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) rb[r] = __ballot((rows >> r) & 1u);
  if (l == 0) {
    s_cnt[0][w] = __popcll(bal);
#pragma unroll
    for (int r = 0; r < 4; ++r) s_cnt[1 + r][w] = __popcll(rb[r]);
  }
  __syncthreads();
  int off = 0, tot = 0, mine = 0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int c = s_cnt[0][v];
    off += v < w ? c : 0;
    tot += c;
    mine += s_cnt[1 + w][v];
  }
  pos = off + __popcll(bal & below);
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if ((rows >> r) & 1u) {
      int o = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) o += v < w ? s_cnt[1 + r][v] : 0;
      s_idx[r][o + __popcll(rb[r] & below)] = (uint8_t)pos;
    }
  }
  wcnt = __builtin_amdgcn_readfirstlane(mine);
  return __builtin_amdgcn_readfirstlane(tot);
}

// The same for kernels whose waves each walk a contiguous copy of their own
// list: at[r] is this thread's slot in the list of quadrant r (valid where bit r
// of quads is set), wcnt the length of the calling wave's list; returns the
// number of entries with any bit set (wcnt and the result are uniform). s_cnt
// holds 5 x 4 wave counts.
__device__ __forceinline__ int quad_slots(uint32_t quads, int (*s_cnt)[4], int (&at)[4], int& wcnt) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const uint64_t below = (1ull << l) - 1ull;
  const uint64_t bal = __ballot(quads != 0u);
  uint64_t rb[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) rb[r] = __ballot((quads >> r) & 1u);
  if (l == 0) {
    s_cnt[0][w] = __popcll(bal);
#pragma unroll
    for (int r = 0; r < 4; ++r) s_cnt[1 + r][w] = __popcll(rb[r]);
  }
  __syncthreads();
  int tot = 0, mine = 0;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    tot += s_cnt[0][v];
    mine += s_cnt[1 + w][v];
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    int o = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) o += v < w ? s_cnt[1 + r][v] : 0;
    at[r] = o + __popcll(rb[r] & below);
  }
  wcnt = __builtin_amdgcn_readfirstlane(mine);
  return __builtin_amdgcn_readfirstlane(tot);
}

// Frames of at most this many tiles (without a split) take the forward and
// backward kernels that give each tile four workgroups, one pixel row per
// wave and four list entries per step of a wave.
constexpr int kRowsTiles = 256;

// In frames of at most kFewTiles tiles (without a split) whose lists hold at most
// kFewPairs (tile, Gaussian) pairs, the backward takes a list of at least
// kRowsList entries in the same layout and a shorter one whole. Only the GPU
// knows the lists: a workgroup for each whole tile and four for its rows are
// launched, and those that the tile's list has no use for return. With so few
// pairs the whole chip would blend them in 10 us and the longest list sets the
// launch's length. Each limit with both sides measured, in us, on 1,024 tiles:
//   whole / rows: 1,024 Gaussians, longest list 722: 65 / 42; 8,000 over 146 tiles,
//   longest 1,263: 62 / 53; on 361 tiles 8,000, longest 2,707: 160 / 79;
//   lists from 96 / 128 / 192 on in rows: 2,000 over 976 tiles, longest 186: 46 /
//   42 / 35 (whole 35); 512 on 272 tiles, longest 222: 19 / 23 / 27 (whole 38),
//   longest 444: 35 / 35 / 35 (whole 68). All lists in rows cost frames with many
//   short ones: 1,024 over 675 tiles, longest 29, 15 -> 24.
// The pairs' limit: 53,380 over 976 tiles are the worst below it (35 whole, 42
// with rows); above, 77,052 pairs over 101 tiles would gain (113 / 86), 218,946
// over 999 and 320,460 over 1,019 lose (55 / 76, 56 / 81).
// The forward keeps one workgroup per tile in such frames: the rows layout
// brought a few us where the lists are long (1,024 Gaussians over 149 of 1,024
// tiles 31 -> 26) and cost 12 to 28 where they are spread out (over 864 of 1,024
// tiles 20 -> 48, 8,192 Gaussians over 769 20 -> 43), and its outputs would no
// longer be the split forward's bit by bit.
constexpr int kFewTiles = 1024;
constexpr uint32_t kFewPairs = 65536;
constexpr uint32_t kRowsList = 128;

// Lane-bit-4 and lane-bit-5 exchanges. v_permlane16_swap of (x, x) leaves
// rows (0, 0, 2, 2) of x in its first result and rows (1, 1, 3, 3) in its
// second; v_permlane32_swap of (x, x) leaves halves (low, low) and (high,
// high). Either way the two results combined give the pair's total with the
// same operands in the same order on both partners, and a lane with the
// exchanged bit set finds its partner's value in the first result.
struct Swapped {
  float first, second;
};
__device__ __forceinline__ Swapped swap_bit4(float x) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(x), __float_as_int(x), false, false);
  return Swapped{__int_as_float(p[0]), __int_as_float(p[1])};
}
__device__ __forceinline__ Swapped swap_bit5(float x) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(x), __float_as_int(x), false, false);
  return Swapped{__int_as_float(p[0]), __int_as_float(p[1])};
}

constexpr int kGroup = 4;  // the forward's group (six spilled four registers)
constexpr int kBwdGroup = 4;  // the backward's group (register budget: 5 waves per SIMD)

BlendConsts consts(const abcd_camera& cam, const abcd_raster_params& prm) {
  BlendConsts k;
  k.width = cam.width;
  k.height = cam.height;
  k.ntx = tiles_x(cam.width);
  k.ntiles = k.ntx * tiles_y(cam.height);
  k.per_xcd = (k.ntiles + 7) / 8;
  k.alpha_min = prm.alpha_min;
  k.alpha_max = prm.alpha_max;
  k.t_min = prm.t_min;
  return k;
}

}  // namespace
}  // namespace abcd
