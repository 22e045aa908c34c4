// render_fwd.hip -- forward tile rasterisation of the active partition,
// composited between F and B (paper, Method section), and the cached-render
// variant (F = B = transparent, fp16 store) used to refresh a partition's
// cached images.
//
// The forward blends each pixel's list front to back and stops a pixel once
// the next blend would take its transmittance below t_min; the workgroup
// stops when all its pixels have stopped.
//
// Each wave (an 8x8 quadrant of the tile) walks only the staged entries whose
// alpha >= alpha_min ellipse reaches its pixels: the others cannot blend at any
// of them, so the result is the same, and in tiles of many small
// Gaussians a wave's walk is a fraction of the tile's list.
#include "blend.h"

namespace abcd {
namespace {

// Workgroup memory of the forward kernels: per wave, the staged entries that
// reach its pixels, in list order, then up to kGroup - 1 entries that blend
// nothing; reads run one group ahead.
constexpr int kSlots = 256 + 2 * kGroup;
struct FwdLds {
  float4 ga[4][kSlots];  // u, v, qa, qb
  float2 gq[4][kSlots];  // qc, opacity
  float2 rg[4][kSlots];  // r, g
  float bl[4][kSlots];   // b
  uint8_t at[4][256];    // position in the batch
  float4 box[4];         // per wave: box of its pixels that can still blend
  int wcnt[5][4];
  unsigned long long nb;
  uint32_t base;
  uint32_t walk;  // largest walk of the tile (split only)
};

// Stages one batch: the thread's entry `rec` (at position tid of the batch) into
// the lists of the waves w whose bit of `reach` is set, and the padding of the
// wave's own list. Returns the number of entries with any bit set and the
// length of the wave's list; ends with a barrier.
__device__ __forceinline__ int stage_fwd(FwdLds& s, const Rec& rec, uint32_t reach, int& wcnt) {
  const int tid = threadIdx.x, w = tid >> 6;
  int at[4];
  const int kept = quad_slots(reach, s.wcnt, at, wcnt);
  if (reach != 0u) {
    const Splat sp = make_splat(rec.m, rec.co);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if ((reach >> r) & 1u) {
        s.ga[r][at[r]] = make_float4(sp.u, sp.v, sp.qa, sp.qb);
        s.gq[r][at[r]] = make_float2(sp.qc, sp.o);
        s.rg[r][at[r]] = make_float2(rec.r, rec.g);
        s.bl[r][at[r]] = rec.b;
        s.at[r][at[r]] = (uint8_t)tid;
      }
    }
  }
  if ((tid & 63) < kGroup) {  // the last group's rest: of opacity 0
    const int p = wcnt + (tid & 63);
    s.ga[w][p] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    s.gq[w][p] = make_float2(0.0f, 0.0f);
    s.rg[w][p] = make_float2(0.0f, 0.0f);
    s.bl[w][p] = 0.0f;
  }
  __syncthreads();
  return kept;
}

// Small frames (at most kRowsTiles tiles, no split): four workgroups per
// tile (rows 4q .. 4q + 3 for quarter q), one pixel row per wave and four
// list entries per step of a wave, as in the backward for small frames. Lane
// l holds column l & 15 of the wave's row and entry l >> 4 of the step (entry
// 0 the frontmost). Per step, the transmittance before and after each entry
// is the running chain T times an exclusive and an inclusive prefix product of
// 1 - alpha over the step's entries (scans over lane bits 4 and 5). The
// inclusive products never increase along the step (each is a rounded product
// of the one before and a factor at most 1), so an entry blends exactly when
// its product is still at or above the threshold, and the first entry that
// fails stops the pixel. Each lane sums the colour, blend count and walk end
// of its own entries; the four rows are combined once, at the end (the
// pixel's transmittance is the smallest of the rows' last blended values).
template <bool kHalf>
__global__ __launch_bounds__(256) void render_fwd_rows_kernel(
    BlendConsts k, const uint32_t* __restrict__ tile_ranges, const uint32_t* __restrict__ values,
    const float2* __restrict__ means2d, const float4* __restrict__ conic_opacity,
    const float* __restrict__ rgb, const float4* __restrict__ F, const float4* __restrict__ B,
    float4* __restrict__ out, float* __restrict__ final_T, uint32_t* __restrict__ last,
    unsigned long long* __restrict__ n_blends, uint2* __restrict__ out16, int* __restrict__ rect,
    int fb_stop) {
  __shared__ FwdLds s;
  const int tile = (int)(blockIdx.x >> 2), quarter = (int)(blockIdx.x & 3);
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63, col = lane & 15, e = lane >> 4;
  const int px = (tile % k.ntx) * kTile + col;
  const int py = (tile / k.ntx) * kTile + 4 * quarter + (tid >> 6);
  const bool inside = px < k.width && py < k.height;
  const TileBox box = tile_box(k, tile);
  const uint32_t start = tile_ranges[2 * tile], end = tile_ranges[2 * tile + 1];
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
  bool done = !inside;
  float thr = k.t_min;  // stop threshold on the next transmittance (see render_fwd_kernel)
  if (!kHalf && fb_stop && F && inside) {
    const float vis = 1.0f - F[(int64_t)py * k.width + px].w;
    thr = vis > 0.0f ? k.t_min / vis : __builtin_huge_valf();
    done = vis < k.t_min;
  }
  float amin_l = done ? __builtin_huge_valf() : fmaxf(k.alpha_min, __FLT_DENORM_MIN__);
  float T = 1.0f;      // the pixel's chain through the steps so far (same in its four lanes)
  float Tlast = 1.0f;  // the chain after this lane's last entry that passed the threshold
  float cr = 0.0f, cg = 0.0f, cb = 0.0f;
  uint32_t lastk = 0, nb = 0;
  const bool odd = lane & 16, high = lane & 32;
  if (tid == 0) s.nb = 0;
  const uint32_t lastpos = end > start ? end - 1 : start;
  Rec rec{};
  uint32_t gid_next = 0;
  if (end > start) {  // uniform
    const uint32_t gid0 = values[min(start + tid, lastpos)];
    gid_next = values[min(start + 256 + tid, lastpos)];
    rec = gather_rec(gid0, start + tid < end, means2d, conic_opacity, rgb);
  }
  for (uint32_t b0 = start; b0 < end; b0 += 256) {
    if (__syncthreads_count(done) == 256) break;
    const float3 cn = conic_of(rec.co);
    const uint32_t rows = rec.valid ? splat_rows_single(rec.m.x, rec.m.y, cn.x, cn.y, cn.z,
                                                        rec.co.w, k.alpha_min, box, 4 * quarter)
                                    : 0u;
    int wcnt;
    stage_fwd(s, rec, rows, wcnt);
    const uint32_t nxt = b0 + 256 + tid;
    const uint32_t gid_after = values[min(b0 + 512 + tid, lastpos)];
    rec = gather_rec(gid_next, nxt < end, means2d, conic_opacity, rgb);
    gid_next = gid_after;
    if (__ballot(!done)) {
      // a step's four entries, one per 16 lanes; the next step's are read while
      // this one blends
      int jl = -1;  // position in the wave's list of the lane's last blended entry
      float4 ga = s.ga[w][e];
      float2 gq = s.gq[w][e], rg = s.rg[w][e];
      float bl = s.bl[w][e];
      for (int j0 = 0; j0 < wcnt; j0 += 4) {
        const int jw = j0 + e;
        const float al = splat_alpha(fx - ga.x, fy - ga.y, ga.z, ga.w, gq.x, gq.y, k.alpha_max);
        const float2 rg0 = rg;
        const float bl0 = bl;
        ga = s.ga[w][jw + 4];
        gq = s.gq[w][jw + 4];
        rg = s.rg[w][jw + 4];
        bl = s.bl[w][jw + 4];
        // 0 where the lane blends nothing: past the list, below alpha_min, or
        // the pixel has stopped
        const float a = al >= amin_l ? al : 0.0f;
        const float om = 1.0f - a;
        const Swapped p1 = swap_bit4(om);
        const float t1 = p1.first * p1.second;
        const Swapped p2 = swap_bit5(t1);
        const float in1 = odd ? t1 : om, ex1 = odd ? p1.first : 1.0f;
        const float Tn = T * (high ? in1 * p2.first : in1);  // after the entry
        const float Tc = T * (high ? ex1 * p2.first : ex1);  // before it
        const bool ok = Tn >= thr;
        // a zero weight adds exactly zero (colours are finite and >= 0)
        const float wgt = ok ? a * Tc : 0.0f;
        cr = fmaf(rg0.x, wgt, cr);
        cg = fmaf(rg0.y, wgt, cg);
        cb = fmaf(bl0, wgt, cb);
        const bool blend = ok && a != 0.0f;
        jl = blend ? jw : jl;
        nb += blend ? 1u : 0u;
        Tlast = ok ? Tn : Tlast;
        T *= p2.first * p2.second;  // through the step's four entries
        done = done || T < thr;
        amin_l = done ? __builtin_huge_valf() : amin_l;
        if (!__ballot(!done)) break;  // wave-uniform
      }
      if (jl >= 0) lastk = (b0 - start) + (uint32_t)s.at[w][jl] + 1u;
    }
    // s_wcnt is rewritten only after the next barrier
  }
  // combine the pixel's four lanes
  {
    const Swapped r1 = swap_bit4(cr), g1 = swap_bit4(cg), c1 = swap_bit4(cb), t1 = swap_bit4(Tlast);
    const Swapped r2 = swap_bit5(r1.first + r1.second), g2 = swap_bit5(g1.first + g1.second),
                  c2 = swap_bit5(c1.first + c1.second), t2 = swap_bit5(fminf(t1.first, t1.second));
    cr = r2.first + r2.second;
    cg = g2.first + g2.second;
    cb = c2.first + c2.second;
    T = fminf(t2.first, t2.second);
    const Swapped k1 = swap_bit4(__uint_as_float(lastk));
    const uint32_t l1 = max(__float_as_uint(k1.first), __float_as_uint(k1.second));
    const Swapped k2 = swap_bit5(__uint_as_float(l1));
    lastk = max(__float_as_uint(k2.first), __float_as_uint(k2.second));
  }
  if (kHalf && rect) {
    // coverage of the cached image: tiles holding any pixel that blended
    if (__syncthreads_or(inside && T < 1.0f) && tid == 0) {
      const int tx = tile % k.ntx, ty = tile / k.ntx;
      atomicMin(&rect[0], tx * kTile);
      atomicMin(&rect[1], ty * kTile);
      atomicMax(&rect[2], min(tx * kTile + kTile, k.width));
      atomicMax(&rect[3], min(ty * kTile + kTile, k.height));
    }
  }
  if (inside && e == 0) {
    const int64_t p = (int64_t)py * k.width + px;
    if (kHalf) {
      const _Float16 h[4] = {(_Float16)cr, (_Float16)cg, (_Float16)cb, (_Float16)(1.0f - T)};
      out16[p] = __builtin_bit_cast(uint2, h);
    } else {
      const float4 f = F ? F[p] : make_float4(0, 0, 0, 0);
      const float4 bb = B ? B[p] : make_float4(0, 0, 0, 0);
      const float s = 1.0f - f.w;
      out[p] = make_float4(f.x + s * (cr + T * bb.x), f.y + s * (cg + T * bb.y),
                           f.z + s * (cb + T * bb.z), f.w + s * (1.0f - T * (1.0f - bb.w)));
      final_T[p] = T;
      last[p] = lastk;
    }
  }
  if (n_blends) {
    const unsigned long long wsum = wave_sum_u32(nb);
    __syncthreads();
    if (lane == 0) atomicAdd(&s.nb, wsum);
    __syncthreads();
    if (tid == 0 && s.nb) atomicAdd(n_blends, s.nb);
  }
}

// kHalf: the cached-render variant: F = B = transparent, the image is written
// as fp16 RGBA to out16 (round to nearest even), no final T or walk lengths.
// Register budget: four waves per SIMD (at most 128 VGPRs).
template <bool kHalf>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void render_fwd_kernel(
    BlendConsts k, const uint32_t* __restrict__ tile_ranges, const uint32_t* __restrict__ values,
    const float2* __restrict__ means2d, const float4* __restrict__ conic_opacity,
    const float* __restrict__ rgb, const float4* __restrict__ F, const float4* __restrict__ B,
    float4* __restrict__ out, float* __restrict__ final_T, uint32_t* __restrict__ last,
    unsigned long long* __restrict__ n_blends, const uint32_t* __restrict__ order,
    uint2* __restrict__ out16, int* __restrict__ rect, int fb_stop, SplitLayout sp) {
  __shared__ FwdLds s;
  const int tile = tile_of_block(k, order);
  if ((unsigned)tile >= (unsigned)k.ntiles) return;
  const int tid = threadIdx.x;
  const int px = (tile % k.ntx) * kTile + quad_x(tid);
  const int py = (tile / k.ntx) * kTile + quad_y(tid);
  const bool inside = px < k.width && py < k.height;
  const uint32_t start = tile_ranges[2 * tile], end = tile_ranges[2 * tile + 1];
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
  float T = 1.0f, cr = 0.0f, cg = 0.0f, cb = 0.0f;
  uint32_t lastk = 0, nb = 0;
  bool done = !inside;  // before the walk
  // Stop threshold on the next transmittance. The compositing-aware rule
  // (1 - F_a) T_next < t_min is applied as T_next < t_min / (1 - F_a); a pixel
  // whose F leaves it less than t_min of weight blends nothing.
  float thr = k.t_min;
  if (!kHalf && fb_stop && F && inside) {
    const float vis = 1.0f - F[(int64_t)py * k.width + px].w;
    done = vis < k.t_min || !(vis > 0.0f);
    thr = done ? 0.0f : k.t_min / vis;
  }
  // alpha below which the lane blends nothing: alpha_min (at least the
  // smallest positive number: an alpha of zero blends nothing), infinite once
  // the pixel has stopped
  float amin_l = done ? __builtin_huge_valf() : fmaxf(k.alpha_min, __FLT_DENORM_MIN__);
  if (tid == 0) {
    s.nb = 0;
    s.walk = 0;
  }
  // Checkpoints for the split backward (uniform state): a slot per boundary
  // the walk crosses, taken when it crosses
  const uint32_t len = end - start;
  const uint32_t cht = (!kHalf && sp.ckpt) ? (uint32_t)sp.ch : 0u;
  const uint32_t chd = cht != 0u ? cht : 1u;  // divisor (only used when splitting)
  bool split_ok = cht != 0u && len > cht;
  bool crossed = false;
  // entries staged in the current chunk and the most in any chunk so far: the
  // backward's cost estimate for ordering its work items
  uint32_t staged = 0, staged_max = 0;
  // Loads run two batches ahead of use: the list values of batch b + 2 and
  // the gathers of batch b + 1 are in flight while batch b blends. Positions
  // past the list read its last entry (valid == false), so every load is
  // unconditional and in bounds.
  const uint32_t lastpos = end > start ? end - 1 : start;
  Rec rec{};
  uint32_t gid_next = 0;
  if (end > start) {  // uniform
    const uint32_t gid0 = values[min(start + tid, lastpos)];
    gid_next = values[min(start + 256 + tid, lastpos)];
    rec = gather_rec(gid0, start + tid < end, means2d, conic_opacity, rgb);
  }
  for (uint32_t b0 = start; b0 < end; b0 += 256) {
    const float4 box = live_box(k, tile, amin_l < __builtin_huge_valf());
    if ((tid & 63) == 0) s.box[tid >> 6] = box;
    if (__syncthreads_count(amin_l == __builtin_huge_valf()) == 256) break;
    if (split_ok && b0 > start && (b0 - start) % chd == 0 && (b0 - start) / chd < kMaxChunks) {
      // state after the positions before b0; no pixel walks past a boundary
      // the loop did not reach
      if (tid == 0) {
        const uint32_t got = atomicAdd(&sp.hdr[0], 1u);
        s.base = got < sp.nslots ? got : kNoSlot;
        sp.slot_of[(size_t)tile * kMaxChunks + (b0 - start) / chd] = s.base;
      }
      __syncthreads();
      const uint32_t slot = s.base;
      if (slot == kNoSlot) {
        split_ok = false;  // out of slots: the backward takes this tile whole
      } else {
        sp.ckpt[(size_t)slot * 256 + tid] = make_float4(T, cr, cg, cb);
        crossed = true;
        staged_max = max(staged_max, staged);
        staged = 0;
      }
    }
    // each wave walks only the staged entries whose ellipse reaches the box of
    // its pixels that have not stopped: the others contribute nothing
    const uint32_t quads = rec.valid ? splat_quads(rec.m, rec.co, k.alpha_min, s.box) : 0u;
    int wcnt;
    staged += (uint32_t)stage_fwd(s, rec, quads, wcnt);
    const int w = tid >> 6;
    // gathers of the next batch and list values of the one after overlap the
    // blend of this one
    const uint32_t nxt = b0 + 256 + tid;
    const uint32_t gid_after = values[min(b0 + 512 + tid, lastpos)];
    rec = gather_rec(gid_next, nxt < end, means2d, conic_opacity, rgb);
    gid_next = gid_after;
    if (__ballot(amin_l < __builtin_huge_valf())) {
      // The wave walks its own list kGroup entries at a time, 85 vector
      // instructions a group, 21 an entry: a tile whose walk sets the launch's
      // length has each SIMD of its CU to a single wave, which issues one
      // instruction every 4.7 clocks, some 100 clocks an entry, so the count is
      // what it costs. The next group's geometry is read while this one blends
      // and a group's colours while its alphas are computed, so no LDS latency is
      // waited for, and consecutive records make two entries one 16-byte read.
      // Against selects on the stop in every entry and reads through a list of
      // slots (28 instructions): 1M Gaussians at 1297x840 180 -> 151 us, 300K
      // 167 -> 138, 4M tiny ones at 2560x1440 486 -> 390, with the opacity inside
      // the exponent; alpha as a product costs one instruction of that (on
      // quadrants 145 -> 148, 129 -> 131 and 283 -> 288).
      int jl = -1;  // position in the wave's list of the last entry the lane blended
      float4 ga[kGroup];
      float2 gq[kGroup];
#pragma unroll
      for (int i = 0; i < kGroup; ++i) {
        ga[i] = s.ga[w][i];
        gq[i] = s.gq[w][i];
      }
      for (int j0 = 0; j0 < wcnt; j0 += kGroup) {
        float2 rg[kGroup];
        float bl[kGroup];
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
          rg[i] = s.rg[w][j0 + i];
          bl[i] = s.bl[w][j0 + i];
        }
        // alpha of each entry at this pixel, 0 where the lane does not blend
        // it: below alpha_min, or the pixel has stopped (amin_l = inf)
        float a[kGroup];
        bool hit[kGroup];
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
          const float al = splat_alpha(fx - ga[i].x, fy - ga[i].y, ga[i].z, ga[i].w, gq[i].x,
                                       gq[i].y, k.alpha_max);
          hit[i] = al >= amin_l;
          a[i] = hit[i] ? al : 0.0f;
        }
        static_assert(kGroup == 4, "four flags");
        uint32_t hits = bits_of(hit);  // entry i of the group in bit 3 - i
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
          ga[i] = s.ga[w][j0 + kGroup + i];
          gq[i] = s.gq[w][j0 + kGroup + i];
        }
        // The chain Tc of every hit blended, T (1 - alpha) with one rounding
        // (exactly T where alpha = 0), holds the values of the entry-by-entry
        // walk up to its first stop. T never increases and only hits change
        // it, so an entry blends exactly when its next value is still at or
        // above the threshold: the first hit below stops the pixel and every
        // later value is below too.
        float Tc[kGroup + 1], wt[kGroup];
        Tc[0] = T;
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
          Tc[i + 1] = fmaf(-Tc[i], a[i], Tc[i]);
          wt[i] = a[i] * Tc[i];
        }
        const bool stops = Tc[kGroup] < thr;  // not of a lane that had stopped: its a = 0
        bool none_left = false;
        if (__ballot(stops)) {
          // some pixel stops in this group: its entries from the stop on get
          // weight zero, which adds exactly zero (colours are finite and >= 0)
          bool ok[kGroup];
          float Tk = T;
#pragma unroll
          for (int i = 0; i < kGroup; ++i) {
            ok[i] = Tc[i + 1] >= thr;
            wt[i] = ok[i] ? wt[i] : 0.0f;
            Tk = ok[i] ? Tc[i + 1] : Tk;
          }
          Tc[kGroup] = Tk;
          hits &= bits_of(ok);
          amin_l = stops ? __builtin_huge_valf() : amin_l;
          none_left = !__ballot(amin_l < __builtin_huge_valf());
        }
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
          cr = fmaf(rg[i].x, wt[i], cr);
          cg = fmaf(rg[i].y, wt[i], cg);
          cb = fmaf(bl[i], wt[i], cb);
        }
        T = Tc[kGroup];
        nb += (uint32_t)__popc(hits);
        jl = hits ? j0 + kGroup - __ffs((int)hits) : jl;
        if (none_left) break;  // wave-uniform
      }
      if (jl >= 0) lastk = (b0 - start) + (uint32_t)s.at[w][jl] + 1u;
    }
    // s.wcnt is rewritten only after the next barrier
  }
  if (cht != 0u) {
    // the tile's largest walk, for the backward's schedule
    uint32_t wmax = lastk;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) wmax = max(wmax, (uint32_t)__shfl_xor((int)wmax, off, 64));
    if ((tid & 63) == 0 && wmax) atomicMax(&s.walk, wmax);
    __syncthreads();  // every thread has read s.base; s.walk is complete
    if (tid == 0) {
      sp.walk[tile] = s.walk;
      uint32_t fin = kNoSlot;
      if (split_ok && crossed) {
        const uint32_t got = atomicAdd(&sp.hdr[0], 1u);
        if (got < sp.nslots) fin = got;
      }
      s.base = fin;
      sp.slot_of[(size_t)tile * kMaxChunks] = fin;
      sp.work[tile] = min(max(staged_max, staged), kSplitTile - 1u) | (fin != kNoSlot ? kSplitTile : 0u);
    }
    __syncthreads();
    const uint32_t slot = s.base;
    if (slot != kNoSlot) sp.ckpt[(size_t)slot * 256 + tid] = make_float4(T, cr, cg, cb);
  }
  if (kHalf && rect) {
    // coverage of the cached image: tiles holding any pixel that blended
    if (__syncthreads_or(inside && T < 1.0f) && tid == 0) {
      const int tx = tile % k.ntx, ty = tile / k.ntx;
      atomicMin(&rect[0], tx * kTile);
      atomicMin(&rect[1], ty * kTile);
      atomicMax(&rect[2], min(tx * kTile + kTile, k.width));
      atomicMax(&rect[3], min(ty * kTile + kTile, k.height));
    }
  }
  if (inside) {
    const int64_t p = (int64_t)py * k.width + px;
    if (kHalf) {
      const _Float16 h[4] = {(_Float16)cr, (_Float16)cg, (_Float16)cb, (_Float16)(1.0f - T)};
      out16[p] = __builtin_bit_cast(uint2, h);
    } else {
      const float4 f = F ? F[p] : make_float4(0, 0, 0, 0);
      const float4 bb = B ? B[p] : make_float4(0, 0, 0, 0);
      const float s = 1.0f - f.w;
      out[p] = make_float4(f.x + s * (cr + T * bb.x), f.y + s * (cg + T * bb.y),
                           f.z + s * (cb + T * bb.z), f.w + s * (1.0f - T * (1.0f - bb.w)));
      final_T[p] = T;
      last[p] = lastk;
    }
  }
  if (n_blends) {
    const unsigned long long wsum = wave_sum_u32(nb);
    __syncthreads();
    if ((tid & 63) == 0) atomicAdd(&s.nb, wsum);
    __syncthreads();
    if (tid == 0 && s.nb) atomicAdd(n_blends, s.nb);
  }
}

__global__ void rect_init_kernel(int* __restrict__ rect, int width, int height) {
  if (threadIdx.x == 0) {
    rect[0] = width;
    rect[1] = height;
    rect[2] = 0;
    rect[3] = 0;
  }
}

}  // namespace

int32_t launch_render_fwd(const abcd_camera& cam, const abcd_raster_params& prm,
                          const uint32_t* tile_ranges, const uint32_t* values_sorted,
                          const float* means2d, const float* conic_opacity, const float* rgb,
                          const float* F, const float* B, float* out_rgba, float* final_T,
                          uint32_t* last, unsigned long long* n_blends, const uint32_t* tile_order,
                          const SplitLayout& split, hipStream_t stream) {
  const BlendConsts k = consts(cam, prm);
  const int grid = tile_order ? k.ntiles : 8 * k.per_xcd;
  if (!split.ckpt && k.ntiles <= kRowsTiles) {
    ABCD_LAUNCH("render_fwd", render_fwd_rows_kernel<false>, 4 * k.ntiles, kBlock, 0, stream, k,
                tile_ranges, values_sorted, reinterpret_cast<const float2*>(means2d),
                reinterpret_cast<const float4*>(conic_opacity), rgb,
                reinterpret_cast<const float4*>(F), reinterpret_cast<const float4*>(B),
                reinterpret_cast<float4*>(out_rgba), final_T, last, n_blends, nullptr, nullptr,
                (int)(prm.flags & ABCD_FLAG_FB_STOP));
    ABCD_HIP(hipGetLastError());
    return ABCD_OK;
  }
  if (split.ckpt) TRY_STATUS(launch_zero(reinterpret_cast<float*>(split.hdr), 16, stream));
  ABCD_LAUNCH("render_fwd", render_fwd_kernel<false>, grid, kBlock, 0, stream, k, tile_ranges,
              values_sorted, reinterpret_cast<const float2*>(means2d),
              reinterpret_cast<const float4*>(conic_opacity), rgb,
              reinterpret_cast<const float4*>(F), reinterpret_cast<const float4*>(B),
              reinterpret_cast<float4*>(out_rgba), final_T, last, n_blends, tile_order, nullptr,
              nullptr, (int)(prm.flags & ABCD_FLAG_FB_STOP), split);
  ABCD_HIP(hipGetLastError());
  return ABCD_OK;
}

int32_t launch_render_cache(const abcd_camera& cam, const abcd_raster_params& prm,
                            const uint32_t* tile_ranges, const uint32_t* tile_order,
                            const uint32_t* values_sorted, const float* means2d,
                            const float* conic_opacity, const float* rgb, uint16_t* image_f16,
                            int32_t* rect, hipStream_t stream) {
  const BlendConsts k = consts(cam, prm);
  const int grid = tile_order ? k.ntiles : 8 * k.per_xcd;
  if (rect) {
    ABCD_LAUNCH("cache_rect_init", rect_init_kernel, 1, 64, 0, stream, rect, k.width, k.height);
    ABCD_HIP(hipGetLastError());
  }
  if (k.ntiles <= kRowsTiles) {
    ABCD_LAUNCH("render_cache", render_fwd_rows_kernel<true>, 4 * k.ntiles, kBlock, 0, stream, k,
                tile_ranges, values_sorted, reinterpret_cast<const float2*>(means2d),
                reinterpret_cast<const float4*>(conic_opacity), rgb, nullptr, nullptr, nullptr,
                nullptr, nullptr, nullptr, reinterpret_cast<uint2*>(image_f16), rect, 0);
    ABCD_HIP(hipGetLastError());
    return ABCD_OK;
  }
  ABCD_LAUNCH("render_cache", render_fwd_kernel<true>, grid, kBlock, 0, stream, k, tile_ranges,
              values_sorted, reinterpret_cast<const float2*>(means2d),
              reinterpret_cast<const float4*>(conic_opacity), rgb, nullptr, nullptr, nullptr,
              nullptr, nullptr, nullptr, tile_order, reinterpret_cast<uint2*>(image_f16), rect, 0,
              SplitLayout{});
  ABCD_HIP(hipGetLastError());
  return ABCD_OK;
}

}  // namespace abcd
