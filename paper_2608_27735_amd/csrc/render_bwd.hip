// render_bwd.hip -- backward of the tile blend (paper, Method section:
// gradients reach the active parameters only).
//
// The backward walks each pixel's list back to front from its last blended
// entry, reduces the 9 screen-space gradients of four Gaussians at a time
// across the wave with cross-lane adds, combines the 4 waves in LDS and adds
// each Gaussian's nine sums to global memory once per tile.
#include "blend.h"

namespace abcd {
namespace {

// DPP lane move inside the wave (all rows and banks enabled; every control
// used here reads a lane of the same row, so bound_ctrl never applies, and
// setting it lets the move fold into the add that consumes it).
template <int kCtrl>
__device__ __forceinline__ float dpp_mov(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xF, 0xF, true));
}

// A product whose result is zero where either factor is, whatever the other holds
// (v_mul_legacy_f32; the plain product otherwise). The weight of an entry that a
// pixel does not blend is zero, and so the NaN or infinity that the upstream
// gradient may hold at that pixel stays out of the entry's sums, for the price of
// a plain product.
extern "C" __device__ __attribute__((const)) float mul_zero_wins(float, float) __asm(
    "llvm.amdgcn.fmul.legacy");

// The sums over a wave's 8x8 pixels of the nine gradient values of four list
// entries. Lane l is pixel (l & 7, l >> 3) of the quadrant, so the column
// factor dx of a moment is common to a lane's column: the pixels' rows are
// summed first, of six values per entry (gp: dL/d alpha times d alpha / d o =
// e^power, so that an opacity of zero divides nothing),
//   v[e] = gp, v[4 + e] = gp dy, v[8 + e] = gp dy^2, v[12 + 4 c + e] = colour c,
// and the moments in dx are formed from those sums, once per column. Lane bits
// 5, 4 and 3 (the rows) are summed by halving: v_permlane32_swap
// (v_permlane16_swap) of two registers leaves one value's upper-half (odd-row)
// partner in the other register, so the sum of the two results holds one value
// in the lower half and the other in the upper; within a 16-lane row, two DPP
// adds that each write half of the banks (groups of four lanes) do the same,
// the partner a rotation by two banks away. That leaves three registers in
// which lane l holds values of entry e = (l >> 5) + 2 (l >> 4 & 1); dx is the
// lane's for that entry. Bit 2 (mirrored within eight lanes: any lane of the
// other quad will do, the quads are summed next) halves again, and the quads
// are summed. 56 instructions, 14 an entry; nine products per pixel and the
// sum of each over the wave took 33.
// On return lane l holds field sum_field(l) of its entry (none: -1).
__device__ __forceinline__ float wave_sums(const float (&v)[24], float dx, int lane) {
  float a[12], b[6];
#pragma unroll
  for (int q = 0; q < 12; ++q) {
    const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(v[2 * q]),
                                                    __float_as_int(v[2 * q + 1]), false, false);
    a[q] = __int_as_float(p[0]) + __int_as_float(p[1]);
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) {
    const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(a[2 * q]),
                                                    __float_as_int(a[2 * q + 1]), false, false);
    b[q] = __int_as_float(p[0]) + __int_as_float(p[1]);
  }
  // A DPP source may be read two wait states after a vector instruction wrote
  // it at the earliest: the order keeps two instructions between, and an s_nop
  // leads.
  float p0, p1, p2, r1, r2, d0, d1, d2;
  asm("s_nop 1\n\t"
      "v_add_f32_dpp %0, %8, %8 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %0, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %1, %10, %10 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %1, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %12, %12 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %2, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_mul_f32 %3, %0, %14\n\t"
      "v_add_f32_dpp %6, %1, %1 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %5, %0, %0 row_half_mirror row_mask:0xf bank_mask:0x5\n\t"
      "v_mul_f32 %4, %3, %14\n\t"
      "v_add_f32_dpp %5, %3, %3 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %6, %2, %2 row_half_mirror row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %7, %4, %4 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %5, %5 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %6, %6, %6 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %7, %7, %7 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %5, %5 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %6, %6, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %7, %7, %7 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf"
      : "=&v"(p0), "=&v"(p1), "=&v"(p2), "=&v"(r1), "=&v"(r2), "=&v"(d0), "=&v"(d1), "=&v"(d2)
      : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(b[4]), "v"(b[5]), "v"(dx));
  return (lane & 3) == 0 ? d0 : (lane & 3) == 1 ? d1 : d2;
}

// The entry of a group of four, and the field of its gradient (0, 1: gp times
// dx, dy; 2, 3, 4: dx^2, dx dy, dy^2; 5: gp; 6-8: the colours), whose sum lane l
// of wave_sums holds.
__device__ __forceinline__ int sum_entry(int l) { return ((l >> 5) & 1) + 2 * ((l >> 4) & 1); }
__device__ __forceinline__ int sum_field(int l) {
  const int b2 = (l >> 2) & 1, b3 = (l >> 3) & 1;
  if ((l & 3) == 0) return b2 ? (b3 ? 3 : 0) : (b3 ? 1 : 5);
  if ((l & 3) == 1) return b2 ? (b3 ? 8 : 7) : (b3 ? 6 : 4);
  return (l & 15) == 2 ? 2 : -1;
}

// Adds the staged entries' gradients to g2d[Gaussian][9] once the workgroup's
// sums are complete: wave w takes entries 64 w .. of cnt. Each lane first turns
// its entry's sums into dL/d(u, v, a, b, c, o, r, g, b): with q = o gp (dx, dy),
// d power / d(u, v) = (a dx + b dy, b dx + c dy), d power / d(a, b, c) =
// (-dx^2 / 2, -dx dy, -dy^2 / 2); ga.zw and gb.x hold the conic's factor times
// s, s^2 = log2(e) / 2, and gb.y the opacity o. Then the wave's lanes add nine
// consecutive floats of seven Gaussians at a time, so that an entry is one
// or two requests at the memory side, where the nine adds of one thread were
// nine: the flush is bound by the rate of atomics to memory that all XCDs
// share, not by issue (replacing the adds by nothing, or by plain stores, was
// worth 58 us of 233 on 300K Gaussians at 1297x840 and 310 of 1055 on the
// heavy-tailed 1M at 1080p; with seven entries an instruction all of it is
// gained: 163 and 707 us, the 1M block 292 -> 244).
__device__ __forceinline__ void flush_entries(int cnt, float (*s_acc)[257], const float4* s_ga,
                                              const float4* s_gb, const float4* s_gc,
                                              float* __restrict__ g2d) {
  const int tid = threadIdx.x, lane = tid & 63, e0 = tid & ~63;
  if (e0 >= cnt) return;  // wave-uniform
  if (tid < cnt) {
    const float4 ga = s_ga[tid];
    const float4 gb = s_gb[tid];
    const float o = gb.y, so = o * (1.0f / kHalfLog2e);
    const float mx = so * s_acc[0][tid], my = so * s_acc[1][tid];
    const float t = ga.z * mx + ga.w * my;
    s_acc[0][tid] = ga.z * t;
    s_acc[1][tid] = ga.w * t + gb.x * gb.x * my;
    s_acc[2][tid] *= -0.5f * o;
    s_acc[3][tid] *= -o;
    s_acc[4][tid] *= -0.5f * o;
  }
  const int end = min(cnt, e0 + 64);
  const int k = lane / 9, f = lane - 9 * k;
#pragma unroll 2
  for (int e = e0 + k; e < end + 7; e += 7) {
    const bool mine = lane < 63 && e < end;
    const int j = mine ? e : e0;
    const float g = s_acc[f < 9 ? f : 0][j];
    const uint32_t gid = __float_as_uint(s_gc[j].z);
    if (mine && g != 0.0f) atomicAdd(g2d + (uint64_t)gid * 9u + (uint32_t)f, g);
  }
}

// Workgroup memory of the backward kernels.
struct BwdLds {
  float4 ga[256];     // u, v, qa, qb
  float4 gb[256];     // qc, opacity, r, g
  float4 gc[256];     // colour b, list position, Gaussian
  float acc[9][257];  // [field][staged entry]; an entry's fields in different banks
  __align__(4) uint8_t idx[4][256];  // per wave: staged slots reaching its pixels
  float4 box[4];  // per wave: box of its pixels whose walk reaches the batch
  int wcnt[5][4];
  uint32_t max;
};

// One work item of the backward: list positions [lo, hi) of `tile`, chunk j
// of a split tile (lo = j ch) or the whole walk (j = 0, hi = 2^32 - 1). Each
// pixel walks the positions below its walk length back to front, starting
// from its final state in its last chunk and from the forward's checkpoint at
// hi otherwise. walk: each tile's longest walk (kDirect: found here, from its
// pixels).
template <bool kDirect>
__device__ __forceinline__ void bwd_item(
    BwdLds& s, const BlendConsts& k, int tile, uint32_t j, const uint32_t* __restrict__ tile_ranges,
    const uint32_t* __restrict__ values, const float2* __restrict__ means2d,
    const float4* __restrict__ conic_opacity, const float* __restrict__ rgb,
    const float4* __restrict__ F, const float4* __restrict__ B, const float* __restrict__ final_T,
    const uint32_t* __restrict__ last, const float4* __restrict__ dL_dout,
    const uint32_t* __restrict__ walk, float* __restrict__ g2d, const SplitLayout& sp) {
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int px = (tile % k.ntx) * kTile + quad_x(tid);
  const int py = (tile / k.ntx) * kTile + quad_y(tid);
  const bool inside = px < k.width && py < k.height;
  // Three rounds of loads before the walk: what the tile's arrays say (uniform),
  // the list's indices with the pixels' state, and the entries.
  const uint32_t start = tile_ranges[2 * tile];
  uint32_t nent = kDirect ? 0u : walk[tile];  // end of the item's walk
  // chunk bounds and checkpoint slots (a tile the forward did not split is
  // one item; all of this is uniform)
  uint32_t lo = 0, hi = 0xFFFFFFFFu, slot_hi = kNoSlot, slot_fin = kNoSlot;
  if (sp.ckpt) {
    const uint32_t* so = sp.slot_of + (size_t)tile * kMaxChunks;
    const uint32_t fin = so[0], end_slot = so[min(j + 1, kMaxChunks - 1)];
    if (fin < sp.nslots && j < kMaxChunks) {
      lo = j * (uint32_t)sp.ch;
      hi = chunk_hi(j, (uint32_t)sp.ch);
      slot_fin = fin;
      if (j + 1 < kMaxChunks && end_slot < sp.nslots) slot_hi = end_slot;
    } else if (j != 0) {
      return;  // not an item of this split
    }
  }
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
  // a pixel outside the image has no walk; it reads the tile's first pixel
  const int64_t p = inside ? (int64_t)py * k.width + px
                           : (int64_t)(tile / k.ntx) * kTile * k.width + (tile % k.ntx) * kTile;
  const uint32_t lastp = inside ? last[p] : 0u;
  if (kDirect) {
    if (tid == 0) s.max = 0;
    __syncthreads();
    if (lastp) atomicMax(&s.max, lastp);
    __syncthreads();
    nent = __builtin_amdgcn_readfirstlane(s.max);
  }
  nent = min(nent, hi);
  // entry j of a batch is list position bend - 1 - j (back to front)
  const uint32_t bstop = start + lo;
  uint32_t bend = nent > lo ? start + nent : bstop;
  // Loads run two batches ahead of use, as in the forward: positions below
  // bstop read the entry at bstop (valid == false), so every load is
  // unconditional and in bounds.
  Rec rec{};
  uint32_t gid_next = 0, gid0 = 0;
  if (bend > bstop) {  // uniform
    const uint32_t b1 = bend - min(256u, bend - bstop);  // end of the next batch
    const uint32_t p0 = bend - 1 - tid, p1 = b1 - 1 - tid;
    gid0 = values[(uint32_t)tid < bend - bstop ? p0 : bstop];
    gid_next = values[(uint32_t)tid < b1 - bstop ? p1 : bstop];
  }
  float T = final_T[p];
  const float4 G = dL_dout[p];
  const float4 f = F ? F[p] : make_float4(0, 0, 0, 0);
  const float4 bb = B ? B[p] : make_float4(0, 0, 0, 0);
  // the forward's state at hi and at the end of the walk
  float4 c_hi = make_float4(1.0f, 0.0f, 0.0f, 0.0f), c_end = c_hi;
  if (slot_hi != kNoSlot) {  // uniform
    c_hi = sp.ckpt[(size_t)slot_hi * 256 + tid];
    c_end = sp.ckpt[(size_t)slot_fin * 256 + tid];
  }
  if (bend > bstop)
    rec = gather_rec(gid0, (uint32_t)tid < bend - bstop, means2d, conic_opacity, rgb);
  const float sf = 1.0f - f.w;
  const float gcr = sf * G.x, gcg = sf * G.y, gcb = sf * G.z;
  const float gT = sf * (G.x * bb.x + G.y * bb.y + G.z * bb.z - G.w * (1.0f - bb.w));
  // d out / d T_final enters every entry's alpha-derivative as T_final g_T / (1 - alpha)
  const float TgT = T * gT;
  // RG = sum over channels of gc_ch R_ch, where R is the colour accumulated
  // behind the current entry (normalised by its transmittance): the
  // alpha-derivative needs R only through this sum.
  float RG = 0.0f;
  if (lastp > hi && slot_hi != kNoSlot) {  // crossed hi: its slot was taken
    // the walk goes on past this chunk: start from the forward's state at
    // hi; the colour behind is what the rest of the walk added
    T = c_hi.x;
    RG = (gcr * (c_end.y - c_hi.y) + gcg * (c_end.z - c_hi.z) + gcb * (c_end.w - c_hi.w)) / c_hi.x;
  }
  // the lane's entry of a group and field
  const int field = sum_field(lane);
  const bool adder = field >= 0;
  const int my_shift = 8 * sum_entry(lane);
  float* const acc_lane = s.acc[adder ? field : 0];
  while (bend > bstop) {
    const uint32_t bbeg = bend - min(256u, bend - bstop);
    const float4 box = live_box(k, tile, lastp > bbeg - start);
    if ((tid & 63) == 0) s.box[tid >> 6] = box;
    __syncthreads();
    // each wave walks only the staged entries whose ellipse reaches the box of
    // its pixels whose walk reaches the batch: the others contribute nothing
    const uint32_t quads = rec.valid ? splat_quads(rec.m, rec.co, k.alpha_min, s.box) : 0u;
    const bool keep = quads != 0u;
    int pos, wcnt;
    const int cnt = compact_rows(keep, quads, s.wcnt, s.idx, pos, wcnt);
    if (keep) {
      const Splat g = make_splat(rec.m, rec.co);
      s.ga[pos] = make_float4(g.u, g.v, g.qa, g.qb);
      s.gb[pos] = make_float4(g.qc, g.o, rec.r, rec.g);
      s.gc[pos] = make_float4(rec.b, __uint_as_float(bend - 1 - tid - start),
                              __uint_as_float(rec.gid), 0.0f);
#pragma unroll
      for (int q = 0; q < 9; ++q) s.acc[q][pos] = 0.0f;
    }
    __syncthreads();
    {
      // gathers of the next batch (ending at bbeg) and list values of the one
      // after (ending at b2) overlap the walk of this one
      const uint32_t b2 = bbeg - min(256u, bbeg - bstop);
      const uint32_t gid_after = values[(uint32_t)tid < b2 - bstop ? b2 - 1 - tid : bstop];
      rec = gather_rec(gid_next, (uint32_t)tid < bbeg - bstop, means2d, conic_opacity, rgb);
      gid_next = gid_after;
    }
    // Entries are read from LDS kGroup at a time, all reads issued before the
    // first is used, so the LDS latency is paid once per group.
    // The wave's list of staged slots, kBwdGroup at a time.
    static_assert(kBwdGroup == 4, "slot indices are read four at a time");
    const uint32_t* my_idx = reinterpret_cast<const uint32_t*>(s.idx[tid >> 6]);
    for (int j0 = 0; j0 < wcnt; j0 += kBwdGroup) {
    float4 gav[kBwdGroup], gbv[kBwdGroup];
    float2 gcv[kBwdGroup];
    // four slots (uniform); past the end of the list the group's first again
    // (a slot of its own might hold anything, and 0 times a NaN is one)
    uint32_t iw = __builtin_amdgcn_readfirstlane(my_idx[j0 / 4]);
    if (j0 + kBwdGroup > wcnt) {
      const uint32_t keep = 0xFFFFFFFFu >> (8 * (j0 + kBwdGroup - wcnt));
      iw = (iw & keep) | (((iw & 255u) * 0x01010101u) & ~keep);
    }
#pragma unroll
    for (int i = 0; i < kBwdGroup; ++i) {
      const int j = (int)((iw >> (8 * i)) & 255u);
      gav[i] = s.ga[j];
      gbv[i] = s.gb[j];
      gcv[i] = make_float2(s.gc[j].x, s.gc[j].y);
    }
    // keep the group's reads ahead of the arithmetic (the compiler would
    // otherwise sink each read into the branch that uses it)
#pragma unroll
    for (int i = 0; i < kBwdGroup; ++i)
      asm volatile("" ::"v"(gav[i].x), "v"(gav[i].y), "v"(gav[i].z), "v"(gav[i].w), "v"(gbv[i].x),
                   "v"(gbv[i].y), "v"(gbv[i].z), "v"(gbv[i].w), "v"(gcv[i].x), "v"(gcv[i].y));
    const int my_slot = (int)((iw >> my_shift) & 255u);
    const float my_u = s.ga[my_slot].x;
    // Per lane and entry: alpha and d alpha / d o, zero where the pixel does not
    // blend it (its walk did not reach it, alpha < alpha_min, or it is past the
    // end of the wave's list), the derivative also at the clamp.
    float a[kBwdGroup], de[kBwdGroup], dy[kBwdGroup];
    uint64_t any = 0;
#pragma unroll
    for (int i = 0; i < kBwdGroup; ++i) {
      const float dx = fx - gav[i].x;
      dy[i] = fy - gav[i].y;
      const float e = splat_exp(dx, dy[i], gav[i].z, gav[i].w, gbv[i].x);
      const float raw = gbv[i].y * e;  // splat_alpha_raw
      const uint64_t m = __builtin_amdgcn_ballot_w64(__float_as_uint(gcv[i].y) < lastp) &
                         __builtin_amdgcn_ballot_w64(raw >= k.alpha_min) &
                         (j0 + i < wcnt ? ~0ull : 0ull);
      a[i] = __builtin_amdgcn_inverse_ballot_w64(m) ? clamp_alpha(raw, k.alpha_max) : 0.0f;
      de[i] = __builtin_amdgcn_inverse_ballot_w64(
                  m & __builtin_amdgcn_ballot_w64(raw <= k.alpha_max)) ? e : 0.0f;
      any |= m;
    }
    if (!any) continue;  // wave-uniform
    // No branch from here on: a lane that does not blend an entry takes alpha
    // = 0, which leaves T and RG unchanged and gives zero gradients. (Skipping
    // the entries that no lane of the wave blends, one in five, cost more in
    // register copies at the joins than it saved.)
    float gr[6 * kBwdGroup];
#pragma unroll
    for (int i = 0; i < kBwdGroup; ++i) {
      const float iom = __builtin_amdgcn_rcpf(1.0f - a[i]);  // 1 - a >= 1 - alpha_max > 0
      T *= iom;  // before the entry
      const float wgt = a[i] * T;
      gr[12 + i] = mul_zero_wins(wgt, gcr);
      gr[16 + i] = mul_zero_wins(wgt, gcg);
      gr[20 + i] = mul_zero_wins(wgt, gcb);
      const float D = fmaf(gcv[i].x, gcb, fmaf(gbv[i].w, gcg, fmaf(gbv[i].z, gcr, -RG)));
      const float dLda = T * D - iom * TgT;
      RG = fmaf(a[i], D, RG);
      // no gradient where the clamp cuts the derivative; the opacity, the conic
      // and the constant factors are applied once per entry at the flush
      const float gp = mul_zero_wins(de[i], dLda);
      const float r = gp * dy[i];
      gr[0 + i] = gp;
      gr[4 + i] = r;
      gr[8 + i] = r * dy[i];
    }
    const float out = wave_sums(gr, fx - my_u, lane);
    if (adder) atomicAdd(acc_lane + my_slot, out);
    }
    __syncthreads();
    flush_entries(cnt, s.acc, s.ga, s.gb, s.gc, g2d);
    bend = bbeg;
  }
}

// Persistent workgroups take work items, heaviest first, from a queue until
// it is empty (every workgroup reaches the end of the queue and exits). An item
// is taken when the one before is done: taken while it runs, heavy items waited
// for workgroups that were still busy (300K Gaussians at 1297x840 159 -> 194 us).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(5))) void render_bwd_kernel(
    BlendConsts k, const uint32_t* __restrict__ tile_ranges, const uint32_t* __restrict__ values,
    const float2* __restrict__ means2d, const float4* __restrict__ conic_opacity,
    const float* __restrict__ rgb, const float4* __restrict__ F, const float4* __restrict__ B,
    const float* __restrict__ final_T, const uint32_t* __restrict__ last,
    const float4* __restrict__ dL_dout, const uint32_t* __restrict__ walk, float* __restrict__ g2d,
    const uint2* __restrict__ items,
    uint32_t* __restrict__ queue, uint32_t max_items, SplitLayout sp) {
  __shared__ BwdLds s;
  __shared__ uint2 s_item;
  const uint32_t n_items = min(queue[0], max_items);
  // Atomic adds to one address are serialised, and light items at the end
  // are taken faster than one counter can serve them. So item i belongs to
  // queue i mod nq (nq = kQueues, fewer for a smaller grid), each queue
  // heaviest first, and workgroup b takes from queue b mod nq (one per XCD,
  // which take workgroups round robin). The first item of workgroup b is item
  // b, taken without an atomic; later ones come from the queue's counter.
  const uint32_t nq = min(gridDim.x, (uint32_t)kQueues);
  const uint32_t q = blockIdx.x % nq;
  const uint32_t gq = (gridDim.x - q + nq - 1) / nq;  // workgroups of queue q
  uint2 it = blockIdx.x < n_items ? items[blockIdx.x] : make_uint2(kNoSlot, 0u);
  while (it.x != kNoSlot) {  // uniform
    if (it.x < (uint32_t)k.ntiles)
      bwd_item<false>(s, k, (int)it.x, it.y, tile_ranges, values, means2d, conic_opacity, rgb, F, B,
                      final_T, last, dL_dout, walk, g2d, sp);
    if (threadIdx.x == 0) {
      const uint32_t r = gq + atomicAdd(&queue[kQueueStride * q + 1], 1u);
      const uint64_t i = (uint64_t)q + (uint64_t)nq * r;
      s_item = i < n_items ? items[i] : make_uint2(kNoSlot, 0u);
    }
    __syncthreads();
    it = s_item;
    it.x = __builtin_amdgcn_readfirstlane(it.x);
    it.y = __builtin_amdgcn_readfirstlane(it.y);
    __syncthreads();
  }
}

constexpr int kDirectTiles = 1024;
static_assert(kDirectTiles <= kFewTiles, "the direct kernel asks for the pairs");

// Sums of nine values over each 16-lane row, by a butterfly over lane bits 3
// (row rotate 8), 2 (half-row mirror, which pairs lanes whose bit 2 differs),
// 1 and 0 (quad permutes): each step halves values 0-7 with one select pair
// and one DPP add. On return lane c of a row holds the row total of value
// rowsum9_slot(c), and every lane the total of value 8 in v8.
__device__ __forceinline__ float row_sum9(const float (&g)[9], int c, float& v8) {
  const bool b3 = c & 8, b2 = c & 4, b1 = c & 2;
  float h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    h[i] = (b3 ? g[2 * i + 1] : g[2 * i]) + dpp_mov<0x128>(b3 ? g[2 * i] : g[2 * i + 1]);
  const float k0 = (b2 ? h[1] : h[0]) + dpp_mov<0x141>(b2 ? h[0] : h[1]);
  const float k1 = (b2 ? h[3] : h[2]) + dpp_mov<0x141>(b2 ? h[2] : h[3]);
  float m = (b1 ? k1 : k0) + dpp_mov<0x4E>(b1 ? k0 : k1);
  m += dpp_mov<0xB1>(m);
  v8 = g[8];
  v8 += dpp_mov<0x128>(v8);
  v8 += dpp_mov<0x141>(v8);
  v8 += dpp_mov<0x4E>(v8);
  v8 += dpp_mov<0xB1>(v8);
  return m;
}
__device__ __forceinline__ int rowsum9_slot(int c) {
  return 4 * ((c >> 1) & 1) + 2 * ((c >> 2) & 1) + ((c >> 3) & 1);
}

// Small frames, where one workgroup per tile leaves most of the chip idle and
// the longest list sets the launch's length: four workgroups per tile (rows
// 4q .. 4q + 3 for quarter q), one pixel row per wave, and four list entries
// per step of a wave. Lane l holds column l & 15 of the wave's row and entry
// l >> 4 of the step (entry 0 the backmost); the four copies of a pixel's
// state stay identical. Within a step the pixel's back-to-front recurrences
// over the four entries run as scans over lane bits 4 and 5: the
// transmittance before each entry is the running one times a prefix product
// of 1 / (1 - alpha), and the colour blended behind it a prefix sum S of
// alpha T (c . g), not normalised by the transmittance, so that the
// alpha-derivative is T (c . g) - (S + T_final g_T) / (1 - alpha).

__device__ __forceinline__ void bwd_rows(
    BwdLds& s, const BlendConsts& k, int tile, int quarter, const uint32_t* __restrict__ tile_ranges,
    const uint32_t* __restrict__ values,
    const float2* __restrict__ means2d, const float4* __restrict__ conic_opacity,
    const float* __restrict__ rgb, const float4* __restrict__ F, const float4* __restrict__ B,
    const float* __restrict__ final_T, const uint32_t* __restrict__ last,
    const float4* __restrict__ dL_dout, float* __restrict__ g2d) {
  const int tid = threadIdx.x, lane = tid & 63, col = lane & 15, e = lane >> 4;
  const int px = (tile % k.ntx) * kTile + col;
  const int py = (tile / k.ntx) * kTile + 4 * quarter + (tid >> 6);
  const bool inside = px < k.width && py < k.height;
  const TileBox box = tile_box(k, tile);
  const uint32_t start = tile_ranges[2 * tile];
  const float fx = (float)px + 0.5f, fy = (float)py + 0.5f;
  float T = 1.0f, gcr = 0, gcg = 0, gcb = 0, gT = 0;
  uint32_t lastp = 0;
  if (tid == 0) s.max = 0;
  __syncthreads();
  if (inside) {
    const int64_t p = (int64_t)py * k.width + px;
    T = final_T[p];
    lastp = last[p];
    const float4 G = dL_dout[p];
    const float4 f = F ? F[p] : make_float4(0, 0, 0, 0);
    const float4 bb = B ? B[p] : make_float4(0, 0, 0, 0);
    const float sf = 1.0f - f.w;
    gcr = sf * G.x;
    gcg = sf * G.y;
    gcb = sf * G.z;
    gT = sf * (G.x * bb.x + G.y * bb.y + G.z * bb.z - G.w * (1.0f - bb.w));
    if (lastp > 0u) atomicMax(&s.max, lastp);
  }
  __syncthreads();
  const uint32_t nent = __builtin_amdgcn_readfirstlane(s.max);  // end of the quarter's walk
  const float TgT = T * gT;  // T is the final transmittance here
  float S = 0.0f;            // colour behind the step (sum of alpha T (c . g))
  uint32_t wml = lastp;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) wml = max(wml, (uint32_t)__shfl_xor((int)wml, off, 64));
  wml = __builtin_amdgcn_readfirstlane(wml);
  const bool odd = lane & 16, high = lane & 32;
  const bool adder = (col & 1) == 0 || col == 1;
  const int slot = col == 1 ? 8 : rowsum9_slot(col);
  const uint32_t bstop = start;
  uint32_t bend = start + nent;
  Rec rec{};
  uint32_t gid_next = 0;
  if (bend > bstop) {  // uniform
    const uint32_t b1 = bend - min(256u, bend - bstop);
    const uint32_t p0 = bend - 1 - tid, p1 = b1 - 1 - tid;
    const uint32_t gid0 = values[(uint32_t)tid < bend - bstop ? p0 : bstop];
    gid_next = values[(uint32_t)tid < b1 - bstop ? p1 : bstop];
    rec = gather_rec(gid0, (uint32_t)tid < bend - bstop, means2d, conic_opacity, rgb);
  }
  while (bend > bstop) {
    const uint32_t bbeg = bend - min(256u, bend - bstop);
    __syncthreads();
    const float3 cn = conic_of(rec.co);
    const uint32_t rows = rec.valid ? splat_rows_single(rec.m.x, rec.m.y, cn.x, cn.y, cn.z,
                                                        rec.co.w, k.alpha_min, box, 4 * quarter)
                                    : 0u;
    const bool keep = rows != 0u;
    int pos, wcnt;
    const int cnt = compact_rows(keep, rows, s.wcnt, s.idx, pos, wcnt);
    if (keep) {
      const Splat sp = make_splat(rec.m, rec.co);
      s.ga[pos] = make_float4(sp.u, sp.v, sp.qa, sp.qb);
      s.gb[pos] = make_float4(sp.qc, sp.o, rec.r, rec.g);
      s.gc[pos] = make_float4(rec.b, __uint_as_float(bend - 1 - tid - start),
                              __uint_as_float(rec.gid), 0.0f);
#pragma unroll
      for (int q = 0; q < 9; ++q) s.acc[q][pos] = 0.0f;
    }
    __syncthreads();
    {
      const uint32_t b2 = bbeg - min(256u, bbeg - bstop);
      const uint32_t gid_after = values[(uint32_t)tid < b2 - bstop ? b2 - 1 - tid : bstop];
      rec = gather_rec(gid_next, (uint32_t)tid < bbeg - bstop, means2d, conic_opacity, rgb);
      gid_next = gid_after;
    }
    // slots past the end of the wave's list hold stale bytes: they still index
    // the staged arrays, and their lanes take part in nothing below. The next
    // step's entries, and the slots of the one after, are read while a step is
    // worked on.
    const uint8_t* my_idx = s.idx[tid >> 6];
    int jn = my_idx[e], jn2 = my_idx[4 + e];
    float4 gan = s.ga[jn], gbn = s.gb[jn], gcn = s.gc[jn];
    for (int j0 = 0; j0 < wcnt; j0 += 4) {
      const bool valid = j0 + e < wcnt;
      const int j = jn;
      const float4 ga = gan, gb = gbn;
      const float cb = gcn.x;
      const uint32_t kk = __float_as_uint(gcn.y);
      jn = jn2;
      jn2 = my_idx[min(j0 + 8 + e, 255)];
      gan = s.ga[jn];
      gbn = s.gb[jn];
      gcn = s.gc[jn];
      if (!__ballot(valid && kk < wml)) continue;  // wave-uniform
      const float dx = fx - ga.x, dy = fy - ga.y;
      const float de = splat_exp(dx, dy, ga.z, ga.w, gb.x);  // d alpha / d o
      const float raw = gb.y * de;  // splat_alpha_raw
      const bool contrib = valid && kk < lastp && raw >= k.alpha_min;
      if (!__ballot(contrib)) continue;  // wave-uniform
      const float a = contrib ? clamp_alpha(raw, k.alpha_max) : 0.0f;
      const float iom = __builtin_amdgcn_rcpf(1.0f - a);  // 1 - a >= 1 - alpha_max > 0
      // transmittance before each entry: T times the inclusive prefix product
      // of 1 / (1 - alpha) over the step's entries, back to front
      const Swapped p1 = swap_bit4(iom);
      const float t1 = p1.first * p1.second;
      const float in1 = odd ? t1 : iom;
      const Swapped p2 = swap_bit5(t1);
      const float Tk = T * (high ? in1 * p2.first : in1);
      const float ptot = p2.first * p2.second;
      const float CG = gb.z * gcr + gb.w * gcg + cb * gcb;
      const float wgt = a * Tk;
      // colour blended behind each entry within the step: exclusive prefix sum
      const float c0 = contrib ? wgt * CG : 0.0f;
      const Swapped s1 = swap_bit4(c0);
      const float u1 = s1.first + s1.second;
      const float ex1 = odd ? s1.first : 0.0f;
      const Swapped s2 = swap_bit5(u1);
      const float behind = S + (high ? ex1 + s2.first : ex1);
      const float stot = s2.first + s2.second;
      const float dLda = Tk * CG - iom * (behind + TgT);
      T *= ptot;
      S += stot;
      const float dm = (contrib && raw <= k.alpha_max) ? dLda : 0.0f;
      const float gp = de * dm;
      const float q = gp * dx, r = gp * dy;
      float gr[9];
      gr[0] = q;
      gr[1] = r;
      gr[2] = q * dx;
      gr[3] = q * dy;
      gr[4] = r * dy;
      gr[5] = gp;
      gr[6] = mul_zero_wins(wgt, gcr);
      gr[7] = mul_zero_wins(wgt, gcg);
      gr[8] = mul_zero_wins(wgt, gcb);
      float v8;
      const float m = row_sum9(gr, col, v8);
      float out = col == 1 ? v8 : m;
      asm volatile("" : "+v"(out));  // the last folds stay outside the branch (DPP add)
      if (adder && valid) atomicAdd(&s.acc[slot][j], out);
    }
    __syncthreads();
    flush_entries(cnt, s.acc, s.ga, s.gb, s.gc, g2d);
    bend = bbeg;
  }
}

__global__ __launch_bounds__(256) void render_bwd_rows_kernel(
    BlendConsts k, const uint32_t* __restrict__ tile_ranges, const uint32_t* __restrict__ values,
    const float2* __restrict__ means2d, const float4* __restrict__ conic_opacity,
    const float* __restrict__ rgb, const float4* __restrict__ F, const float4* __restrict__ B,
    const float* __restrict__ final_T, const uint32_t* __restrict__ last,
    const float4* __restrict__ dL_dout, float* __restrict__ g2d) {
  __shared__ BwdLds s;
  bwd_rows(s, k, (int)(blockIdx.x >> 2), (int)(blockIdx.x & 3), tile_ranges, values, means2d,
           conic_opacity, rgb, F, B, final_T, last, dL_dout, g2d);
}

// Unsplit frames of at most kDirectTiles tiles, without the schedule's two
// launches, in raster order: the first workgroups take a tile each, then come four
// per tile for the lists that are taken in rows (see kRowsList).
__global__ __launch_bounds__(256) void render_bwd_direct_kernel(
    BlendConsts k, const uint32_t* __restrict__ tile_ranges, const uint32_t* __restrict__ values,
    const float2* __restrict__ means2d, const float4* __restrict__ conic_opacity,
    const float* __restrict__ rgb, const float4* __restrict__ F, const float4* __restrict__ B,
    const float* __restrict__ final_T, const uint32_t* __restrict__ last,
    const float4* __restrict__ dL_dout, float* __restrict__ g2d) {
  __shared__ BwdLds s;
  const bool few = tile_ranges[2 * k.ntiles - 1] <= kFewPairs;
  const int b = (int)blockIdx.x, r = b - k.ntiles;
  const int tile = r < 0 ? b : r >> 2;
  const bool rows = few && tile_ranges[2 * tile + 1] - tile_ranges[2 * tile] >= kRowsList;
  if (rows != (r >= 0)) return;
  if (rows)
    bwd_rows(s, k, tile, r & 3, tile_ranges, values, means2d, conic_opacity, rgb, F, B, final_T,
             last, dL_dout, g2d);
  else
    bwd_item<true>(s, k, tile, 0u, tile_ranges, values, means2d, conic_opacity, rgb, F, B, final_T,
                   last, dL_dout, nullptr, g2d, SplitLayout{});
}

}  // namespace

static_assert(kQueueStride * kQueues == 64 * 8, "queue block of bwd_workspace_bytes");

// g2d ([n][9]), then the backward's tile work, tile order, work items (when
// not split) and queue.
size_t render_bwd_workspace_bytes(int64_t n) { return bwd_workspace_bytes(n); }

namespace {
// Workgroups of the persistent backward that fit the device at once.
int bwd_resident_blocks() {
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 1024;
  if (cached[dev] == 0) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, render_bwd_kernel, kBlock, 0) !=
            hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        per_cu <= 0 || cus <= 0) {
      (void)hipGetLastError();
      return 1024;
    }
    cached[dev] = per_cu * cus;
  }
  return cached[dev];
}
}  // namespace

int32_t launch_render_bwd_pixels(const abcd_camera& cam, const abcd_raster_params& prm, int64_t n,
                                 const uint32_t* tile_ranges, const uint32_t* values_sorted,
                                 const float* means2d, const float* conic_opacity,
                                 const float* rgb, const float* F, const float* B,
                                 const float* final_T, const uint32_t* last,
                                 const float* dL_dout, float* g2d, const SplitLayout& split,
                                 hipStream_t stream) {
  const BlendConsts k = consts(cam, prm);
  const int64_t g2d_count = 9 * g2d_stride(n);
  if (!split.ckpt && k.ntiles <= kDirectTiles) {
    TRY_STATUS(launch_zero(g2d, g2d_count, stream));
    if (k.ntiles <= kRowsTiles)
      ABCD_LAUNCH("render_bwd", render_bwd_rows_kernel, 4 * k.ntiles, kBlock, 0, stream, k,
                  tile_ranges, values_sorted, reinterpret_cast<const float2*>(means2d),
                  reinterpret_cast<const float4*>(conic_opacity), rgb,
                  reinterpret_cast<const float4*>(F), reinterpret_cast<const float4*>(B), final_T,
                  last, reinterpret_cast<const float4*>(dL_dout), g2d);
    else
      ABCD_LAUNCH("render_bwd", render_bwd_direct_kernel, 5 * k.ntiles, kBlock, 0, stream, k,
                  tile_ranges, values_sorted, reinterpret_cast<const float2*>(means2d),
                  reinterpret_cast<const float4*>(conic_opacity), rgb,
                  reinterpret_cast<const float4*>(F), reinterpret_cast<const float4*>(B), final_T,
                  last, reinterpret_cast<const float4*>(dL_dout), g2d);
    ABCD_HIP(hipGetLastError());
    return ABCD_OK;
  }
  char* tail = reinterpret_cast<char*>(g2d) + bwd_g2d_bytes(n);
  uint32_t* work = reinterpret_cast<uint32_t*>(tail);
  uint32_t* order = work + ABCD_MAX_TILES;
  uint2* own_items = reinterpret_cast<uint2*>(order + ABCD_MAX_TILES);
  uint32_t* queue = reinterpret_cast<uint32_t*>(own_items + ABCD_MAX_TILES);
  uint2* items = split.ckpt ? split.items : own_items;
  const uint32_t max_items =
      (uint32_t)k.ntiles + (split.ckpt ? split.nslots : 0u);
  // each tile's largest walk: from the forward when split, else from `last`
  const uint32_t* walk = work;
  if (split.ckpt)
    walk = split.walk;
  else
    TRY_STATUS(launch_tile_walk(k.width, k.height, last, work, stream));
  // heaviest items first: by the forward's per-chunk estimate when split,
  // else by the walk
  TRY_STATUS(launch_bwd_schedule(k.ntiles, split.ckpt ? split.work : walk, walk, order, split,
                                 items, max_items, queue, g2d, g2d_count, stream));
  const int grid = (int)std::min<int64_t>(bwd_resident_blocks(), max_items);
  ABCD_LAUNCH("render_bwd", render_bwd_kernel, grid, kBlock, 0, stream, k, tile_ranges,
              values_sorted, reinterpret_cast<const float2*>(means2d),
              reinterpret_cast<const float4*>(conic_opacity), rgb,
              reinterpret_cast<const float4*>(F), reinterpret_cast<const float4*>(B), final_T,
              last, reinterpret_cast<const float4*>(dL_dout), walk, g2d, items, queue,
              max_items, split);
  ABCD_HIP(hipGetLastError());
  return ABCD_OK;
}

}  // namespace abcd
