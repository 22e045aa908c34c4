// adam.hip -- Adam update of the active parameters after a step's backward.
//
// The paper trains the active block with gradient steps and does not name the
// optimizer; the 3DGS line it builds on uses Adam (Kingma and Ba 2015,
// Algorithm 1) with one learning rate per parameter group. One launch updates
// every group in place: a pure HBM stream (parameter, gradient and both
// moments read, parameter and moments written: 28 bytes per element).
// Workgroups are dealt to the groups in proportion to their sizes, 4,096
// elements each; a thread takes four float4s a row of 256 threads apart, so
// that each load of a wave covers 1 KB of consecutive bytes. (With 16
// consecutive elements per thread a wave's load touched 64 lines for a quarter
// of each: 59M elements took 442 us, 3.7 TB/s, against 313 us in rows.) Every
// byte is used once per step and the arrays of a large block exceed the caches,
// so accesses are marked non-temporal: 279 us, 5.9 TB/s. A group's last
// workgroup takes its one to four rows the same way, so a small block's launch
// is one round trip to memory: in us, with 16 elements per thread / the last
// workgroup element by element / now, for N Gaussians of 14 and of 59 floats:
// N = 512: 3.8 / 4.1 / 3.2, 4.7 / 4.1 / 4.2; 1,000: 5.7 / 6.2 / 3.9, 5.7 / 6.2 /
// 4.3; 2,000: 4.6 / 6.1 / 4.1, 4.9 / 6.3 / 4.3; 3,001: 16.3 / 6.0 / 4.2, 16.4 /
// 6.1 / 4.4; 30,000: 5.8 / 6.7 / 4.7, 13.0 / 9.8 / 9.8; 100,000: 11.5 / 8.6 / 8.7,
// 45.1 / 29.3 / 29.1. Unaligned arrays go element by element, also in rows.
#include <math.h>

#include "abcd_internal.h"

namespace abcd {
namespace {

constexpr int kMaxGroups = ABCD_ADAM_MAX_GROUPS;
constexpr int kPerThread = 16;
constexpr int64_t kPerBlock = (int64_t)kBlock * kPerThread;

struct AdamArgs {
  float* theta[kMaxGroups];
  const float* g[kMaxGroups];
  float* m[kMaxGroups];
  float* v[kMaxGroups];
  int64_t count[kMaxGroups];
  float step[kMaxGroups];          // lr / (1 - beta1^t)
  int64_t block0[kMaxGroups + 1];  // first workgroup of each group
  int vec[kMaxGroups];             // 16-byte aligned arrays
  int ngroups;
};

typedef float f4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void adam_one(float& th, float g, float& m, float& v, float b1,
                                         float b2, float ic2, float eps, float step) {
  m = b1 * m + (1.0f - b1) * g;
  v = b2 * v + (1.0f - b2) * (g * g);
  th = th - step * m / (sqrtf(v * ic2) + eps);
}

// Up to kRows rows of kBlock vectors E (a float4 or a float) from the arrays'
// start, n of them in all (kFull: all of the rows'): thread t takes vector t of
// each row, so a wave's accesses are consecutive, and every load is issued before
// the first is used (an index past the end is clamped: a load under a condition
// would be waited for where the branches meet).
template <int kRows, typename E, bool kFull = false>
__device__ __forceinline__ void adam_rows(float* th, const float* g, float* m, float* v, int n,
                                          float b1, float b2, float ic2, float eps, float step) {
  constexpr int kLanes = sizeof(E) / sizeof(float);
  E T[kRows], G[kRows], M[kRows], V[kRows];
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int t = q * kBlock + (int)threadIdx.x, i = kFull ? t : min(t, n - 1);
    T[q] = __builtin_nontemporal_load(reinterpret_cast<const E*>(th) + i);
    G[q] = __builtin_nontemporal_load(reinterpret_cast<const E*>(g) + i);
    M[q] = __builtin_nontemporal_load(reinterpret_cast<const E*>(m) + i);
    V[q] = __builtin_nontemporal_load(reinterpret_cast<const E*>(v) + i);
  }
#pragma unroll
  for (int q = 0; q < kRows; ++q) {
    const int i = q * kBlock + (int)threadIdx.x;
    float* const t1 = reinterpret_cast<float*>(&T[q]);
    const float* const g1 = reinterpret_cast<const float*>(&G[q]);
    float* const m1 = reinterpret_cast<float*>(&M[q]);
    float* const v1 = reinterpret_cast<float*>(&V[q]);
#pragma unroll
    for (int e = 0; e < kLanes; ++e) adam_one(t1[e], g1[e], m1[e], v1[e], b1, b2, ic2, eps, step);
    if (kFull || i < n) {
      __builtin_nontemporal_store(T[q], reinterpret_cast<E*>(th) + i);
      __builtin_nontemporal_store(M[q], reinterpret_cast<E*>(m) + i);
      __builtin_nontemporal_store(V[q], reinterpret_cast<E*>(v) + i);
    }
  }
}

__global__ __launch_bounds__(kBlock) void adam_kernel(AdamArgs a, float b1, float b2, float ic2,
                                                      float eps) {
  int gi = 0;
  while (gi + 1 < a.ngroups && (int64_t)blockIdx.x >= a.block0[gi + 1]) ++gi;
  // the workgroup's elements [b0, b0 + cnt)
  const int64_t b0 = ((int64_t)blockIdx.x - a.block0[gi]) * kPerBlock;
  int cnt = (int)min<int64_t>(kPerBlock, a.count[gi] - b0);
  float* th = a.theta[gi] + b0;
  const float* g = a.g[gi] + b0;
  float* m = a.m[gi] + b0;
  float* v = a.v[gi] + b0;
  const float step = a.step[gi];
  if (a.vec[gi] && cnt >= 4) {
    // a group's last workgroup takes as many rows of float4 as it has
    const int n4 = cnt / 4;
    if (n4 == 4 * kBlock)
      adam_rows<4, f4v, true>(th, g, m, v, n4, b1, b2, ic2, eps, step);
    else if (n4 > 3 * kBlock)
      adam_rows<4, f4v>(th, g, m, v, n4, b1, b2, ic2, eps, step);
    else if (n4 > 2 * kBlock)
      adam_rows<3, f4v>(th, g, m, v, n4, b1, b2, ic2, eps, step);
    else if (n4 > kBlock)
      adam_rows<2, f4v>(th, g, m, v, n4, b1, b2, ic2, eps, step);
    else
      adam_rows<1, f4v>(th, g, m, v, n4, b1, b2, ic2, eps, step);
    th += 4 * n4;
    g += 4 * n4;
    m += 4 * n4;
    v += 4 * n4;
    cnt -= 4 * n4;
  }
  // unaligned arrays, or the one to three elements that are left: in turn, four
  // rows at a time
  for (; cnt > kBlock; cnt -= 4 * kBlock) {
    adam_rows<4, float>(th, g, m, v, cnt, b1, b2, ic2, eps, step);
    th += 4 * kBlock;
    g += 4 * kBlock;
    m += 4 * kBlock;
    v += 4 * kBlock;
  }
  if (cnt > 0) adam_rows<1, float>(th, g, m, v, cnt, b1, b2, ic2, eps, step);
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

int32_t launch_adam(const abcd_adam_group* groups, int ngroups, float beta1, float beta2, float eps,
                    int64_t t, hipStream_t stream) {
  AdamArgs a{};
  const double c1 = 1.0 - pow((double)beta1, (double)t);
  const double c2 = 1.0 - pow((double)beta2, (double)t);
  int64_t blocks = 0;
  int used = 0;
  for (int i = 0; i < ngroups; ++i) {
    const abcd_adam_group& gr = groups[i];
    if (gr.count == 0) continue;
    a.theta[used] = gr.param;
    a.g[used] = gr.grad;
    a.m[used] = gr.exp_avg;
    a.v[used] = gr.exp_avg_sq;
    a.count[used] = gr.count;
    a.step[used] = (float)((double)gr.lr / c1);
    a.vec[used] = aligned16(gr.param) && aligned16(gr.grad) && aligned16(gr.exp_avg) &&
                  aligned16(gr.exp_avg_sq);
    a.block0[used] = blocks;
    blocks += (gr.count + kPerBlock - 1) / kPerBlock;
    ++used;
  }
  a.block0[used] = blocks;
  a.ngroups = used;
  if (blocks == 0) return ABCD_OK;
  ABCD_LAUNCH("adam", adam_kernel, blocks, kBlock, 0, stream, a, beta1, beta2,
              (float)(1.0 / c2), eps);
  ABCD_HIP(hipGetLastError());
  return ABCD_OK;
}

}  // namespace abcd
