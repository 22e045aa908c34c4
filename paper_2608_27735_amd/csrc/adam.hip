// adam.hip -- Adam update of the active parameters after a step's backward.
//
// The paper trains the active block with gradient steps and does not name the
// optimizer; the 3DGS line it builds on uses Adam (Kingma and Ba 2015,
// Algorithm 1) with one learning rate per parameter group. One launch updates
// every group in place: a pure HBM stream (parameter, gradient and both
// moments read, parameter and moments written: 28 bytes per element).
// Workgroups are dealt to the groups in proportion to their sizes, 4,096
// elements each; a thread takes four float4s a row of 256 threads apart, all
// sixteen loads issued first, so that each load of a wave covers 1 KB of
// consecutive bytes. (With 16 consecutive elements per thread a wave's load
// touched 64 lines for a quarter of each: 59M elements took 442 us, 3.7 TB/s,
// against 313 us in rows.) Every byte is used once per step and the arrays of
// a large block exceed the caches, so accesses are marked non-temporal: 279
// us, 5.9 TB/s (300,001 x 59 elements 86 against 99 us; no slower down to
// 1,000 x 59). Unaligned arrays and the last, partial workgroup of a group
// go element by element, also in rows.
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

__global__ __launch_bounds__(kBlock) void adam_kernel(AdamArgs a, float b1, float b2, float ic2,
                                                      float eps) {
  int gi = 0;
  while (gi + 1 < a.ngroups && (int64_t)blockIdx.x >= a.block0[gi + 1]) ++gi;
  // the workgroup's elements [b0, b0 + kPerBlock); thread t takes the float4
  // (or, unaligned, the element) t of each row of kBlock, so a wave's accesses
  // are consecutive
  const int64_t b0 = ((int64_t)blockIdx.x - a.block0[gi]) * kPerBlock;
  const int64_t n = a.count[gi];
  float* th = a.theta[gi] + b0;
  const float* g = a.g[gi] + b0;
  float* m = a.m[gi] + b0;
  float* v = a.v[gi] + b0;
  const float step = a.step[gi];
  const int tid = (int)threadIdx.x;
  if (a.vec[gi] && b0 + kPerBlock <= n) {
    f4v T[4], G[4], M[4], V[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = q * kBlock + tid;
      T[q] = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(th) + i);
      G[q] = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(g) + i);
      M[q] = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(m) + i);
      V[q] = __builtin_nontemporal_load(reinterpret_cast<const f4v*>(v) + i);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = q * kBlock + tid;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float t1 = T[q][e], m1 = M[q][e], v1 = V[q][e];
        adam_one(t1, G[q][e], m1, v1, b1, b2, ic2, eps, step);
        T[q][e] = t1;
        M[q][e] = m1;
        V[q][e] = v1;
      }
      __builtin_nontemporal_store(T[q], reinterpret_cast<f4v*>(th) + i);
      __builtin_nontemporal_store(M[q], reinterpret_cast<f4v*>(m) + i);
      __builtin_nontemporal_store(V[q], reinterpret_cast<f4v*>(v) + i);
    }
    return;
  }
  // the last workgroup of a group, or unaligned arrays
  const int cnt = (int)min<int64_t>(kPerBlock, n - b0);
  for (int i = tid; i < cnt; i += kBlock) {
    float t = th[i], mm = m[i], vv = v[i];
    adam_one(t, g[i], mm, vv, b1, b2, ic2, eps, step);
    th[i] = t;
    m[i] = mm;
    v[i] = vv;
  }
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
