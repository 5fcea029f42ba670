// The coarse stage of short sequences inside the fine kernels: with up to 64 cubes a (b, h) a workgroup of 256 threads forms
// the one row (or column) of the coarse matrices that belongs to its block by itself -- 64 x d multiply-adds a
// product -- while its list and its first tiles are on their way, instead of waiting for a launch of its own that
// hardly fills a compute unit.  fp32 products and sums, in a fixed order.  Bound by latency: the rows that are
// summed are requested before their weights are formed (64 cubes, d = 128, top-1: forward 21.5 -> 15.7 us; 18.7 with a launch for the
// coarse stage).  The chunks of the logits' products are not: at d = 128 those rows leave no registers and they come in eight trips.
// Forwards of 12 to 64 cubes, up to 256 blocks (d = 64: 512), 0.73 to 0.93 of the time; 32 cubes, 2 heads, d = 64, top-8 17.0 ->
// 13.4 us.  In launches of several generations every one of them would pay what one launch costs.
#pragma once
#include <cstddef>

#include "coarse_row.h"
#include "vsa_kernels.h"

namespace vsa {

constexpr int kSmallCubes = 64;
constexpr int kSmallThreads = 256;

template <int D>
struct alignas(16) SmallCoarse {
  static constexpr int PER_ROW = D / 4, PARTS = kSmallThreads / PER_ROW;  // threads a row of the sums, partial sums
  float w[2][kSmallCubes];  // weights of the sums below
  float sum[2][D];
  float part[2][PARTS][D];
};
// (rows of `sum` and `part` are read and written 16 bytes at a time)
template <int D>
constexpr bool kSmallRowsAligned = alignof(SmallCoarse<D>) % 16 == 0 && offsetof(SmallCoarse<D>, sum) % 16 == 0 &&
                                   offsetof(SmallCoarse<D>, part) % 16 == 0;
static_assert(kSmallRowsAligned<64> && kSmallRowsAligned<128>, "16-byte accesses");

__device__ __forceinline__ float dot4(const float4& a, const float4& b, float s) {
  return fmaf(a.w, b.w, fmaf(a.z, b.z, fmaf(a.y, b.y, fmaf(a.x, b.x, s))));
}

// x . rows[n] of thread 4n + p, in every lane of the four (n < Nc; a row past the end repeats the last)
template <int D>
__device__ __forceinline__ float small_dot(const float* __restrict__ x, const float* __restrict__ rows, int Nc, int tid) {
  const int n = min(tid >> 2, Nc - 1), p = tid & 3;
  const float4 *a = (const float4*)x + p, *b = (const float4*)(rows + n * D) + p;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < D / 16; ++i) s = dot4(a[4 * i], b[4 * i], s);
  s += __shfl_xor(s, 1);
  s += __shfl_xor(s, 2);
  return s;
}

// Sums over n < Nc of w[n] rows[n][e]: a thread takes four columns of every PARTS-th row, which it requests well before the
// weights are known (nothing in these kernels hides the trip but that).
template <int D>
struct SmallRows {
  using L = SmallCoarse<D>;
  static constexpr int ROWS = kSmallCubes / L::PARTS;
  float4 x[ROWS];
  __device__ __forceinline__ void request(const float* __restrict__ rows, int Nc, int tid) {
#pragma unroll
    for (int i = 0; i < ROWS; ++i) x[i] = *(const float4*)(rows + min(tid / L::PER_ROW + i * L::PARTS, Nc - 1) * D + tid % L::PER_ROW * 4);
  }
  __device__ __forceinline__ void weigh(const float* w, float (*part)[D], int Nc, int tid) const {
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int i = 0; i < ROWS; ++i) {
      const int n = tid / L::PER_ROW + i * L::PARTS;
      if (n < Nc) {
        const float a = w[n];
        s.x = fmaf(a, x[i].x, s.x); s.y = fmaf(a, x[i].y, s.y); s.z = fmaf(a, x[i].z, s.z); s.w = fmaf(a, x[i].w, s.w);
      }
    }
    *(float4*)&part[tid / L::PER_ROW][tid % L::PER_ROW * 4] = s;
  }
};
template <int D>
__device__ __forceinline__ float small_sum(const float (*part)[D], int e) {
  float s = part[0][e];
#pragma unroll
  for (int i = 1; i < SmallCoarse<D>::PARTS; ++i) s += part[i][e];
  return s;
}

// The coarse stage of query cube `own`: l.sum[0] = O_c, `list` the K cubes it selects; both, and its log-sum-exp, go to memory
// too.  In two steps of all 256 threads, each ending with a barrier: the copies that the list names are issued in between.
template <int D>
__device__ __forceinline__ void small_select(SmallCoarse<D>& l, int32_t* list, int Nc, int K, int own, long long first,
                                             const SmallForwardArgs& a, SmallRows<D>& v, int tid) {
  v.request(a.vc + first * D, Nc, tid);
  const float s = small_dot<D>(a.qc + (first + own) * D, a.kc + first * D, Nc, tid);
  if ((tid & 3) == 0) l.w[0][tid >> 2] = a.scale * s;
  if (tid < kSmallCubes) list[tid] = 0;  // (logits that are not numbers may select fewer)
  __syncthreads();
  if (tid < 64) {
    coarse_row<1>(l.w[0], Nc, K, a.lse_c ? a.lse_c + first + own : nullptr, list, 1, tid);
    __builtin_amdgcn_wave_barrier();  // (a wavefront's LDS accesses stay in order)
    if (tid < K) a.idx[(first + own) * K + tid] = list[tid];
  }
  __syncthreads();
}
template <int D>
__device__ __forceinline__ void small_output(SmallCoarse<D>& l, int Nc, int own, long long first, const SmallForwardArgs& a,
                                             const SmallRows<D>& v, int tid) {
  v.weigh(l.w[0], l.part[0], Nc, tid);
  __syncthreads();
  if (tid < D) {
    const float o = small_sum<D>(l.part[0], tid);
    l.sum[0][tid] = o;
    a.oc[(first + own) * D + tid] = o;
  }
  __syncthreads();
}

// The coarse backward of one query cube (KEYS false: sum[0] = dQc of the cube) or key cube (KEYS true: sum[0] = dKc, sum[1] =
// dVc) `own` of the head that starts at cube `first`:  A = exp(scale Qc Kc^T - lse), dS = A (dOc Vc^T - dot),
// dQc = scale dS Kc, dKc = scale dS^T Qc, dVc = A^T dOc.  All 256 threads; ends with a barrier.
template <int D, bool KEYS>
__device__ __forceinline__ void small_coarse_bwd(SmallCoarse<D>& l, int Nc, int own, long long first, float scale,
                                                 const float* __restrict__ qc, const float* __restrict__ kc,
                                                 const float* __restrict__ vc, const float* __restrict__ doc,
                                                 const float* __restrict__ lse_c, const float* __restrict__ dot, int tid) {
  const float *x = (KEYS ? kc : qc) + (first + own) * D, *y = (KEYS ? vc : doc) + (first + own) * D;
  const float *p = (KEYS ? qc : kc) + first * D, *r = (KEYS ? doc : vc) + first * D;
  const int n = tid >> 2;
  const long long row = first + (KEYS ? min(n, Nc - 1) : own);  // the query cube the row terms belong to
  const float lse = lse_c[row], dt = dot[row];
  SmallRows<D> rp, rr;
  rp.request(p, Nc, tid);
  if (KEYS) rr.request(r, Nc, tid);
  const float s = small_dot<D>(x, p, Nc, tid), da = small_dot<D>(y, r, Nc, tid);
  if ((tid & 3) == 0) {
    const float a = fast_exp2((scale * s - lse) * kLog2e);
    l.w[0][n] = a * (da - dt);
    l.w[1][n] = a;
  }
  __syncthreads();
  rp.weigh(l.w[0], l.part[0], Nc, tid);
  if (KEYS) rr.weigh(l.w[1], l.part[1], Nc, tid);
  __syncthreads();
  if (tid < D) {
    l.sum[0][tid] = scale * small_sum<D>(l.part[0], tid);
    if (KEYS) l.sum[1][tid] = small_sum<D>(l.part[1], tid);
  }
  __syncthreads();
}

}  // namespace vsa
