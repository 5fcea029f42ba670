// The coarse stage of short sequences inside the fine kernels: with up to 64 cubes a (b, h) a workgroup of 256 threads forms
// the one row (or column) of the coarse matrices that belongs to its block by itself -- 64 x d multiply-adds a
// product -- while its list and its first tiles are on their way, instead of waiting for a launch of its own that
// hardly fills a compute unit.  fp32 products and sums, in a fixed order.
#pragma once
#include "vsa_common.h"

namespace vsa {

constexpr int kSmallCubes = 64;
constexpr int kSmallThreads = 256;

template <int D>
struct SmallCoarse {
  float w[2][kSmallCubes];             // weights of the sums below
  float sum[2][D];
  float part[2][kSmallThreads];
};

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

// sum over n < Nc of w[n] rows[n][e], e = tid % D, the partial sum of n = tid / D, tid / D + 256 / D, ...
template <int D>
__device__ __forceinline__ float small_part(const float* w, const float* __restrict__ rows, int Nc, int tid) {
  const int e = tid % D;
  float s = 0.f;
#pragma unroll 8
  for (int n = tid / D; n < Nc; n += kSmallThreads / D) s = fmaf(w[n], rows[n * D + e], s);
  return s;
}
template <int D>
__device__ __forceinline__ float small_sum(const float* part, int e) {
  float s = part[e];
#pragma unroll
  for (int i = 1; i < kSmallThreads / D; ++i) s += part[i * D + e];
  return s;
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
  const float s = small_dot<D>(x, p, Nc, tid), da = small_dot<D>(y, r, Nc, tid);
  if ((tid & 3) == 0) {
    const float a = fast_exp2((scale * s - lse) * kLog2e);
    l.w[0][n] = a * (da - dt);
    l.w[1][n] = a;
  }
  __syncthreads();
  l.part[0][tid] = small_part<D>(l.w[0], p, Nc, tid);
  if (KEYS) l.part[1][tid] = small_part<D>(l.w[1], r, Nc, tid);
  __syncthreads();
  if (tid < D) {
    l.sum[0][tid] = scale * small_sum<D>(l.part[0], tid);
    if (KEYS) l.sum[1][tid] = small_sum<D>(l.part[1], tid);
  }
  __syncthreads();
}

}  // namespace vsa
