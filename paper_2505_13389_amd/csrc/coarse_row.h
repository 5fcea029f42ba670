// One row of the coarse stage by one wavefront: log-sum-exp, probabilities and the top-K list (Sec. 2.2; Sec. 2.4 fuses
// softmax, top-K and mask->index conversion).
#pragma once
#include "vsa_common.h"

namespace vsa {

__device__ __forceinline__ uint32_t sortable_key(float s) {
  uint32_t b = __float_as_uint(s);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
// Reductions over the 64 lanes of a wavefront, result in every lane: four data-parallel-primitive
// steps inside each row of 16 lanes (quad swaps, half-row mirror, row mirror: register-to-register,
// no trip through the LDS permute path), then the four row results are combined through scalar
// registers.  The order of the additions is fixed.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_move(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce_bits(uint32_t x, Op op) {
  x = op(x, dpp_move<0xB1>(x));   // quad_perm [1,0,3,2]
  x = op(x, dpp_move<0x4E>(x));   // quad_perm [2,3,0,1]
  x = op(x, dpp_move<0x141>(x));  // row_half_mirror
  x = op(x, dpp_move<0x140>(x));  // row_mirror
  const uint32_t a = __builtin_amdgcn_readlane(x, 0), b = __builtin_amdgcn_readlane(x, 16);
  const uint32_t c = __builtin_amdgcn_readlane(x, 32), d = __builtin_amdgcn_readlane(x, 48);
  return op(op(a, b), op(c, d));
}
__device__ __forceinline__ float wave_max(float x) {
  return __uint_as_float(wave_reduce_bits(__float_as_uint(x), [](uint32_t p, uint32_t q) {
    return __float_as_uint(fmaxf(__uint_as_float(p), __uint_as_float(q))); }));
}
__device__ __forceinline__ float wave_sum(float x) {
  return __uint_as_float(wave_reduce_bits(__float_as_uint(x), [](uint32_t p, uint32_t q) {
    return __float_as_uint(__uint_as_float(p) + __uint_as_float(q)); }));
}
__device__ __forceinline__ uint32_t wave_umin(uint32_t x) { return wave_reduce_bits(x, [](uint32_t p, uint32_t q) { return min(p, q); }); }
__device__ __forceinline__ uint32_t wave_umax(uint32_t x) { return wave_reduce_bits(x, [](uint32_t p, uint32_t q) { return max(p, q); }); }

// One row of the score matrix worked off by one wavefront; lane j holds logits j, j+64, ... (NCH per
// lane).  `srow` may point into global memory or into LDS.  Writes the row's probabilities back over
// the logits, its log-sum-exp to *lse_out (if given) and, with emit_idx, the ascending list of its K
// largest logits (ties to the lower index) to `out`.
// `kcnt` (optional): valid tokens per key cube; a key cube with none is dead -- its logit counts as -inf,
// so it gets probability 0 and, K not exceeding the number of live key cubes, is never selected.
template <int NCH>
__device__ __forceinline__ void coarse_row(float* srow, int Nc, int K, float* lse_out, int32_t* out, int emit_idx,
                                           int lane, const int32_t* __restrict__ kcnt = nullptr) {
  const int nch = (Nc + 63) / 64;
  float s[NCH];
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) {
    const int j = ch * 64 + lane;
    s[ch] = (j < Nc && (!kcnt || kcnt[j] > 0)) ? srow[j] + 0.f : -INFINITY;
  }

  float m = -INFINITY;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) m = fmaxf(m, s[ch]);
  m = wave_max(m);
  float l = 0.f;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch) l += fast_exp2((s[ch] - m) * kLog2e);
  l = wave_sum(l);
  const float lse = m + fast_log2(l) * kLn2;
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
    if (ch * 64 + lane < Nc) srow[ch * 64 + lane] = fast_exp2((s[ch] - lse) * kLog2e);
  if (lane == 0 && lse_out) *lse_out = lse;

  if (emit_idx) {
    // Order-preserving integer keys; lanes beyond Nc hold key 0 and never count (every threshold
    // tried is >= 1).  T = the K-th largest key, by bisection of the key range [min, max]:
    // cnt(x) = #(key >= x) is non-increasing, cnt(lo) >= K > cnt(hi) throughout.  The search stops
    // as soon as a threshold separates exactly K keys (all counts are wave-uniform, so is the
    // exit): about log2(range / gap at rank K) steps on spread-out logits, 32 at most.
    uint32_t key[NCH];
    uint32_t kmin = 0xffffffffu, kmax = 0u;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      const bool valid = ch * 64 + lane < Nc;
      key[ch] = valid ? sortable_key(s[ch]) : 0u;
      if (valid) kmin = min(kmin, key[ch]);
      kmax = max(kmax, key[ch]);
    }
    kmin = wave_umin(kmin);
    kmax = wave_umax(kmax);
    auto count_ge = [&](uint32_t x) {
      int cnt = 0;
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
        if (ch < nch) cnt += __popcll(__ballot(key[ch] >= x));
      return cnt;
    };
    unsigned long long lo = kmin, hi = (unsigned long long)kmax + 1ull;
    uint32_t T = (uint32_t)lo;
    while (hi - lo > 1ull) {
      const uint32_t mid = (uint32_t)((lo + hi) >> 1);
      const int cnt = count_ge(mid);
      if (cnt >= K) {
        lo = mid;
        T = mid;
        if (cnt == K) break;  // exactly K keys at or above mid: they are the set
      } else {
        hi = mid;
      }
    }
    int n_gt = 0;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
      if (ch < nch) n_gt += __popcll(__ballot(key[ch] > T));
    const int need = K - n_gt;  // entries equal to the threshold still to take, lowest index first
    int eq_seen = 0, base = 0;
    const uint64_t lt = (1ull << lane) - 1ull;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch)
      if (ch < nch) {
        const bool eq = (key[ch] == T) && (ch * 64 + lane < Nc);
        const uint64_t beq = __ballot(eq);
        const bool take = (key[ch] > T) || (eq && (eq_seen + (int)__popcll(beq & lt) < need));
        eq_seen += __popcll(beq);
        const uint64_t bsel = __ballot(take);
        const int pos = base + __popcll(bsel & lt);
        if (take && pos < K) out[pos] = ch * 64 + lane;  // (pos < K always holds for finite logits)
        base += __popcll(bsel);
      }
  }
}

}  // namespace vsa
