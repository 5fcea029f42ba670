// Small backward steps: the elementwise preprocess, the coarse-stage backward (fp32) and the
// transposed block map.  The gradient formulas are the chain rule through Sec. 2.2's gated sum,
// coarse softmax attention and mean pooling.
#include "gemm32_tile.h"
#include "list_rules.h"
#include "vsa_kernels.h"

namespace vsa {

// ---------------------------------------------------------------------------------------------
// Up to three independent problems of the same shape run as one launch (blockIdx.z = problem *
// batch + batch index): the small coarse-stage products do not fill the chip one at a time.
struct GemmOperands {
  const float* a; long long sab; int sam, sak;
  const float* b; long long sbb; int sbk, sbn;
  float* c; long long scb; float alpha;
};
struct GemmSet { GemmOperands p[3]; };

__global__ __launch_bounds__(256) void k_gemm32(int M, int N, int Kd, int batch, GemmSet set) {
  __shared__ __attribute__((aligned(16))) float As[64][36];
  __shared__ __attribute__((aligned(16))) float Bs[64][36];
  const GemmOperands& g = set.p[blockIdx.z / batch];
  const int b = blockIdx.z % batch, m0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  const int sam = g.sam, sak = g.sak, sbk = g.sbk, sbn = g.sbn;
  const float* ab = g.a + b * g.sab + (long long)m0 * sam;
  const float* bb = g.b + b * g.sbb + (long long)n0 * sbn;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1, l32 = lane & 31, h = lane >> 5;
  f32x16g acc;
  gemm_tile_global(As, Bs, ab, sam, sak, M - m0, bb, sbn, sbk, N - n0, Kd, tid, acc);
  float* cb = g.c + b * g.scb;
  const float alpha = g.alpha;
  const int n = n0 + wn * 32 + l32;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int m = m0 + wm * 32 + 8 * (i / 4) + 4 * h + (i % 4);
    if (m < M && n < N) cb[(long long)m * N + n] = alpha * acc[i];
  }
}

static GemmOperands gemm_operands(float alpha, const float* a, long long sab, int sam, int sak, const float* b,
                                  long long sbb, int sbk, int sbn, float* c, long long scb) {
  GemmOperands o;
  o.a = a; o.sab = sab; o.sam = sam; o.sak = sak;
  o.b = b; o.sbb = sbb; o.sbk = sbk; o.sbn = sbn;
  o.c = c; o.scb = scb; o.alpha = alpha;
  return o;
}
static hipError_t gemm32_set(int nprob, int batch, int M, int N, int Kd, const GemmSet& set, hipStream_t s) {
  dim3 grid((N + 63) / 64, (M + 63) / 64, batch * nprob);
  k_gemm32<<<grid, 256, 0, s>>>(M, N, Kd, batch, set);
  return hipGetLastError();
}
hipError_t gemm32(int batch, int M, int N, int Kd, float alpha, const float* a, long long sab, int sam, int sak,
                  const float* b, long long sbb, int sbk, int sbn, float* c, long long scb, hipStream_t s) {
  GemmSet set;
  set.p[0] = set.p[1] = set.p[2] = gemm_operands(alpha, a, sab, sam, sak, b, sbb, sbk, sbn, c, scb);
  return gemm32_set(1, batch, M, N, Kd, set, s);
}

// Row-wise softmax backward on the coarse score matrix, in place:
//   sc  holds scale*Qc.Kc^T  -> becomes Ac  = exp(sc - lse_c[row])
//   dsc holds dOc.Vc^T (dAc) -> becomes dSc = Ac * (dAc - sum_j Ac*dAc)
// One wavefront per row, fixed reduction order.
__global__ __launch_bounds__(256) void k_coarse_softmax_bwd(int rows, int Nc, const float* __restrict__ lse_c,
                                                            float* __restrict__ sc, float* __restrict__ dsc,
                                                            const int32_t* __restrict__ kcnt) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= rows) return;
  float* s = sc + (long long)row * Nc;
  float* ds = dsc + (long long)row * Nc;
  const float lse = lse_c[row];
  float dot = 0.f;
  for (int j = lane; j < Nc; j += 64) {
    const float a = (!kcnt || kcnt[j] > 0) ? fast_exp2((s[j] - lse) * kLog2e) : 0.f;  // (a dead key cube: no weight)
    s[j] = a;
    dot = fmaf(a, ds[j], dot);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) dot += __shfl_xor(dot, o);
  for (int j = lane; j < Nc; j += 64) ds[j] = s[j] * (ds[j] - dot);
}

// The whole coarse backward in ONE launch.  With dot[q] = dOc[q] . Oc[q] (= sum_j Ac dAc, left by the preprocess pass)
// nothing couples the columns of a row any more, so every product can be formed where it is used, from either side:
//   query side, 16 query cubes:  A, dS [16 x Nc] -> dQc = scale dS Kc
//   key side, 16 key cubes:      A^T, dS^T [16 x Nc] -> dVc = A^T dOc, dKc = scale dS^T Qc
// with A = exp(scale Qc Kc^T - lse), dS = A (dOc Vc^T - dot): nothing but the gradients goes to memory.  One
// workgroup of 16 wavefronts per 16 cubes and side walks the other side in chunks of 256 cubes: one 16 x 16 block of both
// products per wavefront (v_mfma_f32_16x16x4_f32: fp32 products and sums), A and dS into LDS, then their products with
// the other side's tensors, 16 columns per wavefront, the wavefronts left over splitting the contraction (partial
// sums added in a fixed order).  Operands come straight from L2 (see k_coarse_fused for the relabelling of k).
// Bound by latency (two dependent chains of L2 loads and matrix instructions per chunk).  Measured against three
// launches through [Nc x Nc] matrices in memory, us: 32 cubes, 2 heads, d = 64: 14.8 -> 7.4 (train step 56 -> 49); 64 cubes,
// 12 heads, d = 128: 19.7 -> 12.1; 280 cubes, 5 heads: 33 -> 26; 256 cubes, 16 heads, d = 64: 31 -> 24; 256 cubes, 12 heads,
// d = 128: 38 -> 40; 32 heads: 56 -> 79; 480 cubes, 16 heads: 100 -> 150; 624, 12 heads: 117 -> 178 -- the staged
// 64 x 64 tiles of the launches read every operand four times less often, which is what counts once the chip is full.
typedef float f32x4c __attribute__((ext_vector_type(4)));
constexpr long long kCoarseBwdOneMax = 80ll << 20;  // multiply-adds of one product, all heads
template <int D>
__global__ __launch_bounds__(1024) void k_coarse_bwd_one(int Nc, float scale, const float* __restrict__ qc,
                                                         const float* __restrict__ kc, const float* __restrict__ vc,
                                                         const float* __restrict__ doc, const float* __restrict__ lse_c,
                                                         const float* __restrict__ dot, float* __restrict__ dqc,
                                                         float* __restrict__ dkc, float* __restrict__ dvc) {
  constexpr int R = 16, CH = 256, ROW = CH + 4, OWN = D + 4;  // (rows start 4 banks apart)
  constexpr int CB = D / 16;  // 16-column blocks of an output
  __shared__ __attribute__((aligned(16))) float A[R * ROW], G[R * ROW];
  __shared__ __attribute__((aligned(16))) float X[R * OWN], Y[R * OWN];
  __shared__ __attribute__((aligned(16))) float part[16][64][4];
  const int blocks = (Nc + R - 1) / R;
  const bool keys = blockIdx.x & 1;  // which side
  const int m0 = (int)((blockIdx.x >> 1) % blocks) * R;
  const long long bh = (blockIdx.x >> 1) / blocks, first = bh * Nc;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const int rows_valid = min(R, Nc - m0);
  const float *own_x = (keys ? kc : qc) + (first + m0) * D, *own_y = (keys ? vc : doc) + (first + m0) * D;
  const float *oth_p = (keys ? qc : kc) + first * D, *oth_r = (keys ? doc : vc) + first * D;
  for (int i = tid; i < R * D; i += 1024) {
    const int r = i / D, e = i % D;
    X[r * OWN + e] = r < rows_valid ? own_x[i] : 0.f;
    Y[r * OWN + e] = r < rows_valid ? own_y[i] : 0.f;
  }
  // the outputs' blocks: query side dQc, 16 / CB wavefronts a block; key side the first 8 wavefronts dKc, the last dVc
  const int per_out = keys ? 8 : 16, ksplit = per_out / CB;
  const int ow = wave % per_out, cb = ow % CB, ks = ow / CB;
  const bool second = wave >= per_out;
  const float* M = second ? A : G;
  const float* col = (second ? oth_r : oth_p) + cb * 16 + l16;
  f32x4c out = {0.f, 0.f, 0.f, 0.f};
  for (int c0 = 0; c0 < Nc; c0 += CH) {
    __syncthreads();  // own rows are there; A and G of the chunk before have been read
    const int n = c0 + wave * 16 + l16;
    if (c0 + wave * 16 < ((Nc + 15) & ~15)) {
      const long long at = (long long)min(n, Nc - 1) * D + 4 * kq;
      f32x4c s = {0.f, 0.f, 0.f, 0.f}, da = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int k0 = 0; k0 < D; k0 += 16) {
        const float4 x = *(const float4*)&X[l16 * OWN + k0 + 4 * kq], y = *(const float4*)&Y[l16 * OWN + k0 + 4 * kq];
        const float4 p = *(const float4*)(oth_p + at + k0), r = *(const float4*)(oth_r + at + k0);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, p.x, s, 0, 0, 0);
        da = __builtin_amdgcn_mfma_f32_16x16x4f32(y.x, r.x, da, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, p.y, s, 0, 0, 0);
        da = __builtin_amdgcn_mfma_f32_16x16x4f32(y.y, r.y, da, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(x.z, p.z, s, 0, 0, 0);
        da = __builtin_amdgcn_mfma_f32_16x16x4f32(y.z, r.z, da, 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x4f32(x.w, p.w, s, 0, 0, 0);
        da = __builtin_amdgcn_mfma_f32_16x16x4f32(y.w, r.w, da, 0, 0, 0);
      }
      // lane: rows 4*kq + i, column n; the row terms belong to the query cube
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int m = 4 * kq + i;
        const long long qrow = first + (keys ? min(n, Nc - 1) : min(m0 + m, Nc - 1));
        const float a = n < Nc ? fast_exp2((scale * s[i] - lse_c[qrow]) * kLog2e) : 0.f;
        A[m * ROW + wave * 16 + l16] = a;
        G[m * ROW + wave * 16 + l16] = n < Nc ? a * (da[i] - dot[qrow]) : 0.f;  // (chosen, not multiplied: Inf stays where it is)
      }
    }
    __syncthreads();
    const int kend = min(CH, ((Nc + 15) & ~15) - c0);
    for (int k0 = ks * 16; k0 < kend; k0 += 16 * ksplit) {
      const float4 a = *(const float4*)&M[l16 * ROW + k0 + 4 * kq];
      const int kk = c0 + k0 + 4 * kq;
      float b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float x = col[(long long)min(kk + j, Nc - 1) * D];
        b[j] = kk + j < Nc ? x : 0.f;
      }
      out = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b[0], out, 0, 0, 0);
      out = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b[1], out, 0, 0, 0);
      out = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b[2], out, 0, 0, 0);
      out = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b[3], out, 0, 0, 0);
    }
  }
  *(float4*)part[wave][lane] = make_float4(out[0], out[1], out[2], out[3]);
  __syncthreads();
  if (ks == 0) {
    float sum[4] = {0.f, 0.f, 0.f, 0.f};
    for (int o = 0; o < ksplit; ++o) {
      const float4 x = *(const float4*)part[wave + o * CB][lane];
      sum[0] += x.x; sum[1] += x.y; sum[2] += x.z; sum[3] += x.w;
    }
    float* dst = second ? dvc : (keys ? dkc : dqc);
    const float mul = second ? 1.f : scale;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int m = 4 * kq + i;
      if (m < rows_valid) dst[(first + m0 + m) * D + cb * 16 + l16] = mul * sum[i];
    }
  }
}

// Coarse backward: dVc = Ac^T dOc, dQc = scale dSc Kc, dKc = scale dSc^T Qc, for Nq query cubes and Nk
// key cubes (see launch_coarse).  `ac` and `dsc` are [BH,Nq,Nk] scratch, `dot` as the preprocess pass leaves it.
hipError_t launch_coarse_bwd(int BH, int Nq, int Nk, int d, float scale, const float* qc, const float* kc,
                             const float* vc, const float* lse_c, const float* doc, const float* dot, float* ac,
                             float* dsc, float* dqc, float* dkc, float* dvc, const int32_t* kcnt, hipStream_t s) {
  if (Nq == Nk && !kcnt && (long long)BH * Nq * Nk * d <= kCoarseBwdOneMax) {
    const unsigned grid = 2u * (unsigned)(BH * ((Nq + 15) / 16));
    if (d == 128) k_coarse_bwd_one<128><<<grid, 1024, 0, s>>>(Nq, scale, qc, kc, vc, doc, lse_c, dot, dqc, dkc, dvc);
    else k_coarse_bwd_one<64><<<grid, 1024, 0, s>>>(Nq, scale, qc, kc, vc, doc, lse_c, dot, dqc, dkc, dvc);
    return hipGetLastError();
  }
  const long long sq = (long long)Nq * d, sk = (long long)Nk * d, ss = (long long)Nq * Nk;
  hipError_t e;
  GemmSet set;
  // one launch: sc = scale * Qc Kc^T ; dAc = dOc Vc^T
  set.p[0] = gemm_operands(scale, qc, sq, d, 1, kc, sk, 1, d, ac, ss);
  set.p[1] = set.p[2] = gemm_operands(1.f, doc, sq, d, 1, vc, sk, 1, d, dsc, ss);
  if ((e = gemm32_set(2, BH, Nq, Nk, d, set, s)) != hipSuccess) return e;
  k_coarse_softmax_bwd<<<(BH * Nq + 3) / 4, 256, 0, s>>>(BH * Nq, Nk, lse_c, ac, dsc, kcnt);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  // dVc[j][e] = sum_c Ac[c][j] dOc[c][e] ; dQc[c][e] = scale sum_j dSc[c][j] Kc[j][e] ;
  // dKc[j][e] = scale sum_c dSc[c][j] Qc[c][e]: one launch when the three have the same shape
  GemmOperands dv_ = gemm_operands(1.f, ac, ss, 1, Nk, doc, sq, d, 1, dvc, sk);
  GemmOperands dq_ = gemm_operands(scale, dsc, ss, Nk, 1, kc, sk, d, 1, dqc, sq);
  GemmOperands dk_ = gemm_operands(scale, dsc, ss, 1, Nk, qc, sq, d, 1, dkc, sk);
  if (Nq == Nk) {
    set.p[0] = dv_, set.p[1] = dq_, set.p[2] = dk_;
    return gemm32_set(3, BH, Nq, d, Nq, set, s);
  }
  set.p[0] = dv_, set.p[1] = set.p[2] = dk_;
  if ((e = gemm32_set(2, BH, Nk, d, Nq, set, s)) != hipSuccess) return e;
  set.p[0] = set.p[1] = set.p[2] = dq_;
  return gemm32_set(1, BH, Nq, d, Nk, set, s);
}

// ---------------------------------------------------------------------------------------------
// Transposed block map (CSR): for every key cube j the ascending list of the query cubes that
// selected it.  Built through a bit matrix so that every step is parallel over the whole grid and
// the result does not depend on any execution order (no float or ordering-sensitive atomics; the
// only atomic is a bitwise OR in LDS):
//   bits[bh][j][w], bit q%32 of word q/32  <-  1 for every (q, j) in the index list
//   row_ptr = exclusive scan over j of popcount(row j)        (a wavefront per row, then one
//                                                               workgroup per (b, h) for the scan)
//   col     = positions of the set bits of row j, ascending   (one wavefront per (b, h, j))
constexpr int kMaxCubes = 4096;  // = 4 entries per thread of the 1024-thread scan

// One workgroup per (b, h, word column w): the 32 query cubes 32w .. 32w+31 OR their bits into a
// per-key word held in LDS, then every key row gets its word w written exactly once (no global
// atomics, nothing to clear beforehand).
// (Nq query cubes, Nrows key rows: Nrows = Nq, or 4 Nq when the lists name key cubes of 16 tokens)
__global__ __launch_bounds__(256) void k_map_bits(int Nq, int Nrows, int K, int W32, const int32_t* __restrict__ idx,
                                                  uint32_t* __restrict__ bits) {
  __shared__ uint32_t word[kMaxCubes];
  const int w = blockIdx.x % W32, tid = threadIdx.x;
  const long long bh = blockIdx.x / W32;
  for (int j = tid; j < Nrows; j += 256) word[j] = 0u;
  __syncthreads();
  const int q_lo = w * 32, nq = min(32, Nq - q_lo);
  const int32_t* my = idx + (bh * Nq + q_lo) * (long long)K;
  for (int e = tid; e < nq * K; e += 256) {
    const int c = my[e];
    if (map_takes(c, Nrows)) atomicOr(&word[c], 1u << (e / K));  // (a caller-supplied list is not trusted)
  }
  __syncthreads();
  for (int j = tid; j < Nrows; j += 256) bits[(bh * Nrows + j) * W32 + w] = word[j];
}

// in-degree of every key cube: one wavefront per (b, h, j), written to row_ptr[bh][j] (scanned next)
__global__ __launch_bounds__(256) void k_map_degree(int Nc, int W32, long long rows, const uint32_t* __restrict__ bits,
                                                    int32_t* __restrict__ row_ptr) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);  // bh * Nc + j
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const uint32_t* r = bits + row * W32;
  int c = 0;
  for (int w = lane; w < W32; w += 64) c += __popc(r[w]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if (lane == 0) row_ptr[(row / Nc) * (Nc + 1) + row % Nc] = c;
}

// Exclusive scan over PT * NT values, PT consecutive ones per thread of an NT-thread workgroup:
// v[i] is replaced by the sum of everything before it; returns the grand total.
template <int PT, int NT>
__device__ __forceinline__ int block_scan(int* v, int* wsum, int tid) {
  const int lane = tid & 63, wave = tid >> 6;
  int sum = 0;
#pragma unroll
  for (int i = 0; i < PT; ++i) sum += v[i];
  int incl = sum;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  __syncthreads();  // wsum may still be read by a previous call
  if (lane == 63) wsum[wave] = incl;
  __syncthreads();
  int base = 0, total = 0;
  for (int w = 0; w < NT / 64; ++w) {
    if (w < wave) base += wsum[w];
    total += wsum[w];
  }
  int run = base + incl - sum;
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    const int t = v[i];
    v[i] = run;
    run += t;
  }
  return total;
}

// sum of one value per thread over an NT-thread workgroup, returned to every thread
template <int NT>
__device__ __forceinline__ int block_sum(int x, int* wsum, int tid) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  __syncthreads();  // wsum may still be read by a previous call
  if ((tid & 63) == 0) wsum[tid >> 6] = x;
  __syncthreads();
  int total = 0;
  for (int w = 0; w < NT / 64; ++w) total += wsum[w];
  return total;
}

// exclusive scan of the in-degrees of one (b, h), in place; row_ptr[Nc] = total.  Also cuts the
// work of the dK/dV pass into items and sorts them by length, longest first (counting sort; the
// order among equal lengths is whatever the LDS atomics give, it only decides which workgroup
// starts when).  An item is a key cube's whole list, or -- for a list longer than the split length
// -- one of ceil(deg / length) nearly equal runs of it; each run of such a SPLIT list accumulates
// fp32 partial dK, dV into a numbered slot, summed in slot order by the last run to arrive, so the
// result does not depend on which workgroup ran when.  The split length of a (b, h) is the smallest
// one, not below `seg_min`, at which the runs of all its long lists fit into the `cap` slots the
// slot buffer holds per (b, h): it depends on the in-degrees alone.
//   order: one 16-byte descriptor (key cube, begin, end of the run in col, run_word or -1) per dK/dV workgroup, Nc + cap of them
//          per (b, h); unused ones carry key cube -1
//   split: per (b, h) cap/2 + 1 descriptors: [0] is not used, then (key cube, first slot, number of slots, runs arrived: 0) per
//          split list, in cube order
// (the body, for the NT threads of one workgroup: thread `tid` owns cubes PT*tid .. PT*tid+PT-1, Nc <= PT*NT, whose
// in-degrees it passes in `deg`; `v` returns where their lists begin.  wsum[NT/64] and hist[PT*NT] are
// LDS scratch: bucket x of hist counts the items that go by the length Nc - x (the last bucket also takes what
// lies beyond it), then holds the next free slot of the bucket)
template <int PT, int NT>
__device__ __forceinline__ void map_scan_body(int Nc, int seg_min, int cap, int bh, int tid, const int (&deg)[PT], int (&v)[PT],
                                              int32_t* __restrict__ row_ptr, int32_t* __restrict__ order,
                                              int32_t* __restrict__ split, int* wsum, int* hist) {
  int32_t* rp = row_ptr + (long long)bh * (Nc + 1);
  const int j0 = tid * PT;
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    v[i] = deg[i];
    hist[j0 + i] = 0;
  }
  const int total = block_scan<PT, NT>(v, wsum, tid);  // (its barriers also cover the clearing of hist)
#pragma unroll
  for (int i = 0; i < PT; ++i)
    if (j0 + i < Nc) rp[j0 + i] = v[i];
  if (tid == 0) rp[Nc] = total;

  // the split length: slots_wanted is non-increasing in it and 0 at Nc (no list is longer than Nc)
  auto wanted = [&](int len) {
    int w = 0;
#pragma unroll
    for (int i = 0; i < PT; ++i) w += slots_wanted(deg[i], len);
    return block_sum<NT>(w, wsum, tid);
  };
  int seg = seg_min;
  if (wanted(seg) > cap) {
    int lo = seg, hi = max(Nc, seg + 1);  // wanted(lo) > cap >= wanted(hi)
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (wanted(mid) <= cap) hi = mid; else lo = mid;
    }
    seg = hi;
  }
  // which lists are split, and into how many runs
  int nseg[PT], slot[PT], rank[PT];
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    nseg[i] = split_runs(deg[i], seg);
    slot[i] = nseg[i] > 1 ? nseg[i] : 0;
  }
  block_scan<PT, NT>(slot, wsum, tid);
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    if (nseg[i] > 1 && !split_granted(nseg[i], slot[i], cap)) nseg[i] = 1;
    rank[i] = nseg[i] > 1 ? 1 : 0;
  }
  block_scan<PT, NT>(rank, wsum, tid);
  int4* sp = (int4*)split + (long long)bh * (cap / 2 + 1);
  int extra[PT];
#pragma unroll
  for (int i = 0; i < PT; ++i) {
    if (nseg[i] > 1) sp[1 + rank[i]] = make_int4(j0 + i, slot[i], nseg[i], 0);
    extra[i] = nseg[i] - 1;
  }
  const int items = Nc + block_scan<PT, NT>(extra, wsum, tid);

  // counting sort of the items by length, descending; the runs of a split list as if they were kRunExtra entries longer,
  // which is about what leaving and adding up the partial results takes (as whole lists of their length they would
  // come last and end after everything else)
  constexpr int kRunExtra = 10;
  auto bucket = [&](int len, int runs) { return min(Nc - min(Nc, runs > 1 ? len + kRunExtra : len), PT * NT - 1); };
#pragma unroll
  for (int i = 0; i < PT; ++i)
    if (j0 + i < Nc)
      for (int r = 0; r < nseg[i]; ++r) {
        const int len = run_bound(deg[i], nseg[i], r + 1) - run_bound(deg[i], nseg[i], r);
        atomicAdd(&hist[bucket(len, nseg[i])], 1);
      }
  __syncthreads();
  int first[PT];
#pragma unroll
  for (int i = 0; i < PT; ++i) first[i] = hist[j0 + i];
  block_scan<PT, NT>(first, wsum, tid);
#pragma unroll
  for (int i = 0; i < PT; ++i) hist[j0 + i] = first[i];
  __syncthreads();
  int4* ord = (int4*)order + (long long)bh * (Nc + cap);
#pragma unroll
  for (int i = 0; i < PT; ++i)
    if (j0 + i < Nc)
      for (int r = 0; r < nseg[i]; ++r) {
        const int lo = run_bound(deg[i], nseg[i], r), hi = run_bound(deg[i], nseg[i], r + 1);
        ord[atomicAdd(&hist[bucket(hi - lo, nseg[i])], 1)] =
            make_int4(j0 + i, v[i] + lo, v[i] + hi, nseg[i] > 1 ? run_word(rank[i], slot[i] + r) : -1);
      }
  for (int e = items + tid; e < Nc + cap; e += NT) ord[e] = make_int4(-1, 0, 0, -1);
}

__global__ __launch_bounds__(1024) void k_map_scan(int Nc, int seg_min, int cap, int32_t* __restrict__ row_ptr,
                                                   int32_t* __restrict__ order, int32_t* __restrict__ split) {
  __shared__ int wsum[16];
  __shared__ int hist[kMaxCubes];
  const int bh = blockIdx.x, tid = threadIdx.x;
  const int32_t* rp = row_ptr + (long long)bh * (Nc + 1);
  int deg[4], v[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) deg[i] = (4 * tid + i < Nc) ? rp[4 * tid + i] : 0;
  map_scan_body<4, 1024>(Nc, seg_min, cap, bh, tid, deg, v, row_ptr, order, split, wsum, hist);
}

// the list of key cube j: positions of the set bits of its row `r` (W32 words, global memory or LDS),
// ascending, written to cl[base ..]; one wavefront per row
__device__ __forceinline__ void map_fill_row(const uint32_t* r, int W32, int base, int32_t* __restrict__ cl, int lane) {
  for (int w0 = 0; w0 < W32; w0 += 64) {
    uint32_t word = (w0 + lane < W32) ? r[w0 + lane] : 0u;
    const int c = __popc(word);
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    int pos = base + incl - c;
    while (word) {
      const int b = __ffs(word) - 1;
      cl[pos++] = (w0 + lane) * 32 + b;
      word &= word - 1;
    }
    base += __shfl(incl, 63);
  }
}
__global__ __launch_bounds__(256) void k_map_fill(int Nc, int W32, long long rows, const uint32_t* __restrict__ bits,
                                                  const int32_t* __restrict__ row_ptr, int32_t* __restrict__ col,
                                                  long long col_stride) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);  // bh * Nc + j
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const long long bh = row / Nc;
  map_fill_row(bits + row * W32, W32, row_ptr[bh * (Nc + 1) + row % Nc], col + bh * col_stride, lane);
}

// Lists that name key cubes of 16 tokens (Sec. 3.2, the 64 x 16 row of the tile-size tables): the bit
// matrix has one row per key cube, four per 64-row key block.  The dK/dV pass works on key blocks, so
// the list of block j is the union of its four rows, and every entry carries, above the query block
// number (bits 16..19), which of the four key cubes that query block selected.
__global__ __launch_bounds__(256) void k_map_degree_sub(int Nc, int W32, long long rows, const uint32_t* __restrict__ bits,
                                                        int32_t* __restrict__ row_ptr) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);  // bh * Nc + j
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const uint32_t* r = bits + row * 4 * W32;
  int c = 0;
  for (int w = lane; w < W32; w += 64) c += __popc(r[w] | r[W32 + w] | r[2 * W32 + w] | r[3 * W32 + w]);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if (lane == 0) row_ptr[(row / Nc) * (Nc + 1) + row % Nc] = c;
}
__global__ __launch_bounds__(256) void k_map_fill_sub(int Nc, int W32, long long rows, const uint32_t* __restrict__ bits,
                                                      const int32_t* __restrict__ row_ptr, int32_t* __restrict__ col,
                                                      long long col_stride) {
  const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);  // bh * Nc + j
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const long long bh = row / Nc;
  const uint32_t* r = bits + row * 4 * W32;
  int32_t* cl = col + bh * col_stride;
  int base = row_ptr[bh * (Nc + 1) + row % Nc];
  for (int w0 = 0; w0 < W32; w0 += 64) {
    uint32_t u[4] = {0u, 0u, 0u, 0u};
    if (w0 + lane < W32) {
#pragma unroll
      for (int x = 0; x < 4; ++x) u[x] = r[x * W32 + w0 + lane];
    }
    uint32_t word = u[0] | u[1] | u[2] | u[3];
    const int c = __popc(word);
    int incl = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      int t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    int pos = base + incl - c;
    while (word) {
      const int b = __ffs(word) - 1;
      const uint32_t sel = ((u[0] >> b) & 1u) | (((u[1] >> b) & 1u) << 1) | (((u[2] >> b) & 1u) << 2) | (((u[3] >> b) & 1u) << 3);
      cl[pos++] = (int32_t)(((w0 + lane) * 32 + b) | (sel << 16));
      word &= word - 1;
    }
    base += __shfl(incl, 63);
  }
}

// The whole map of one (b, h) by ONE workgroup, for short sequences (the bit matrix of a (b, h) fits in LDS up to
// kMapOneMaxCubes key cubes): the four steps above -- bits OR-ed into LDS, in-degrees, scan and work items, lists --
// with barriers between them instead of launches.  It needs nothing but the index lists, so it shares the launch
// of the preprocess pass, whose first B*H workgroups do it.
constexpr int kMapOneMaxCubes = 384;
constexpr int kPreThreads = 512;
struct MapOneLds {
  uint32_t bits[kMapOneMaxCubes * (kMapOneMaxCubes / 32 + 1)];
  int start[kPreThreads], hist[kPreThreads];
  int wsum[kPreThreads / 64];
};
static_assert(kMapOneMaxCubes <= kPreThreads, "a cube per thread");
__device__ __forceinline__ void map_one(MapOneLds& l, const MapArgs& a, int bh, int tid) {
  const int Nc = a.Nc, K = a.K, W32 = (Nc + 31) / 32;
  const int WS = W32 | 1;  // odd row stride: the rows the OR step and the count step touch together fall into different banks
  for (int i = tid; i < Nc * WS; i += kPreThreads) l.bits[i] = 0u;
  __syncthreads();
  const int32_t* my = a.idx + (long long)bh * Nc * K;
  for (int e0 = tid; e0 < Nc * K; e0 += 8 * kPreThreads) {  // (eight loads in flight per thread, then their bits)
    int c[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) c[u] = e0 + u * kPreThreads < Nc * K ? my[e0 + u * kPreThreads] : -1;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int q = (e0 + u * kPreThreads) / K;
      if (map_takes(c[u], Nc)) atomicOr(&l.bits[c[u] * WS + (q >> 5)], 1u << (q & 31));  // (a caller-supplied list is not trusted)
    }
  }
  __syncthreads();
  int deg[1] = {0}, v[1];
  if (tid < Nc)
    for (int w = 0; w < W32; ++w) deg[0] += __popc(l.bits[tid * WS + w]);
  map_scan_body<1, kPreThreads>(Nc, a.seg, a.cap, bh, tid, deg, v, a.row_ptr, a.order, a.split, l.wsum, l.hist);
  l.start[tid] = v[0];
  __syncthreads();
  // lists: one thread per word of the bit matrix (a row has at most 12 words here, so the count of the
  // bits before a word is a short loop over LDS)
  int32_t* cl = a.col + bh * ((long long)Nc * K);
  for (int i = tid; i < Nc * W32; i += kPreThreads) {
    const int j = i / W32, w = i - j * W32;
    uint32_t word = l.bits[j * WS + w];
    if (!word) continue;
    int pos = l.start[j];
    for (int x = 0; x < w; ++x) pos += __popc(l.bits[j * WS + x]);
    while (word) {
      cl[pos++] = w * 32 + __ffs(word) - 1;
      word &= word - 1;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// Preprocess.  Per token i of cube c (pad rows produce zeros):
//   dGc_i = dO_i * Oc[c]      dGf_i = dO_i * Of_i      dOf_i = dO_i * Gf_i  (bf16, feeds the MFMAs)
//   Delta_i = sum_d dOf_i * Of_i                       dOc[c] = sum_i dO_i * Gc_i   dot[c] = dOc[c] . Oc[c]
//   rowd   per 32 rows: 32 values of -lse_i * log2(e) / sl2 (so that P = exp2((S + value) * sl2); -30000 on
//          pad rows, where P then underflows to 0), then 32 values of -Delta_i
// 256 threads per (b*h, cube), which walk the cube's m blocks of 64 rows; thread layout as in the
// pooling kernel.  Bound by its seven tensors' traffic (39936 tokens, 12 heads: 0.86 GB in 137 us).
// The first `map_blocks` workgroups transpose the block map instead: a serial chain of short steps that keeps B*H
// CUs busy for 11 to 40 us and used to be a launch of its own.  Train step, own launch -> shared: 32 blocks 65 -> 55 us;
// 256 blocks, 12 heads 1044 -> 1035, d = 64, 16 heads 795 -> 783; 280 blocks, 5 heads, through the op 562 -> 548.
// (Workgroups of 256 threads: 57 and, for the last, whose map is then the longer part, 555; of 1024: 57 and 544, but
// 788 for the one before.)
// KIND 0, 1: dout and the gates' gradients tiled, 1 past the caches; 2: raster.
template <int D, int KIND>
__global__ __launch_bounds__(kPreThreads) void k_bwd_pre(int map_blocks, MapArgs map_args, unsigned cubes, int Nc, int m_blocks, const uint64_t* __restrict__ mask, const uint4* __restrict__ dout,
                                                 const uint4* __restrict__ gc, const uint4* __restrict__ gf,
                                                 const uint4* __restrict__ of, const float* __restrict__ oc,
                                                 uint4* __restrict__ dgc, uint4* __restrict__ dgf,
                                                 uint4* __restrict__ dof, float* __restrict__ rowd, float inv_sl2,
                                                 float* __restrict__ doc, float* __restrict__ dot,
                                                 const float* __restrict__ lse_f, int H, long long do_head_stride,
                                                 long long do_row_stride, RasterMap raster) {
  constexpr bool ONCE = KIND == 1;
  constexpr int CPR = D / 8, RG = 256 / CPR, RPT = kTile / RG;
  __shared__ union {
    float part[kPreThreads / 256][RG][D + 4];
    MapOneLds map;
  } lds;
  if ((int)blockIdx.x < map_blocks) {  // (uniform) the transposed map of one (b, h)
    map_one(lds.map, map_args, blockIdx.x, threadIdx.x);
    return;
  }
  // two cubes a workgroup, 256 threads each
  const int tid = threadIdx.x & 255;
  auto& part = lds.part[threadIdx.x >> 8];
  const unsigned at = (blockIdx.x - map_blocks) * (kPreThreads / 256) + (threadIdx.x >> 8), cube = min(at, cubes - 1);
  const bool live = at < cubes;  // (the last workgroup's spare threads store nothing)
  const int c = cube % Nc;
  const long long bh = cube / Nc;
  const int ch = tid % CPR, rg = tid / CPR;
  float ocv[8];
  {
    const float* p = oc + (bh * Nc + c) * D + ch * 8;
    const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
    ocv[0] = a.x; ocv[1] = a.y; ocv[2] = a.z; ocv[3] = a.w; ocv[4] = b.x; ocv[5] = b.y; ocv[6] = b.z; ocv[7] = b.w;
  }
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int sb = 0; sb < (live ? m_blocks : 0); ++sb) {
  const long long blk = (bh * Nc + c) * m_blocks + sb;  // block index over all (b, h)
  const uint64_t m = mask[c * m_blocks + sb];
  const long long row0 = blk * (long long)kTile;
  const RasterRows rows_r(raster, bh, c * m_blocks + sb, CPR);
  // dout may be head-major [B,H,Np,D] or token-major [B,Np,H,D] (see the forward's `out`)
  const long long Npad = (long long)Nc * m_blocks * kTile;
  const long long do0 = (bh / H) * ((long long)H * Npad * CPR) + (bh % H) * do_head_stride +
                        ((long long)c * m_blocks + sb) * kTile * do_row_stride;
#pragma unroll
  for (int i = 0; i < RPT; ++i) {
    const int r = rg + i * RG;
    const long long g = (row0 + r) * CPR + ch;
    const bool valid = (m >> r) & 1;
    uint4 z = make_uint4(0, 0, 0, 0), o_gc = z, o_gf = z, o_dof = z;
    float dsum = 0.f;
    if (valid) {
      float go[8], gcv[8], gfv[8], ofv[8], t0[8], t1[8], t2[8];
      unpack8(load16<ONCE>(dout + (KIND == 2 ? rows_r.at(r) : do0 + r * do_row_stride) + ch), go);
      unpack8(load16<ONCE>(gc + g), gcv);
      unpack8(load16<ONCE>(of + g), ofv);
      if (gf) unpack8(load16<ONCE>(gf + g), gfv);
      else {
#pragma unroll
        for (int e = 0; e < 8; ++e) gfv[e] = 1.f;
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        t0[e] = go[e] * ocv[e];
        t1[e] = go[e] * ofv[e];
        t2[e] = go[e] * gfv[e];
        acc[e] += go[e] * gcv[e];
      }
      o_gc = pack8(t0); o_gf = pack8(t1); o_dof = pack8(t2);
      float t2r[8];
      unpack8(o_dof, t2r);  // Delta uses the rounded dOf, the value the fine kernels multiply with
#pragma unroll
      for (int e = 0; e < 8; ++e) dsum = fmaf(t2r[e], ofv[e], dsum);
    }
    if (KIND < 2 || valid) {
      const long long to = KIND == 2 ? rows_r.at(r) + ch : g;
      store16<ONCE>(dgc + to, o_gc);
      if (dgf) store16<ONCE>(dgf + to, o_gf);
    }
    dof[g] = o_dof;
#pragma unroll
    for (int o = CPR / 2; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
    if (ch == 0) {
      float* p = rowd + 2 * (row0 + (r & ~31)) + (r & 31);
      p[0] = valid ? -lse_f[row0 + r] * kLog2e * inv_sl2 : -30000.f;
      p[32] = -dsum;
    }
  }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[rg][ch * 8 + e] = acc[e];
  __syncthreads();
  if (tid < 64 && live) {  // one wavefront: its lanes take columns lane and, at d = 128, lane + 64
    float dsum = 0.f;
#pragma unroll
    for (int e = tid; e < D; e += 64) {
      float s = 0;
      for (int r = 0; r < RG; ++r) s += part[r][e];
      doc[(bh * Nc + c) * D + e] = s;
      dsum = fmaf(s, oc[(bh * Nc + c) * D + e], dsum);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dsum += __shfl_xor(dsum, o);
    if (tid == 0) dot[bh * Nc + c] = dsum;
  }
}

hipError_t launch_bwd_pre(int BH, int Nc, int m_blocks, int d, const uint64_t* mask, const void* dout, const void* gate_c,
                          const void* gate_f, const void* out_fine, const float* oc, void* dgate_c, void* dgate_f,
                          void* dof, float* rowd, float scale, float* doc, float* dot, const float* lse_f, int H,
                          int dout_token_major, const MapArgs* map, const RasterMap& raster, hipStream_t s) {
  const MapArgs m = map ? *map : MapArgs{};
  const int mb = map ? BH : 0;  // workgroups that transpose the map, ahead of the others
  const unsigned cubes = (unsigned)(BH * Nc), per = kPreThreads / 256, grid = (cubes + per - 1) / per + (unsigned)mb;
  const float inv_sl2 = 1.0f / (scale * kLog2e);
  const long long cpr = d / 8, Np = (long long)Nc * m_blocks * kTile;
  const long long dhs = dout_token_major ? cpr : Np * cpr, drs = dout_token_major ? H * cpr : cpr;
  const bool stream = (long long)BH * Np * d * 2 >= kStreamBytes;
#define VSA_PRE(D_, KIND_)                                                                                              \
  k_bwd_pre<D_, KIND_><<<grid, kPreThreads, 0, s>>>(mb, m, cubes, Nc, m_blocks, mask, (const uint4*)dout, (const uint4*)gate_c, \
                                                    (const uint4*)gate_f, (const uint4*)out_fine, oc, (uint4*)dgate_c,  \
                                                    (uint4*)dgate_f, (uint4*)dof, rowd, inv_sl2, doc, dot, lse_f, H, dhs, drs, raster)
  if (d == 128) {
    if (raster.on) VSA_PRE(128, 2);
    else if (stream) VSA_PRE(128, 1);
    else VSA_PRE(128, 0);
  } else {
    if (raster.on) VSA_PRE(64, 2);
    else if (stream) VSA_PRE(64, 1);
    else VSA_PRE(64, 0);
  }
#undef VSA_PRE
  return hipGetLastError();
}

bool map_with_bwd_pre(int Nc, int key_cubes_16) { return !key_cubes_16 && Nc <= kMapOneMaxCubes; }

hipError_t launch_transpose_map(int BH, const MapArgs& a, uint32_t* bits, int key_cubes_16, hipStream_t s) {
  const int Nc = a.Nc, K = a.K, seg = a.seg, cap = a.cap;
  const int32_t* idx = a.idx;
  int32_t *row_ptr = a.row_ptr, *col = a.col, *order = a.order, *split = a.split;
  const int W32 = (Nc + 31) / 32;
  const long long rows = (long long)BH * Nc;
  hipError_t e;
  if (key_cubes_16) {  // K entries per query block, each a key cube of 16 tokens; bits is [BH, 4 Nc, W32]
    k_map_bits<<<(unsigned)(BH * W32), 256, 0, s>>>(Nc, 4 * Nc, K, W32, idx, bits);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_map_degree_sub<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(Nc, W32, rows, bits, row_ptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_map_scan<<<BH, 1024, 0, s>>>(Nc, seg, cap, row_ptr, order, split);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    k_map_fill_sub<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(Nc, W32, rows, bits, row_ptr, col, (long long)Nc * K);
    return hipGetLastError();
  }
  k_map_bits<<<(unsigned)(BH * W32), 256, 0, s>>>(Nc, Nc, K, W32, idx, bits);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_map_degree<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(Nc, W32, rows, bits, row_ptr);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_map_scan<<<BH, 1024, 0, s>>>(Nc, seg, cap, row_ptr, order, split);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_map_fill<<<(unsigned)((rows + 3) / 4), 256, 0, s>>>(Nc, W32, rows, bits, row_ptr, col, (long long)Nc * K);
  return hipGetLastError();
}

}  // namespace vsa
