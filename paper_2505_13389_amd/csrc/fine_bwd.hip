// Fine stage backward (Sec. 2.4 states a backward kernel exists; this is FlashAttention-style
// recomputation of P from the saved log-sum-exp, on the block-sparse pattern):
//   P_ij = exp(S_ij - lse_i),  dP_ij = dOf_i . v_j,  dS_ij = P_ij (dP_ij - Delta_i)
//   dQ_i = scale sum_j dS_ij k_j      (query-tile-major pass over the index list)
//   dK_j = scale sum_i dS_ij q_i,  dV_j = sum_i P_ij dOf_i   (key-tile-major pass over the
//                                                             transposed block map)
// Both passes add the pooled-path gradient dXc[cube]/cnt to every valid row in their epilogue
// and write zeros to pad rows.  Work split and operand layouts follow the forward kernel: the
// streamed tiles are copied global -> LDS asynchronously (two stages in the dQ pass, four in the
// dK/dV pass), the resident tile sits in registers, and each wavefront pair owning the same output
// rows is merged once at the end.  The per-row terms (lse, Delta) and the pad-key mask enter the
// products through extra MFMA steps rather than per-element vector arithmetic.
#include <type_traits>

#include "fine_tile.h"
#include "vsa_kernels.h"

namespace vsa {

// ---------------------------------------------------------------------------------------------
// dQ pass: one workgroup per (b, h, query cube); streams the K selected (K tile, V tile) pairs.
// Wavefront (qh, kh): query rows qh*32..+31, key rows kh*32..+31 of each tile.  LIST as in the forward
// kernel: one list entry per tile, or four key cubes of 16 tokens gathered into one.
template <int D, class LIST>
__global__ __launch_bounds__(256, 2) void k_fine_bwd_dq(int Nc, int K, float sl2, float scale, const uint4* __restrict__ q,
                                                        const uint4* __restrict__ k, const uint4* __restrict__ v,
                                                        const uint4* __restrict__ dof, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ rowd,
                                                        const float* __restrict__ dqc, const uint64_t* __restrict__ mask,
                                                        uint4* __restrict__ dq, int m_blocks) {
  using TL = Tile<D>;
  constexpr int CPR = TL::CPR, KS = D / 16, DVB = D / 32, LPT = TL::LPT;
  constexpr int OS = D;
  constexpr int STAGE = 2 * TL::BYTES;  // K tile + V tile
  __shared__ __attribute__((aligned(16))) unsigned char stage0[STAGE];
  __shared__ __attribute__((aligned(16))) unsigned char stage1[STAGE];
  static_assert(2 * 32 * OS * 4 <= STAGE, "merge buffer must fit in one stage");

  // (K = Nc: plain blockIdx order and staggered walks, as in the forward kernel)
  const int NT = (K + LIST::kEntriesPerTile - 1) / LIST::kEntriesPerTile;  // the walk is in tiles of 64 keys
  const bool same_lists = K == Nc * LIST::kEntriesPerTile;
  const unsigned wg = same_lists ? blockIdx.x : xcd_chunked_id(blockIdx.x, gridDim.x);
  const int c = wg % Nc;
  const long long bh = wg / Nc;
  const int rot = same_lists ? ((c >> 3) & 15) % NT : 0;
  auto ent = [&](int t) { const int e = t + rot; return e >= NT ? e - NT : e; };
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qh = wave & 1, kh = wave >> 1, l32 = lane & 31, h = lane >> 5;
  const long long rows0 = bh * (long long)Nc * kTile;
  const int32_t* my_idx = idx + (bh * Nc + c) * (long long)K;
  const uint64_t qmask = mask[c];

  // Start-up order: the list first (one round trip), then the copy of tile 0, and only then the
  // loads of the key masks, Q, dO_f and the per-row terms, so that everything the first iteration
  // needs is in flight together.  The empty asm consumes the loaded registers: the compiler has to
  // place its wait for them right there (it also drains the copy, which it cannot see), and its own
  // vmcnt bookkeeping has nothing left to wait for inside the loop (see Tile::async_load).
  unsigned goff[TL::IPW];
  LIST::template offsets<TL>(wave, lane, goff);
  LIST cubes;
  cubes.init(my_idx, mask, K, kh, wave, lane, Nc);
  {
    const int jt = cubes.first_row(ent(0));  // first source row of this wave's share
    TL::async_load(k, rows0 + jt, stage0, wave, goff);
    TL::async_load(v, rows0 + jt, stage0 + TL::BYTES, wave, goff);
  }
  cubes.load_masks();
  const long long qrow_g = rows0 + c * kTile + qh * 32 + l32;
  bf16x8 qreg[KS], doreg[KS];
  {
    const uint4* qrow = q + qrow_g * CPR;
    const uint4* dorow = dof + qrow_g * CPR;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qreg[s] = __builtin_bit_cast(bf16x8, qrow[2 * s + h]);
      doreg[s] = __builtin_bit_cast(bf16x8, dorow[2 * s + h]);
    }
  }
  // row terms -lse*log2(e)/sl2 (-30000 on pad query rows: then P = 0 and the row contributes nothing) and -Delta
  const float* qterm = rowd + 2 * (rows0 + c * kTile + qh * 32) + l32;
  float nlse = qterm[0], ndelta = qterm[32];
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qreg[s]), "+v"(doreg[s]));
  asm volatile("" : "+v"(nlse), "+v"(ndelta), "+v"(cubes.km_v));
  uint32_t km_cur;  // valid-key mask (this wave's key half) of the tile of this iteration
  {
    int jt;
    cubes.get_tile(ent(0), jt, km_cur);
  }

  f32x16 acc[DVB];
#pragma unroll
  for (int x = 0; x < DVB; ++x)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[x][i] = 0.f;

  const int lane_a = TL::rowmajor_lane(kh * 32, lane);
  int lane_b0, lane_b1;
  TL::transposed_lane(kh * 32, lane, lane_b0, lane_b1);

  // Per-row terms folded into the matrix products (the vector pipe is the scarcer resource here):
  // one extra MFMA step adds -lse2[q]/sl2 to S^T, so that P = exp2(S' * sl2), plus a large negative
  // bias on pad keys; one extra step subtracts Delta[q] from dP^T.  Query-side operands (lane = query
  // column, slots 0..2 = the fp32 value split into three bf16 parts, slot 3 = 1 resp. 0) are fixed for
  // the workgroup; the key-side operand is (1, 1, 1, bias of key l%32).  Only the lane half h = 0
  // carries contraction slots 0..7; the other half is zero.
  constexpr uint32_t kOneBits = 0x3f80u, kBiasBits = 0xc6eau;  // bf16 1.0 and bf16(-29952)
  bf16x8 bq_s, bq_d, a_d;
  {
    const uint2 sb = split3_bf16(nlse, 1.f), db = split3_bf16(ndelta, 0.f);
    bq_s = __builtin_bit_cast(bf16x8, make_uint4(h == 0 ? sb.x : 0u, h == 0 ? sb.y : 0u, 0u, 0u));
    bq_d = __builtin_bit_cast(bf16x8, make_uint4(h == 0 ? db.x : 0u, h == 0 ? db.y : 0u, 0u, 0u));
    a_d = __builtin_bit_cast(bf16x8, make_uint4(h == 0 ? kOneBits * 0x10001u : 0u, h == 0 ? kOneBits : 0u, 0u, 0u));
  }

  // Per tile: wait for this wave's share of tile t, barrier (tile t complete, and every wave is
  // done with tile t-1), start the copy of tile t+1 into the other stage, do the math on tile t.
  auto body = [&](auto copy_tag, const unsigned char* cur, unsigned char* nxt, int t) {
    constexpr bool COPY = decltype(copy_tag)::value;  // false for the last tile of the list
    const uint32_t mh = km_cur;
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    // The copy of the next tile is not issued in one burst here -- eight wavefronts doing that at
    // the same moment queue up behind one another in the load path and stall -- but one
    // instruction per matrix step below.
    int jt = 0;
    if (COPY) cubes.get_tile(ent(t + 1), jt, km_cur);
    const void* gk = uniform_ptr(k + (rows0 + jt) * CPR);
    const void* gv = uniform_ptr(v + (rows0 + jt) * CPR);
    const unsigned ln = __builtin_amdgcn_readfirstlane(lds_address(nxt) + (unsigned)(wave * TL::IPW) * 1024u);
    auto copy_piece = [&](int i) {
      if (!COPY) return;
      if (i == 0) set_m0(ln);
      if (i == TL::IPW) set_m0(ln + TL::BYTES);
      if (i < 2 * TL::IPW) {
        const void* g = i < TL::IPW ? gk : gv;
        const int r = i % TL::IPW;
        if (r == 0) lds_dma16_at<0>(g, goff[0]);
        if (r == 1) lds_dma16_at<1024>(g, goff[1 % TL::IPW]);
        if (r == 2) lds_dma16_at<2048>(g, goff[2 % TL::IPW]);
        if (r == 3) lds_dma16_at<3072>(g, goff[3 % TL::IPW]);
      }
    };
    __builtin_amdgcn_sched_barrier(0);
    const unsigned char* Ks = cur;
    const unsigned char* Vs = cur + TL::BYTES;

    // The LDS operands are requested a fixed number of matrix instructions ahead of their use, in
    // a pinned order (left to itself the compiler reads, waits and multiplies one operand at a
    // time).  Operand i: K rows (S^T steps), then V rows (dP^T steps), then transposed K (dQ^T
    // steps).  Operand addresses are rebuilt from three lane-dependent values (one XOR per read)
    // rather than held in registers across the loop: the register file is the scarce resource.
    int la = lane_a, lb0 = lane_b0, lb1 = lane_b1;
    asm volatile("" : "+v"(la), "+v"(lb0), "+v"(lb1));
    constexpr int NOP = 2 * KS + 2 * DVB, AHEAD = 4;
    bf16x8 op[NOP];
    auto read_op = [&](int i) {
      if (i < KS) return TL::rowmajor_at(Ks, la, i);
      if (i < 2 * KS) return TL::rowmajor_at(Vs, la, i - KS);
      const int j = i - 2 * KS;
      return TL::transposed_at(Ks, lb0, lb1, j & 1, j >> 1);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) op[i] = read_op(i);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 sacc, dpacc;
#pragma unroll
    for (int i = 0; i < 16; ++i) { sacc[i] = 0.f; dpacc[i] = 0.f; }
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      if (i < KS) sacc = mfma32(op[i], qreg[i < KS ? i : 0], sacc);
      else dpacc = mfma32(op[i], doreg[i < KS ? 0 : i - KS], dpacc);
      if (i + AHEAD < NOP) op[i + AHEAD] = read_op(i + AHEAD);
      if (!(i & 1)) copy_piece(i >> 1);
      __builtin_amdgcn_sched_barrier(0);
    }

    // one more step on each product brings in the per-row terms and the pad-key bias (see bq_s)
    {
      const bool dead = !((mh >> l32) & 1);
      const uint32_t w1 = kOneBits | ((dead ? kBiasBits : 0u) << 16);
      const bf16x8 a_s = __builtin_bit_cast(bf16x8, make_uint4(h == 0 ? kOneBits * 0x10001u : 0u, h == 0 ? w1 : 0u, 0u, 0u));
      sacc = mfma32(a_s, bq_s, sacc);
      dpacc = mfma32(a_d, bq_d, dpacc);
    }
    float ds[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) ds[i] = fast_exp2(sacc[i] * sl2) * dpacc[i];
    const bf16x8 b0 = acc_to_operand(ds), b1 = acc_to_operand(ds + 8);
#pragma unroll
    for (int j = 0; j < 2 * DVB; ++j) {
      const int i = 2 * KS + j;
      acc[j >> 1] = mfma32(op[i], (j & 1) ? b1 : b0, acc[j >> 1]);
      if (i + AHEAD < NOP) op[i + AHEAD] = read_op(i + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  {
    const std::true_type copy;
    const std::false_type last;
    int t = 0;
    for (; t + 2 < NT; t += 2) {
      body(copy, stage0, stage1, t);
      body(copy, stage1, stage0, t + 1);
    }
    if (t + 1 < NT) {
      body(copy, stage0, stage1, t);
      body(last, stage1, stage0, t + 1);
    } else {
      body(last, stage0, stage1, t);
    }
  }
  // the pooled-gradient term of this thread's column chunk (the same chunk for all of its items),
  // requested before the partial results go through LDS
  static_assert(256 % CPR == 0, "a thread keeps its column chunk");
  const float* dqcr = dqc + ((bh * Nc + c) / m_blocks) * D + (tid % CPR) * 8;  // per cube = m_blocks blocks
  const float4 pc0 = *(const float4*)dqcr, pc1 = *(const float4*)(dqcr + 4);
  __syncthreads();

  {
    float* Op = (float*)(kh == 0 ? stage0 : stage1) + qh * 32 * OS;
#pragma unroll
    for (int x = 0; x < DVB; ++x)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        float4 val = make_float4(acc[x][4 * g4], acc[x][4 * g4 + 1], acc[x][4 * g4 + 2], acc[x][4 * g4 + 3]);
        *(float4*)&Op[merge_offset(l32, x * 32 + 8 * g4 + 4 * h, OS)] = val;
      }
  }
  __syncthreads();

  const float inv_cnt = 1.0f / (float)cube_count(mask, c, m_blocks);
  const float pooled[8] = {pc0.x * inv_cnt, pc0.y * inv_cnt, pc0.z * inv_cnt, pc0.w * inv_cnt,
                           pc1.x * inv_cnt, pc1.y * inv_cnt, pc1.z * inv_cnt, pc1.w * inv_cnt};
#pragma unroll
  for (int it = 0; it < LPT; ++it) {
    const int item = it * 256 + tid, r = item / CPR, ch = item % CPR;
    const int m0 = merge_offset(r, ch * 8, OS), m1 = merge_offset(r, ch * 8 + 4, OS);
    const float4 a0 = *(const float4*)((const float*)stage0 + m0), a1 = *(const float4*)((const float*)stage0 + m1);
    const float4 b0 = *(const float4*)((const float*)stage1 + m0), b1 = *(const float4*)((const float*)stage1 + m1);
    const float sum[8] = {a0.x + b0.x, a0.y + b0.y, a0.z + b0.z, a0.w + b0.w, a1.x + b1.x, a1.y + b1.y, a1.z + b1.z, a1.w + b1.w};
    uint4 ov = make_uint4(0, 0, 0, 0);
    if ((qmask >> r) & 1) {
      float res[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) res[e] = fmaf(sum[e], scale, pooled[e]);
      ov = pack8(res);
    }
    dq[(rows0 + c * kTile + r) * CPR + ch] = ov;
  }
}

hipError_t launch_fine_bwd_dq(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                              const void* dof, const int32_t* idx, const float* rowd,
                              const float* dqc, const uint64_t* mask, void* dq, int m_blocks, int key_cubes_16,
                              hipStream_t s) {
  const float sl2 = scale * kLog2e;
  const unsigned grid = (unsigned)(BH * Nc);
#define VSA_DQ(D_, LIST_)                                                                                          \
  k_fine_bwd_dq<D_, LIST_><<<grid, 256, 0, s>>>(Nc, K, sl2, scale, (const uint4*)q, (const uint4*)k, (const uint4*)v, \
                                                (const uint4*)dof, idx, rowd, dqc, mask, (uint4*)dq, m_blocks)
  if (key_cubes_16) {  // K counts key cubes of 16 tokens
    if (d == 128) VSA_DQ(128, SubCubeList);
    else VSA_DQ(64, SubCubeList);
  } else {
    if (d == 128) VSA_DQ(128, CubeList);
    else VSA_DQ(64, CubeList);
  }
#undef VSA_DQ
  return hipGetLastError();
}

}  // namespace vsa
