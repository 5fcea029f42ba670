// Fine stage backward (Sec. 2.4 states a backward kernel exists; this is FlashAttention-style
// recomputation of P from the saved log-sum-exp, on the block-sparse pattern):
//   P_ij = exp(S_ij - lse_i),  dP_ij = dOf_i . v_j,  dS_ij = P_ij (dP_ij - Delta_i)
//   dQ_i = scale sum_j dS_ij k_j      (query-block-major pass over the index list: this file)
//   dK_j = scale sum_i dS_ij q_i,  dV_j = sum_i P_ij dOf_i   (key-block-major pass over the transposed
//                                                             block map: fine_bwd_dkv.h)
// Both passes add the pooled-path gradient dXc[cube]/cnt to every valid row in their epilogue
// and write zeros to pad rows.
#include <type_traits>

#include "fine_bwd_dkv.h"
#include "ticks.h"

namespace vsa {

// Workgroups of two wavefronts (four in small launches) that stream units of 32 keys like the forward's (fine_fwd.hip),
// each of a block of its own or sharing one (paired_workgroups).  A unit is S^T, dP^T and dQ^T, 16 queries (d = 128) or 32 after the other,
// so that the vector work of some, P = exp2(S sl2 - lse) and dS = P dP', lies behind the matrix work of the others
// without a second unit in flight; the LDS operands of a product stay in registers for all of them.
// The row terms are per-lane scalars here (a lane owns query columns): lse goes
// into the exponential's fma, -Delta is the initial value of the dP accumulators.
//
// d = 128: one wavefront per SIMD; dQ takes 128 of the accumulation registers and Q and dO_f the other 128 (a
// matrix instruction reads an operand from either file).  16x16x32 instructions, 96 a unit, with what lies behind each dealt by DqTicks
// (ticks.h; why the small ones, see fine_bwd_dkv.h: 3.9 other instructions per 32 cycles of matrix work).  Pad keys' rows of S^T start from
// a large negative value, which is formed where a unit or the one before has some.
// d = 64: two wavefronts per SIMD, whose 256 registers do not
// hold both halves' S and dP, and 32x32x16 instructions: S 0 | dP 0 | S 1 | dP 1 | dQ 0 | dQ 1, -Delta is added in vector arithmetic.
//
// What bounds it (d = 128): the clock, which falls as the pipe fills, and instruction issue: a unit is 96 matrix instructions (1536 cycles of
// the matrix pipe) and 187 others (191 where all blocks are shared, 195 for those shared beside paired ones), 1870 to 1900 cycles by the costs of ticks.h
// where the form before it, with 48 large instructions, had 1930, at a clock 7 % lower (39936 tokens: 1.72 GHz, now 1.84): 1468 -> 1405 us of 39936
// tokens, 12 heads, top-78.  With dK/dV's
// like form, whole steps: 16384 tokens, top-32 961 -> 922 us, 39936 tokens, top-78 4850 -> 4696, B = 2, 16 heads, top-128 of 256, local
// lists 7953 -> 7535, 256-token cubes 918 -> 881, the op at 13338 tokens 453 -> 444.  Most matrix instructions take 16 to 25 cycles
// with what lies behind them, those with a part of the list entry's scalar chain up to 30, the seam of two units 38 to 42.
// Launches that leave SIMDs idle, the pass against the form before: 32 to 128 blocks 0.99 to 1.015 of the time, 192 to 512 0.93 to 1.005 (4 to 128 entries,
// 16 to 256 key cubes of 16 tokens; run to run 0.01).
// Start-up, merge and stores are about 7 us of a shared block's 95; with a wavefront per block 39936 tokens, 12 heads, d =
// 128, top-78 took 1500 -> 1470 us, 16384 tokens, top-32 281 -> 269, top-8 121 -> 96, 1024 blocks, top-8 0.84 of the time.
// Measured against 32 keys x 32 queries per wavefront, four wavefronts in step, two per SIMD: 39936 tokens, 12 heads, d = 128,
// top-78 of 624: 1.61 -> 1.49 ms; 16384 tokens, top-32 of 256: 303 -> 277 us; B = 2, 16 heads, top-128
// of 256, local lists: 2.83 -> 2.58 ms; d = 64, B = 2, 8 heads, top-32: 220 -> 210 us.
template <int D, int NW>
struct DqShape {
  static constexpr int HALF = Tile<D>::BYTES / 2;  // 32 rows
  static constexpr int LDS = NW * 4 * HALF;        // per wavefront: K of two units, V of two units
};

// d = 128: what lies behind which of the 96 matrix instructions of a unit (ticks.h): S of the queries 0 .. 15, 16 .. 31, ... | dP likewise |
// dQ likewise.
struct DqTicks : TickTable<96, 32> {
  static constexpr int KS = 8, PH = 4 * KS;  // LDS operands of a product; its ticks
  enum Kind { V, K_T, K_NEXT };
  static constexpr int kFirstCopyV = PH + 2 * KS, kFirstCopyK = 2 * PH + 1;  // of the unit after the next, where V, where K lay
  static constexpr int kRowsReady = 2 * PH + 12;  // K and V of the next unit are waited for here
  static constexpr int kTile = 2, kChunk = 4, kRows = 6, kValid = 8;  // the list entry of the unit after the next, a scalar chain, in parts
  static constexpr int v_copy(int t) { return t >= kFirstCopyV && t < kFirstCopyV + 2 * KS && (t - kFirstCopyV) % 2 == 0 ? (t - kFirstCopyV) / 2 : -1; }
  static constexpr int k_copy(int t) { return t >= kFirstCopyK && t < kFirstCopyK + 4 * KS && (t - kFirstCopyK) % 4 == 0 ? (t - kFirstCopyK) / 4 : -1; }
  static constexpr int k_copies_before(int t) { return t <= kFirstCopyK ? 0 : (t - kFirstCopyK + 3) / 4; }
  // P and dS in operations, and how many of them lie ahead of tick t
  static constexpr int kPOps = 64, kSOps = 48;
  Work pw[kPOps] = {}, sw[kSOps] = {};
  int p[T + 1] = {}, s[T + 1] = {};
  constexpr DqTicks() {
    int n = 0;
    auto add = [&](int tick, int use, int kind, int i, int part) { r[n++] = Read{tick, use, kind, i, part}; };
    for (int i = 0; i < KS; ++i) add(i, PH, V, i, 0);
    for (int j = 0; j < 2 * KS; ++j) add(KS + 2 * j, 2 * PH, K_T, j / 2, j & 1);  // (all of them are there before their place is copied over)
    for (int i = 0; i < KS; ++i) add(kRowsReady + 1 + 2 * i, T + (i & ~1), K_NEXT, i, 0);
    order_reads();
    for (int t = 0; t < T; ++t) {
      if (v_copy(t) >= 0) cycles[t] += kCopy + (v_copy(t) % 4 == 0 ? kScalar : 0);
      if (k_copy(t) >= 0) cycles[t] += kCopy + (k_copy(t) % 4 == 0 ? kScalar : 0);
    }
    // P: an item's first exponential, the arithmetic of the next, its second exponential; dS: the products of an item, the
    // conversion of the one before
    n = 0;
    pw[n++] = {MUL, 0, 0};
    pw[n++] = {MUL, 0, 1};
    for (int g = 0; g < 16; ++g) {
      pw[n++] = {EXP, g, 0};
      if (g < 15) pw[n++] = {MUL, g + 1, 0};
      if (g < 15) pw[n++] = {MUL, g + 1, 1};
      pw[n++] = {EXP, g, 1};
    }
    n = 0;
    for (int k = 0; k < 17; ++k) {
      if (k < 16) sw[n++] = {MUL, k, 0};
      if (k > 0) sw[n++] = {CVT, k - 1, 0};
      if (k < 16) sw[n++] = {MUL, k, 1};
    }
    // from two instructions behind the first S, the first dP, to the last dP, the last dQ
    deal(s, sw, kSOps, PH + KS + 2, 3 * PH - KS - 1);
    deal(p, pw, kPOps, KS + 2, 2 * PH + 2);
  }
  // Every 16 queries' operations lie behind what they need and ahead of what needs them (4 items each).
  constexpr bool in_order() const {
    for (int b = 0; b < 4; ++b) {
      const int s_there = (b + 1) * KS + 2, dp_there = PH + (b + 1) * KS + 2, dq_begins = 2 * PH + b * KS;
      for (int n = 0; n < p[s_there]; ++n)
        if (pw[n].item >= 4 * (b + 1)) return false;
      for (int n = p[dp_there]; n < kPOps; ++n)
        if (pw[n].item < 4 * (b + 1) && s[dp_there + 1] > 12 * b) return false;
      for (int n = 0; n < s[dp_there]; ++n)
        if (sw[n].item >= 4 * (b + 1)) return false;
      for (int n = s[dq_begins - 1]; n < kSOps; ++n)
        if (sw[n].item < 4 * (b + 1) && sw[n].op == CVT) return false;
    }
    for (int t = 0; t < T; ++t)  // P of an item ahead of its dS
      for (int n = s[t]; n < s[t + 1]; ++n)
        for (int m = p[t]; m < kPOps; ++m)
          if (pw[m].item <= sw[n].item) return false;
    return ordered(pw, kPOps) && ordered(sw, kSOps);
  }
};
static_assert(DqTicks().in_order(), "operations of dQ");

// `smem`: DqShape::LDS bytes, aligned to 1024; `masks`: 128 words per wavefront.  `block` of `grid` workgroups.  PAIRS: the
// first `pairs` of them take two blocks (NW = 2; launches without pairs have instances of their own, as in the forward).  COARSE: the
// pooled-gradient term is formed here (NW = 4, cubes of one block), in `lc`, and dqc is not read.
template <int D, int NW, template <class> class UNITS, bool PAIRS, bool COARSE>
__device__ __forceinline__ void dq_block(
    unsigned char* smem, uint32_t* masks, unsigned block, unsigned grid, int Nc, int K, float sl2, float scale,
    const uint4* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v, const uint4* __restrict__ dof,
    const int32_t* __restrict__ idx, const float* __restrict__ rowd, const float* __restrict__ dqc,
    const uint64_t* __restrict__ mask, uint4* __restrict__ dq, int m_blocks, unsigned blocks, unsigned pairs, int stream,
    const RasterMap& raster, const SmallCoarseArgs& sc, SmallCoarse<D>* lc) {
  constexpr bool kNarrow = D == 128;  // 16x16x32 matrix instructions, else 32x32x16
  using TL = std::conditional_t<kNarrow, NarrowTile<D>, Tile<D>>;
  using UL = UNITS<TL>;
  using UC = UnitCopy<TL, UL>;
  constexpr int CPR = TL::CPR, KS = D / 16, DVB = D / 32;
  constexpr int HALF = DqShape<D, NW>::HALF;
  constexpr int NC = UC::NC;            // copy instructions per 32 rows
  constexpr int G = KS;                 // matrix instructions of a group
  constexpr int OS = D;
  // blocks of the matrix instruction's size: columns of d, queries
  constexpr int MT = kNarrow ? 16 : 32, XB = D / MT, QB = kTile / MT, AV = kNarrow ? 4 : 16, CS = D / (kNarrow ? 32 : 16);
  using Acc = std::conditional_t<kNarrow, f32x4, f32x16>;
  static_assert(HALF % 256 == 0, "the operand addresses XOR the bits below 256");
  static_assert(G == 2 * DVB && G == NC && G % 4 == 0, "phase interleave: one copy instruction per matrix instruction");
  static_assert(!COARSE || 64 * NW == kSmallThreads, "the coarse backward takes 256 threads");

  // (as in the forward kernel: the first `pairs` workgroups take two blocks; with K = Nc plain blockIdx order and staggered walks)
  const int tiles = (K + UL::kEntriesPerTile - 1) / UL::kEntriesPerTile;
  const bool same_lists = K == Nc * UL::kEntriesPerTile;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5, l16 = lane & 15, g16 = lane >> 4;
  const bool paired = PAIRS && block < pairs;
  const unsigned from = paired ? 0u : pairs, those = paired ? pairs : grid - pairs;
  const unsigned id = same_lists ? block - from : xcd_chunked_id(block - from, those);
  const unsigned wg = paired ? 2 * id + wave : 2 * pairs + id;
  if (paired && wg >= blocks) return;  // (an odd number of blocks)
  const int c = wg % Nc;
  const long long bh = wg / Nc;
  const int rot = same_lists ? ((paired ? c >> 4 : c >> 3) & 15) % tiles : 0;
  const int nu = paired ? 2 * tiles : tiles > (wave >> 1) ? (tiles - (wave >> 1) + NW / 2 - 1) / (NW / 2) : 0;
  auto tile_of = [&](int u) {
    const int t = (paired ? u >> 1 : (wave >> 1) + (NW / 2) * u) + rot;
    return t >= tiles ? t - tiles : t;
  };
  auto half_of = [&](int u) { return (paired ? u : wave) & 1; };
  const long long rows0 = bh * (long long)Nc * kTile;
  const unsigned char* kb = (const unsigned char*)uniform_ptr(k + rows0 * CPR);
  const unsigned char* vb = (const unsigned char*)uniform_ptr(v + rows0 * CPR);

  // dQ and the resident operands: accumulation registers where the kernel has them (one wavefront per SIMD)
  auto pin_acc = [](Acc& acc) {
    if (D == 128) asm volatile("" : "+a"(acc));
    else asm volatile("" : "+v"(acc));
  };
  auto pin_op = [](bf16x8& op) {
    if (D == 128) asm volatile("" : "+a"(op));
    else asm volatile("" : "+v"(op));
  };

  // Start-up: the list, Q, dO_f and the row terms (one round trip), then the key masks and the first two units, of
  // which the first products need the first alone.  Q and dO_f wait in stages: a wavefront of its own block has all of
  // them (and the copies of its first unit behind them), where a block is shared the first two wavefronts have one half
  // each in their second stages.
  UC copy;
  copy.init(lane);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem)) + (unsigned)wave * (4 * HALF);
  UL list;
  if (!PAIRS) list.only = wave & 1;
  list.request(idx + (bh * Nc + c) * (long long)K, mask, K, lane, Nc, nu > 0 ? tile_of(0) : 0);
  Unit un[3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // the current unit and the two after it
  const long long q0 = rows0 + (long long)c * kTile;  // first row of this query block
  {
    UnitCopy<TL, CubeUnits<TL>> cq;
    cq.init(lane);
    const unsigned char* qb = (const unsigned char*)uniform_ptr(q + q0 * CPR);
    const unsigned char* db = (const unsigned char*)uniform_ptr(dof + q0 * CPR);
    const Unit lo = {0, HALF / 2, 0}, hi = {HALF, HALF + HALF / 2, 0};
    if (paired) {
      cq.all(qb, lo, lds0 + 3 * HALF);
      cq.all(qb, hi, lds0 + 2 * HALF);
      cq.all(db, lo, lds0 + HALF);
      cq.all(db, hi, lds0);
    } else if (NW == 2 || wave < 2) {
      cq.all(qb, wave & 1 ? hi : lo, lds0 + 3 * HALF);
      cq.all(db, wave & 1 ? hi : lo, lds0 + HALF);
    }
  }
  // row terms of the lane's two query columns: -lse*log2(e)/sl2 (-30000 on pad rows: then P = 0 and the row
  // contributes nothing) and -Delta
  float nlse[QB], ndelta[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) {  // (per 32 rows: 32 of the first, 32 of the second)
    const float* qterm = rowd + 2 * q0 + (kNarrow ? 64 * (b >> 1) + 16 * (b & 1) + l16 : 64 * b + l32);
    nlse[b] = qterm[0], ndelta[b] = qterm[32];
  }
  list.arrived();
  const unsigned ml0 = __builtin_amdgcn_readfirstlane(lds_address(masks)) + (unsigned)wave * 512u;
  request_masks(list, ml0);
  auto copy_first = [&]() {
    list.rows(tile_of(0), half_of(0), un[0]);
    copy.all(kb, un[0], lds0);
    copy.all(vb, un[0], lds0 + 2 * HALF);
  };
  if (!paired && nu > 0) copy_first();
  Acc acc[XB][QB];
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int i = 0; i < AV; ++i) acc[x][b][i] = 0.f;
#pragma unroll
  for (int x = 0; x < XB; ++x)  // (zeroed once, right here, while the first copies are in flight)
#pragma unroll
    for (int b = 0; b < QB; ++b) pin_acc(acc[x][b]);
#pragma unroll
  for (int b = 0; b < QB; ++b) asm volatile("" : "+v"(nlse[b]), "+v"(ndelta[b]));
  if (COARSE) small_coarse_bwd<D, false>(*lc, Nc, c, bh * Nc, scale, sc.qc, sc.kc, sc.vc, sc.doc, sc.lse_c, sc.dot, tid);
  wait_vmcnt<0>();
  __builtin_amdgcn_sched_barrier(0);
  if (!paired) __syncthreads();
  bf16x8 qreg[QB][CS], doreg[QB][CS];  // [queries][contraction step]
  {
    // halves of a wavefront's own: stages 3 and 2 (Q), 1 and 0 (dO_f); shared: stages 3 and 1 of the first two wavefronts
    const unsigned char* base = smem + (paired ? wave * (4 * HALF) : 0);
    const unsigned char* base1 = paired ? base - HALF : base + 4 * HALF;
    if constexpr (kNarrow) {
      const int lane_q = TL::rowmajor_lane(lane);
#pragma unroll
      for (int s = 0; s < CS; ++s)
#pragma unroll
        for (int b = 0; b < QB; ++b) {
          qreg[b][s] = TL::rowmajor_at((b < 2 ? base : base1) + 3 * HALF, lane_q, b & 1, s);
          doreg[b][s] = TL::rowmajor_at((b < 2 ? base : base1) + HALF, lane_q, b & 1, s);
        }
    } else {
      const int lane_q = TL::rowmajor_lane(0, lane);
#pragma unroll
      for (int s = 0; s < CS; ++s) {
        qreg[0][s] = TL::rowmajor_at(base + 3 * HALF, lane_q, s);
        qreg[1][s] = TL::rowmajor_at(base1 + 3 * HALF, lane_q, s);
        doreg[0][s] = TL::rowmajor_at(base + HALF, lane_q, s);
        doreg[1][s] = TL::rowmajor_at(base1 + HALF, lane_q, s);
      }
    }
  }
#pragma unroll
  for (int b = 0; b < QB; ++b)
#pragma unroll
    for (int s = 0; s < CS; ++s) {
      pin_op(qreg[b][s]);
      pin_op(doreg[b][s]);
    }
  if (!paired) __syncthreads();  // every wavefront has Q and dO_f: the second stages may be filled
  take_masks(list, masks + wave * 128);
  if (paired && nu > 0) copy_first();
  if (nu > 0) list.get(tile_of(0), half_of(0), un[0]);
  if (nu > 1) {
    list.get(tile_of(1), half_of(1), un[1]);
    copy.all(kb, un[1], lds0 + HALF);
    copy.all(vb, un[1], lds0 + 3 * HALF);
    wait_vmcnt<2 * NC>();  // the first unit has landed; newer: the second
  } else {
    wait_vmcnt<0>();
  }
  __builtin_amdgcn_sched_barrier(0);

  const int my = wave * (4 * HALF);
  // all units: `body(kind, own, par, u)` is one.  KIND 2: the units up to u + 2 exist; 1: u + 1 exists; 0: u is the last one.  OWN: the
  // wavefront has a block of its own (then the half of a unit of the steady walk is known: `par`).  `par` = u & 1.
  auto walk = [&](auto body) {
    if (nu == 0) return;
    const std::integral_constant<int, 2> steady;
    const std::integral_constant<int, 1> inner;
    const std::integral_constant<int, 0> last;
    const std::true_type own;
    const std::false_type shared;
    int u = 0;
    if constexpr (PAIRS && kNarrow) {
      if (paired)
        for (; u + 3 < nu; u += 2) {
          body(steady, own, 0, u);
          body(steady, own, 1, u + 1);
        }
    }
    if (!(PAIRS && kNarrow && paired))
      for (; u + 3 < nu; u += 2) {  // (kNarrow: the unit itself gets that after the next, in parts)
        if (!kNarrow) list.get(tile_of(u + 2), half_of(u + 2), un[2]);
        body(steady, shared, 0, u);
        if (!kNarrow) list.get(tile_of(u + 3), half_of(u + 3), un[2]);
        body(steady, shared, 1, u + 1);
      }
    for (; u + 1 < nu; ++u) {
      if (u + 2 < nu) list.get(tile_of(u + 2), half_of(u + 2), un[2]);
      body(inner, shared, u & 1, u);
    }
    body(last, shared, u & 1, u);
  };
  if constexpr (kNarrow) {
  using TK = DqTicks;
  constexpr TK ticks;
  constexpr int PH = TK::PH;
  const int lane_a = TL::rowmajor_lane(lane) + my, lane_b = TL::transposed_lane(lane) + my;
  float crow[QB];
  f32x4 dinit[QB];  // -Delta of the lane's query columns: the initial values of dP^T
#pragma unroll
  for (int b = 0; b < QB; ++b) {
    crow[b] = nlse[b] * sl2;
    dinit[b] = {ndelta[b], ndelta[b], ndelta[b], ndelta[b]};
    asm volatile("" : "+v"(dinit[b]));
  }
  // Pad keys never take part: their rows of S^T start from a large negative value (keys 16*a + 4*g16 ..), all others from zero.
  f32x4 sinit[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
  asm volatile("" : "+v"(sinit[0]), "+v"(sinit[1]));
  uint32_t all_valid = 0xffffffffu;  // what sinit was made for: this unit's valid keys and the next's
  // Operand i of K and of V: key rows 16*(i%2) .., contraction step i/2.
  bf16x8 ka[KS];  // K rows, read during the dQ products of the unit before
  if (nu > 0) {
#pragma unroll
    for (int i = 0; i < KS; ++i) ka[i] = TL::rowmajor_at(smem, lane_a, i & 1, i >> 1);
  }
  int next_tile = nu > 2 ? tile_of(1) : 0;  // tile of the unit that is fetched next in the steady walk
  walk([&](auto kind_tag, auto own_tag, int par, int u) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool OWN = decltype(own_tag)::value;
    constexpr bool more1 = KIND >= 1;
    const bool more2 = KIND == 2 || (KIND == 1 && u + 2 < nu);
    const unsigned char *kc = smem + par * HALF, *vc = smem + (2 + par) * HALF, *kn = smem + (1 - par) * HALF;  // K(u), V(u), K(u+1)
    const unsigned k_at = lds0 + par * HALF, v_at = lds0 + (2 + par) * HALF;
    bf16x8 va[KS];
    bf16x4 kt[KS][2];         // K^T, columns 16 x ..
    f32x4 S[2][QB], P[2][QB];  // S^T and then P^T; dP^T: [keys 16 a ..][queries 16 b ..]
    uint4 ds[QB];             // dS^T as operands
    float xf[2][2], xd[2][2];
    auto put = [](uint4& u4, int w, uint32_t x) {
      if (w == 0) u4.x = x;
      if (w == 1) u4.y = x;
      if (w == 2) u4.z = x;
      if (w == 3) u4.w = x;
    };
    // item of 16: two values of a query column, four items, the operand of 16 queries, one after the other
    auto p_ops = [&](auto from, auto count) {
      in_steps<decltype(count)::value>([&](auto number) {
        constexpr TK::Work w = ticks.pw[decltype(from)::value + decltype(number)::value];
        constexpr int it = w.item, i = 2 * (it & 1) + w.i;
        f32x4& x = S[(it >> 1) & 1][it >> 2];
        if constexpr (w.op == TK::MUL) {
          xf[it & 1][w.i] = fmaf(x[i], sl2, crow[it >> 2]);
          asm volatile("" : : "v"(xf[it & 1][w.i]));  // (pure arithmetic has no place of its own in the order: tie it to this tick)
        } else {
          const float e = fast_exp2(xf[it & 1][w.i]);
          asm volatile("" : : "v"(e));
          x[i] = e;
        }
      });
    };
    auto s_ops = [&](auto from, auto count) {
      in_steps<decltype(count)::value>([&](auto number) {
        constexpr TK::Work w = ticks.sw[decltype(from)::value + decltype(number)::value];
        constexpr int it = w.item, i = 2 * (it & 1) + w.i;
        if constexpr (w.op == TK::MUL) {
          xd[it & 1][w.i] = S[(it >> 1) & 1][it >> 2][i] * P[(it >> 1) & 1][it >> 2][i];
          asm volatile("" : : "v"(xd[it & 1][w.i]));
        } else {
          const uint32_t x = pack_bf16(xd[it & 1][0], xd[it & 1][1]);
          put(ds[it >> 2], it & 3, x);
          asm volatile("" : : "v"(x));
        }
      });
    };
    // everything of tick t but its matrix instruction
    auto ahead = [&](auto tick) {
      constexpr int t = decltype(tick)::value, n = ticks.newer[t];
      if constexpr (n >= 0) {
        wait_lgkmcnt<(n < 15 ? n : 15)>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (KIND == 2 && TK::v_copy(t) >= 0) copy.aim(v_at, TK::v_copy(t));
      if (KIND == 2 && TK::k_copy(t) >= 0) copy.aim(k_at, TK::k_copy(t));
    };
    auto behind = [&](auto tick) {
      constexpr int t = decltype(tick)::value;
      __builtin_amdgcn_sched_barrier(0);
      if (KIND == 2 && TK::v_copy(t) >= 0) copy.piece(vb, un[2], v_at, TK::v_copy(t), true);
      if (KIND == 2 && TK::k_copy(t) >= 0) copy.piece(kb, un[2], k_at, TK::k_copy(t), true);
      // (where the last units are near: all of it at once, one branch)
      if (KIND == 1 && t == TK::kFirstCopyV && more2) copy.all(vb, un[2], v_at);
      if (KIND == 1 && t == TK::kFirstCopyK && more2) copy.all(kb, un[2], k_at);
      if (KIND == 2) {  // (both halves of a tile one after the other where the block is the wavefront's own)
        const int half = OWN ? par : wave & 1;
        if (t == TK::kTile && !(OWN && half)) {
          next_tile += OWN ? 1 : NW / 2;
          if (next_tile >= tiles) next_tile -= tiles;
        }
        if (t == TK::kChunk && !(OWN && half)) list.load(next_tile);
        if (t == TK::kRows) list.rows(next_tile, half, un[2]);
        if (t == TK::kValid) list.valid(next_tile, half, un[2]);
      }
      if (more1 && t == TK::kRowsReady) {  // K(u+1) and V(u+1) have landed; newer: V(u+2) and K(u+2), as far as requested
        if (more2) wait_vmcnt<NC + (KIND == 2 ? TK::k_copies_before(TK::kRowsReady) : NC)>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int n = ticks.issued[t + 1] - ticks.issued[t];
      static_assert(n <= 1, "at most one");
      if constexpr (n == 1) {
        constexpr TK::Read r = ticks.r[ticks.issued[t]];
        if constexpr (r.kind == TK::V) va[r.i] = TL::rowmajor_at(vc, lane_a, r.i & 1, r.i >> 1);
        if constexpr (r.kind == TK::K_T) kt[r.i][r.part] = TL::transposed_half(kc, lane_b, r.i, r.part);
        if constexpr (r.kind == TK::K_NEXT && more1) ka[r.i] = TL::rowmajor_at(kn, lane_a, r.i & 1, r.i >> 1);
      }
      p_ops(std::integral_constant<int, ticks.p[t]>{}, std::integral_constant<int, ticks.p[t + 1] - ticks.p[t]>{});
      s_ops(std::integral_constant<int, ticks.s[t]>{}, std::integral_constant<int, ticks.s[t + 1] - ticks.s[t]>{});
      __builtin_amdgcn_sched_barrier(0);
    };
    if (__builtin_expect((un[0].valid & all_valid) != 0xffffffffu, 0)) {
      all_valid = un[0].valid;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int i = 0; i < 4; ++i) sinit[a][i] = (un[0].valid >> (16 * a + 4 * g16 + i)) & 1 ? 0.f : kMaskBias;
      asm volatile("s_nop 1" : "+v"(sinit[0]), "+v"(sinit[1]));  // (two wait states ahead of the matrix instructions)
    }
    __builtin_amdgcn_sched_barrier(0);
    in_steps<PH>([&](auto tick) {  // ---- S
      constexpr int t = decltype(tick)::value, i = t % KS, b = t / KS;
      ahead(tick);
      if (i < 2) mfma_v_from_qa(S[i & 1][b], ka[i], qreg[b][i >> 1], sinit[i & 1]);
      else mfma_v_qa(S[i & 1][b], ka[i], qreg[b][i >> 1]);
      if (i == 5) asm volatile("" : "+v"(sinit[0]), "+v"(sinit[1]));  // (initial values are not written over while they may still be read)
      behind(tick);
    });
    in_steps<PH>([&](auto number) {  // ---- dP
      constexpr int n = decltype(number)::value, i = n % KS, b = n / KS;
      const std::integral_constant<int, PH + n> tick;
      ahead(tick);
      if (i < 2) mfma_v_from_qa(P[i & 1][b], va[i], doreg[b][i >> 1], dinit[b]);
      else mfma_v_qa(P[i & 1][b], va[i], doreg[b][i >> 1]);
      if (i == 5) asm volatile("" : "+v"(dinit[b]));
      behind(tick);
    });
    in_steps<PH>([&](auto number) {  // ---- dQ
      constexpr int n = decltype(number)::value, x = n % KS, b = n / KS;
      const std::integral_constant<int, 2 * PH + n> tick;
      ahead(tick);
      mfma_a(acc[x][b], __builtin_shufflevector(kt[x][0], kt[x][1], 0, 1, 2, 3, 4, 5, 6, 7), __builtin_bit_cast(bf16x8, ds[b]));
      behind(tick);
    });
    un[0] = un[1];
    un[1] = un[2];
  });
  } else {
  const int lane_a = TL::rowmajor_lane(0, lane) + my;
  int lane_b0, lane_b1;
  TL::transposed_lane(0, lane, lane_b0, lane_b1);
  lane_b0 += my;
  lane_b1 += my;
  const float crow[2] = {nlse[0] * sl2, nlse[1] * sl2};
  f32x16 zero16;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero16[i] = 0.f;

  bf16x8 ka[KS];  // K rows, read during the last group of the unit before
  if (nu > 0) {
#pragma unroll
    for (int s = 0; s < KS; ++s) ka[s] = TL::rowmajor_at(smem, lane_a, s);
  }

  walk([&](auto kind_tag, auto, int par, int u) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool more1 = KIND >= 1;
    const bool more2 = KIND == 2 || (KIND == 1 && u + 2 < nu);
    const unsigned char* kc = smem + par * HALF;        // K(u)
    const unsigned char* vc = smem + (2 + par) * HALF;  // V(u)
    bf16x8 va[KS], kt[2 * DVB];
    f32x16 S[2], P[2];  // S^T and then P^T; dP^T
    uint4 ds[2][2];     // dS^T as operands: [query half][contraction step]
    auto put = [](uint4& u4, int w, uint32_t x) {
      if (w == 0) u4.x = x;
      if (w == 1) u4.y = x;
      if (w == 2) u4.z = x;
      if (w == 3) u4.w = x;
    };
    // items 0..7 of a query half, two values each; the first four make up contraction step 0
    auto p_items = [&](int b, int from, int to) {
#pragma unroll
      for (int it = from; it < to; ++it) {
        float x0 = fast_exp2(fmaf(S[b][2 * it], sl2, crow[b])), x1 = fast_exp2(fmaf(S[b][2 * it + 1], sl2, crow[b]));
        asm volatile("" : "+v"(x0), "+v"(x1));  // (pure arithmetic has no place of its own in the order: tie it to this step)
        S[b][2 * it] = x0;
        S[b][2 * it + 1] = x1;
      }
    };
    auto d_items = [&](int b, int from, int to) {
#pragma unroll
      for (int it = from; it < to; ++it) {
        const float p0 = P[b][2 * it] + ndelta[b], p1 = P[b][2 * it + 1] + ndelta[b];
        const uint32_t x = pack_bf16(S[b][2 * it] * p0, S[b][2 * it + 1] * p1);
        put(ds[b][it >> 2], it & 3, x);
        asm volatile("" : : "v"(x));
      }
    };
    // pad keys never take part: one extra matrix step adds a large negative bias to their rows of S^T
    auto bias = [&](int b) {
      if (__builtin_expect(un[0].valid != 0xffffffffu, 0)) {
        int ln = threadIdx.x & 63;
        asm volatile("" : "+v"(ln));  // (built here, not held in registers across the loop)
        const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
        bf16x8 ab = zero8, ones_b = zero8;
        ones_b[0] = ln < 32 ? (__bf16)1.f : (__bf16)0.f;
        ab[0] = (ln < 32 && !((un[0].valid >> (ln & 31)) & 1)) ? (__bf16)kMaskBias : (__bf16)0.f;
        S[b] = mfma32(ab, ones_b, S[b]);
      }
    };
    // the share of `n` items that step m of the steps [lo, hi) of a group does: [from, to)
    auto share = [](int n, int m, int lo, int hi) { return m < lo ? 0 : (m >= hi ? n : n * (m - lo) / (hi - lo)); };
    __builtin_amdgcn_sched_barrier(0);
    // the groups of matrix instructions; `with(m)` is the rest of step m
    auto s_group = [&](int b, auto with) {
#pragma unroll
      for (int m = 0; m < G; ++m) {
        if (b == 0 && m == 0) wait_lgkmcnt<G / 2>();      // the first half of the K operands; newer: the second
        if (b == 0 && m == G / 2) wait_lgkmcnt<G / 2>();  // the second half; newer: the V operands read so far
        S[b] = mfma32(ka[m], qreg[b][m], m == 0 ? zero16 : S[b]);
        if (b == 0) va[m] = TL::rowmajor_at(vc, lane_a, m);
        with(m);
        __builtin_amdgcn_sched_barrier(0);
      }
      bias(b);
    };
    auto d_group = [&](int b, auto with) {
      if (b == 0) wait_lgkmcnt<0>();
#pragma unroll
      for (int m = 0; m < G; ++m) {
        P[b] = mfma32(va[m], doreg[b][m], m == 0 ? zero16 : P[b]);
        if (b == 0) kt[m] = TL::transposed_at(kc, lane_b0, lane_b1, m / DVB, m % DVB);
        // the copy of V(u+2) (V(u) is in registers; where the last units are near: all of it at once, one branch)
        if (KIND == 1 && b == 1 && m == 0 && more2) copy.all(vb, un[2], lds0 + (2 + par) * HALF);
        if (KIND == 2 && b == 1) copy.piece(vb, un[2], lds0 + (2 + par) * HALF, m);
        with(m);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    // one half after the other: fewer registers, and another wavefront fills the gaps
    s_group(0, [&](int) {});
    d_group(0, [&](int m) { p_items(0, share(8, m, 1, G), share(8, m + 1, 1, G)); });
    s_group(1, [&](int m) { d_items(0, share(4, m, 1, G), share(4, m + 1, 1, G)); });
    d_group(1, [&](int m) { p_items(1, share(8, m, 1, G), share(8, m + 1, 1, G)); });
    // ---- dQ of half 0 | the rest of its dS, the first half of dS of half 1, the copy of K(u+2)
    wait_lgkmcnt<0>();
    asm volatile("s_nop 1");  // (two wait states between the last item and the matrix instruction that reads it)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < G; ++m) {
      if (KIND == 2) copy.aim(lds0 + par * HALF, m);
      mfma_v(acc[m % DVB][0], kt[m], __builtin_bit_cast(bf16x8, ds[0][m / DVB]));
      if (KIND == 1 && m == 0 && more2) copy.all(kb, un[2], lds0 + par * HALF);
      if (KIND == 2) copy.piece(kb, un[2], lds0 + par * HALF, m, true);
      d_items(0, 4 + share(4, m, 0, DVB - 1), 4 + share(4, m + 1, 0, DVB - 1));
      d_items(1, share(4, m, DVB - 1, G), share(4, m + 1, DVB - 1, G));
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- dQ of half 1 | the rest of its dS, the K operands of the next unit
    if (more1) {  // K(u+1) and V(u+1) have landed; newer: V(u+2) and K(u+2)
      if (more2) wait_vmcnt<2 * NC>();
      else wait_vmcnt<0>();
    }
    asm volatile("s_nop 1");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < G; ++m) {
      // (behind the last unit no operand reads lie between the last item of step 1 and the matrix instruction that reads it)
      if (!more1 && m == DVB) asm volatile("s_nop 1");
      mfma_v(acc[m % DVB][1], kt[m], __builtin_bit_cast(bf16x8, ds[1][m / DVB]));
      d_items(1, 4 + share(4, m, 0, DVB - 1), 4 + share(4, m + 1, 0, DVB - 1));
      if (more1) ka[m] = TL::rowmajor_at(smem + (1 - par) * HALF, lane_a, m);
      __builtin_amdgcn_sched_barrier(0);
    }
    un[0] = un[1];
    un[1] = un[2];
  });
  }
  mfma_fence();  // the last matrix results land before they are read
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int b = 0; b < QB; ++b) pin_acc(acc[x][b]);
  __builtin_amdgcn_sched_barrier(0);

  // Merge the partial results of the block's wavefronts (P of them), scale, add the pooled-gradient term, store.
  const uint64_t qmask = mask[c];
  const float inv_cnt = 1.0f / (float)cube_count(mask, c, m_blocks);
  // KIND 0, 1: dQ tiled, 1 past the caches; 2: raster
  auto finish = [&](auto parts_tag, auto kind_tag) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool ONCE = KIND == 1;
    const RasterRows rows_r(raster, bh, c, CPR);
    constexpr int P = decltype(parts_tag)::value, NT = 64 * P, LPT = kTile * CPR / NT;
    static_assert(NT % CPR == 0, "a thread keeps its column chunk");
    int t = P == 1 ? lane : tid;
    asm volatile("" : "+v"(t));  // (rows worked out anew: the copies' own, kept through the walk, took private memory at d = 64)
    const int ch = t % CPR;
    float* const bufs = (float*)smem + (P == 1 ? wave * 64 * OS : 0);
    // the pooled-gradient term of this thread's column chunk, requested before the partial results go through LDS
    const float* dqcr = COARSE ? lc->sum[0] + ch * 8 : dqc + ((bh * Nc + c) / m_blocks) * D + ch * 8;  // per cube = m_blocks blocks
    const float4 pc0 = *(const float4*)dqcr, pc1 = *(const float4*)(dqcr + 4);
    if (P > 1) __syncthreads();  // every wavefront is done with its stages
    {
      float* Op = bufs + (P == 1 ? 0 : wave) * 64 * OS;
#pragma unroll
      for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int x = 0; x < XB; ++x)
#pragma unroll
          for (int g4 = 0; g4 < AV / 4; ++g4) {
            const int at = kNarrow ? merge_offset(b * 16 + l16, x * 16 + 4 * g16, OS) : merge_offset(b * 32 + l32, x * 32 + 8 * g4 + 4 * h, OS);
            *(float4*)&Op[at] = make_float4(acc[x][b][4 * g4], acc[x][b][4 * g4 + 1], acc[x][b][4 * g4 + 2], acc[x][b][4 * g4 + 3]);
          }
    }
    if (P > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();  // (a wavefront's LDS accesses stay in order)

    const float pooled[8] = {pc0.x * inv_cnt, pc0.y * inv_cnt, pc0.z * inv_cnt, pc0.w * inv_cnt,
                             pc1.x * inv_cnt, pc1.y * inv_cnt, pc1.z * inv_cnt, pc1.w * inv_cnt};
#pragma unroll
    for (int it = 0; it < LPT; ++it) {
      const int r = (it * NT + t) / CPR;
      const int m0 = merge_offset(r, ch * 8, OS), m1 = merge_offset(r, ch * 8 + 4, OS);
      float4 a = *(const float4*)(bufs + m0), b = *(const float4*)(bufs + m1);
#pragma unroll
      for (int w = 1; w < P; ++w) {
        const float4 x = *(const float4*)(bufs + w * 64 * OS + m0);
        const float4 y = *(const float4*)(bufs + w * 64 * OS + m1);
        a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
        b.x += y.x; b.y += y.y; b.z += y.z; b.w += y.w;
      }
      const float sum[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
      uint4 ov = make_uint4(0, 0, 0, 0);
      if ((qmask >> r) & 1) {
        float res[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) res[e] = fmaf(sum[e], scale, pooled[e]);
        ov = pack8(res);
      }
      if (KIND < 2) store16<ONCE>(dq + (q0 + r) * CPR + ch, ov);
      else if ((qmask >> r) & 1) dq[rows_r.at(r) + ch] = ov;
    }
  };
  const std::integral_constant<int, 1> one;
  const std::integral_constant<int, NW> all;
  const std::integral_constant<int, 0> plain;
  const std::integral_constant<int, 2> out_of_order;
  if (PAIRS && paired) raster.on ? finish(one, out_of_order) : stream ? finish(one, one) : finish(one, plain);
  else raster.on ? finish(all, out_of_order) : NW == 2 && stream ? finish(all, one) : finish(all, plain);  // (four: small launches)
}

template <int D, int NW, template <class> class UNITS, bool PAIRS>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 2) void k_fine_bwd_dq(
    int Nc, int K, float sl2, float scale, const uint4* __restrict__ q, const uint4* __restrict__ k,
    const uint4* __restrict__ v, const uint4* __restrict__ dof, const int32_t* __restrict__ idx,
    const float* __restrict__ rowd, const float* __restrict__ dqc, const uint64_t* __restrict__ mask,
    uint4* __restrict__ dq, int m_blocks, unsigned blocks, unsigned pairs, int stream, RasterMap raster) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DqShape<D, NW>::LDS];
  __shared__ uint32_t masks[NW * 128];
  dq_block<D, NW, UNITS, PAIRS, false>(smem, masks, blockIdx.x, gridDim.x, Nc, K, sl2, scale, q, k, v, dof, idx, rowd, dqc, mask, dq,
                                m_blocks, blocks, pairs, stream, raster, SmallCoarseArgs{}, nullptr);
}

// Both passes of a small problem in one launch, four wavefronts per workgroup: neither fills the chip, so they run side by
// side, dK/dV, whose walks are the longer ones, first.  COARSE: with the coarse backward (see coarse_small.h).
// Bound by latency.  32 cubes, 2 heads, d = 64, top-8: dQ 9.3, dK/dV with its reduction 14.1 and the coarse backward 7.2 us
// between events became 15.0 of one launch; the whole backward 31 -> 19 us, 64 cubes, 4 heads 0.77 to 0.94 of the time.  Not for
// larger launches: at 256 blocks each pass fills the chip by itself.
template <int D, bool COARSE, bool NARROW>
__global__ __launch_bounds__(256, 1) void k_fine_bwd_one(
    unsigned dkv_blocks, int BH, int Nc, int K, float sl2, float scale, const uint4* __restrict__ q, const uint4* __restrict__ k,
    const uint4* __restrict__ v, const uint4* __restrict__ dof, const int32_t* __restrict__ idx, const int32_t* __restrict__ col,
    const int32_t* __restrict__ order, int items, int32_t* __restrict__ split, float* parts, int cap,
    const float* __restrict__ rowd, const float* __restrict__ dqc, const float* __restrict__ dkc, const float* __restrict__ dvc,
    const uint64_t* __restrict__ mask, uint4* __restrict__ dq, uint4* __restrict__ dk, uint4* __restrict__ dv, int m_blocks,
    RasterMap raster, SmallCoarseArgs sc) {
  constexpr int LDS = DkvShape<D, 4>::LDS > DqShape<D, 4>::LDS ? DkvShape<D, 4>::LDS : DqShape<D, 4>::LDS;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[LDS];
  __shared__ uint32_t masks[4 * 128];
  __shared__ int last_run;
  __shared__ SmallCoarse<D> lc;
  if (blockIdx.x < dkv_blocks)
    dkv_block<D, 4, false, COARSE, NARROW>(smem, &last_run, blockIdx.x, BH, Nc, K, sl2, scale, q, k, v, dof, col, order, items, split, parts,
                                   cap, rowd, dkc, dvc, mask, dk, dv, m_blocks, 0, raster, sc, &lc);
  else
    dq_block<D, 4, CubeUnits, false, COARSE>(smem, masks, blockIdx.x - dkv_blocks, gridDim.x - dkv_blocks, Nc, K, sl2, scale, q, k, v, dof,
                                      idx, rowd, dqc, mask, dq, m_blocks, (unsigned)(BH * Nc), 0, 0, raster, sc, &lc);
}

bool fine_bwd_in_one(int BH, int Nc, int key_cubes_16) { return !key_cubes_16 && BH * Nc <= kDkvFourWaves; }
bool fine_bwd_with_coarse(int Nc, int m_blocks) { return m_blocks == 1 && Nc <= kSmallCubes; }

hipError_t launch_fine_bwd_one(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                               const void* dof, const int32_t* idx, const int32_t* col, const int32_t* order, int32_t* split,
                               float* parts, int cap, const float* rowd, const float* dqc, const float* dkc, const float* dvc,
                               const uint64_t* mask, void* dq, void* dk, void* dv, int m_blocks, const float* qc, const float* kc,
                               const float* vc, const float* doc, const float* lse_c, const float* dot, const RasterMap& raster, hipStream_t s) {
  const int items = Nc + cap;
  const unsigned dkv_blocks = dkv_grid(BH, items, dkv_heads_at_once(Nc, d)), grid = dkv_blocks + (unsigned)(BH * Nc);  // (dkv_grid is a multiple of 8: the XCDs stay)
  const SmallCoarseArgs sc = {qc, kc, vc, doc, lse_c, dot};
#define VSA_ONE(D_, COARSE_, NARROW_)                                                                                             \
  k_fine_bwd_one<D_, COARSE_, NARROW_><<<grid, 256, 0, s>>>(dkv_blocks, BH, Nc, K, scale * kLog2e, scale, (const uint4*)q, (const uint4*)k, \
                                                   (const uint4*)v, (const uint4*)dof, idx, col, order, items, split, parts, cap, \
                                                   rowd, dqc, dkc, dvc, mask, (uint4*)dq, (uint4*)dk, (uint4*)dv, m_blocks, raster, sc)
  const bool coarse = fine_bwd_with_coarse(Nc, m_blocks);
  if (d == 128) {
    const bool narrow = dkv_narrow(BH * Nc, K, 0);
    if (coarse && narrow) VSA_ONE(128, true, true);
    else if (coarse) VSA_ONE(128, true, false);
    else if (narrow) VSA_ONE(128, false, true);
    else VSA_ONE(128, false, false);
  } else {
    if (coarse) VSA_ONE(64, true, false);
    else VSA_ONE(64, false, false);
  }
#undef VSA_ONE
  return hipGetLastError();
}

// Up to this many query blocks, four wavefronts per workgroup, as in the forward.  (d = 64, top-33: 324 blocks 31.0 against
// 46.3 us, 432 blocks 31.9 against 46.9; d = 128, 324 blocks 48.6 against 45.0.)
template <int D>
constexpr unsigned kDqFourWaves = D == 128 ? 256 : 512;

FineRoute fine_bwd_dq_route(int BH, int Nc, int d) {
  const unsigned grid = (unsigned)(BH * Nc);
  if (grid <= (d == 128 ? kDqFourWaves<128> : kDqFourWaves<64>)) return {4, 0};
  return {2, paired_workgroups(grid, d == 128 ? 512 : 1024)};
}

hipError_t launch_fine_bwd_dq(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                              const void* dof, const int32_t* idx, const float* rowd,
                              const float* dqc, const uint64_t* mask, void* dq, int m_blocks, int key_cubes_16,
                              const RasterMap& raster, hipStream_t s) {
  const float sl2 = scale * kLog2e;
  const unsigned grid = (unsigned)(BH * Nc);
  const int stream = (long long)grid * kTile * d * 2 >= kStreamBytes;
  const FineRoute route = fine_bwd_dq_route(BH, Nc, d);
  const bool four = route.waves == 4;
  const unsigned pairs = route.pairs;
#define VSA_DQ(D_, NW_, LIST_)             \
  do {                                     \
    if (NW_ == 2 && pairs) VSA_DQ_AS(D_, NW_, LIST_, (NW_ == 2)); \
    else VSA_DQ_AS(D_, NW_, LIST_, false); \
  } while (0)
#define VSA_DQ_AS(D_, NW_, LIST_, PAIRS_)                                                                               \
  k_fine_bwd_dq<D_, NW_, LIST_, PAIRS_><<<workgroups(grid, pairs), 64 * NW_, 0, s>>>(Nc, K, sl2, scale, (const uint4*)q, (const uint4*)k, (const uint4*)v, \
                                                (const uint4*)dof, idx, rowd, dqc, mask, (uint4*)dq, m_blocks, grid, pairs, stream, raster)
  if (key_cubes_16) {  // K counts key cubes of 16 tokens
    if (d == 128 && four) VSA_DQ(128, 4, SubCubeUnits);
    else if (d == 128) VSA_DQ(128, 2, SubCubeUnits);
    else if (four) VSA_DQ(64, 4, SubCubeUnits);
    else VSA_DQ(64, 2, SubCubeUnits);
  } else {  // (with 256 blocks and fewer: launch_fine_bwd_one)
    if (d == 128) VSA_DQ(128, 2, CubeUnits);
    else if (four) VSA_DQ(64, 4, CubeUnits);
    else VSA_DQ(64, 2, CubeUnits);
  }
#undef VSA_DQ
#undef VSA_DQ_AS
  return hipGetLastError();
}

}  // namespace vsa
