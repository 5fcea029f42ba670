// Fine stage backward, dK/dV pass (the formulas are in fine_bwd.hip): key-block-major over the transposed
// block map.  The body of a workgroup; the kernels are in fine_bwd_dkv.hip and, for small launches, fine_bwd.hip.
#pragma once
#include <type_traits>

#include "coarse_small.h"
#include "ticks.h"
#include "unit_stream.h"
#include "vsa_kernels.h"

namespace vsa {

// Key cubes of 16 tokens: the pooled-gradient term of row r of a key block, chunk ch -- the pooled
// gradient of the row's key cube (rows 4*block .. 4*block+3 of `pooled`) over the cube's valid tokens.
__device__ __forceinline__ void subcube_pooled_term(const float* __restrict__ pooled, long long first_row, uint64_t kmask,
                                                    int r, int D, int ch, float* out) {
  const int sc = 2 * (r >> 5) + ((r >> 1) & 1);
  const float inv = 1.0f / (float)__popcll(kmask & subcube_pattern(sc));  // (row r is valid: at least 1)
  const float* p = pooled + (first_row + sc) * D + ch * 8;
  const float4 p0 = *(const float4*)p, p1 = *(const float4*)(p + 4);
  out[0] = p0.x * inv; out[1] = p0.y * inv; out[2] = p0.z * inv; out[3] = p0.w * inv;
  out[4] = p1.x * inv; out[5] = p1.y * inv; out[6] = p1.z * inv; out[7] = p1.w * inv;
}

// One workgroup of NW = 2 wavefronts per (b, h, key block), two per CU (512 registers per wavefront: one
// wavefront per SIMD); NW = 4 for launches too small to fill the chip that way.  The streamed work is cut
// into UNITS of 32 query rows: wavefront w takes half w & 1 of the list entries w >> 1, (w >> 1) + NW/2, ...
// and multiplies its units with ALL 64 keys:
//   S [32 q x 64 k] = Q K^T,  dP = dO_f V^T,   P = exp2(S'),  dS = P dP',   dV += P^T dO_f,  dK += dS^T Q
// so every operand it reads from LDS is multiplied with all of them, and since nobody else reads its
// rows it copies them into stages of its own: the loop has no barrier, the wavefronts drift freely.
// dK and dV [64 x d] are 2*d accumulation registers; K stays in registers (d/2 of them), and V of the first 32 keys (d/4);
// V of the other 32 is in LDS, once for the workgroup.  S and dP (64 registers) become P and dS in place.  The NW partial
// results are added once, through LDS, at the end.
//
// The order inside a unit is the dependency order, S | dP | dV | dK: P is formed while dP is multiplied,
// dS while dV is, so the vector work hides behind matrix work without a second set of registers.
//
// NARROW (d = 128, where dkv_narrow says so): 16x16x32 instructions (128 of 16 cycles), an operand with the four 16-key blocks one after the
// other; behind each lies what DkvTicks deals to it, a read, a copy or two or three vector instructions, and P of the first 32 keys begins
// while S of the others is multiplied.  Else 32x32x16 instructions (d = 128 64, d = 64 32, of 32 cycles) in STEPS: one step = one LDS
// operand multiplied with both key halves, the operand reads of the step kAhead later, and behind either instruction a share of the
// copies and of the vector work (DkvStages).
// Why: under the power limit the chip gets 1.86 PFLOP/s out of the large instructions on N(0,1) operands and 2.11 to 2.29 out of the small ones,
// but each costs 6 cycles of issue where a large one, for the work of two, costs 4.  With so many multiplications among them, per 32 cycles of matrix
// work: 3 1.75 / 1.95, 4 1.73 / 1.92, 5 1.71 / 1.78, 6 1.65 / 1.67, 7 1.55 / 1.59 (profiles/rates_copy_matrix_permute.txt).  A unit has
// 3.9 others per 32 cycles at d = 128 (4.6 with key cubes of 16 tokens), 6.6 at d = 64, which has not been tried.  (Nor has the forward, 5.9 now, in this
// form.  With 6.5 then and two small instructions behind one another, the form that made this pass slower too, it took 254 -> 257 us, 16384 tokens,
// top-32, and 1232 -> 1302, 39936 tokens, top-78.)
// The row terms enter through the accumulators' initial value: the preprocess kernel stores -lse*log2e/sl2
// (then P = exp2(S' * sl2); -30000 on pad rows, whose P underflows to 0) and -Delta per row, and a lane
// reads those of its rows straight into the first matrix instruction's C operand.  Pad KEY rows need
// no bias: a key's products only ever meet its own rows of dK and dV, which are stored as zeros.
//
// SUB: the lists name key cubes of 16 tokens (Sec. 3.2, the 64 x 16 row of the tile-size tables).  The
// workgroup still owns a 64-row key block; its list is the union of the lists of the block's four key
// cubes, and every entry says (bits 16..19) which of them the query block selected: a large number is
// subtracted from S of the other keys (NARROW: in the initial values; else by one more matrix instruction per key half).  The
// pooled-gradient terms are per key cube.
//
// What bounds it: the clock, which falls as the matrix pipe fills, and the instructions of one wavefront.  d = 128: a unit is 128
// matrix instructions (2048 cycles of the pipe) and 251 others (291 with key cubes of 16 tokens), 2520 cycles (2720) by the costs of fine_fwd.hip; a whole launch (39936 tokens, 12
// heads, top-78) 3.21 M cycles at 1.66 GHz where the same order with 64 large instructions took 3.05 M at 1.53: a unit takes a fifth less
// energy.  Steps of 16384 tokens, top-32 964 -> 942 us, 39936 tokens, top-78 4838 -> 4764, B = 2, 16 heads, top-128 of 256 7929 -> 7705, 256-token
// cubes 933 -> 918, of which this pass is 35 to 40 %.  Two small instructions behind one another with the vector work of both behind
// them: 21 % more cycles than the large ones, and slower; behind each a share of its own, but dealt by the count of instructions: 12 % more.
// d = 64: 32 and 212 in 1480 cycles, where 55 to 70 cycles
// lie behind each matrix instruction of the dP phase and 4 to 20 behind those of S and the end of dK.  3 us of start-up and 5 us
// of merge and stores per workgroup, while nothing uses its SIMDs' matrix pipes.  d = 64 with two wavefronts per SIMD (256
// registers each, four to a workgroup; K and V in LDS) took 0.93 of the time of an earlier order (B = 2, 8 heads, top-32,
// local lists: 317 -> 296 us) where the stages take 0.96 to 0.98 of it; with stages it has not been tried.
// Before (32 keys x 32 queries per wavefront, 4 wavefronts in step, one workgroup per CU: every LDS operand fed one matrix instruction): 39936 tokens,
// 12 heads, d = 128, top-78 of 624: 2.68 -> 1.97 ms (1.22 PFLOP/s executed); 16384 tokens, top-32: 529 -> 370
// us; d = 64, B = 2, 8 heads, top-32: 485 -> 288 us.  Four wavefronts (one workgroup
// per CU, merging four partial results) instead of two: 2.20 ms, 426 us, 216 us, 349 us.
template <int D, int NW>
struct DkvShape {
  static constexpr int HALF = Tile<D>::BYTES / 2;    // 32 rows
  static constexpr int STAGE = 2 * HALF + 256;       // Q rows, dO_f rows, row terms of one unit
  static constexpr int NST = D == 128 ? 2 : 4;       // stages per wavefront
  static constexpr int LDS = HALF + NW * NST * STAGE;
};
// 32x32x16 instructions: what lies behind which of them in a unit: the P stages ahead of instruction j of the dP phase and, behind those, of the dV
// phase; the dS stages ahead of instruction j of the dV and dK phases; the copy of dO_f rows behind instruction j of the dK phase (-1: none).
template <int D>
struct DkvStages {
  static constexpr int p_at(int j) {
    constexpr int wide[32] = {1, 1, 2, 1, 2, 2, 1, 2, 1, 2, 1, 2, 1, 2, 1, 2, 2, 2, 2, 2, 1, 1}, narrow[16] = {3, 3, 3, 3, 3, 3, 3, 3, 4, 3, 3};
    return D == 128 ? wide[j] : narrow[j];
  }
  static constexpr int s_at(int j) {
    constexpr int wide[32] = {0, 0, 0, 0, 0, 0, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1}, narrow[16] = {0, 0, 0, 2, 2, 2, 2, 2, 3, 2, 2};
    return D == 128 ? wide[j] : narrow[j];
  }
  static constexpr int p(int j) { return j == 0 ? 0 : p(j - 1) + p_at(j - 1); }
  static constexpr int s(int j) { return j == 0 ? 0 : s(j - 1) + s_at(j - 1); }
  static constexpr int copy(int j) {
    constexpr int wide[16] = {-1, 0, -1, 1, -1, 2, -1, 3, 4, 5, 6, 7, -1, -1, -1, -1};
    return D == 128 ? wide[j] : j < 4 ? j : -1;
  }
};
// P of contraction step 0 (18 stages and its last conversion) ahead of dV, all of it ahead of step 1; dS likewise in dK
static_assert(DkvStages<128>::p(16) > 18 && DkvStages<128>::p(23) == 34 && DkvStages<128>::s(16) > 8 && DkvStages<128>::s(23) == 17, "d = 128");
static_assert(DkvStages<64>::p(8) > 18 && DkvStages<64>::p(11) == 34 && DkvStages<64>::s(8) > 8 && DkvStages<64>::s(11) == 17, "d = 64");

// 16x16x32 instructions: what lies behind which of the 128 (ticks) of a unit: S of the first 32 keys | S of the other 32 | dP | dV | dK.
struct DkvTicks : TickTable<128, 60> {
  static constexpr int KS = 8, PH = 4 * KS;  // LDS operands of a phase; its ticks
  static constexpr int kAhead = 4;           // Q operands of a unit that are read in the unit before
  static constexpr int kRowsReady = T - 14;  // the rows of the next unit are waited for here
  static constexpr int kRowTerms = 15;       // their copy (an M0 of its own: between two groups of copies)
  enum Kind { Q, DP_INIT, DO, V, DO_T, Q_T, S_INIT, Q_NEXT };
  // P and dS in operations, and how many of them lie ahead of tick t
  static constexpr int kPOps = 80, kSOps = 48;
  Work pw[kPOps] = {}, sw[kSOps] = {};
  int p[T + 1] = {}, s[T + 1] = {};
  // the copies of Q rows (of the S phase) and of dO_f rows (of the dK phase) behind tick t, -1: none.  A copy in 64 cycles is what the
  // four wavefronts of a compute unit get through.
  static constexpr int q_copy(int t) { return t < PH && t % 4 == 1 ? t / 4 : -1; }
  static constexpr int do_copy(int t) { return t > 3 * PH && t < 3 * PH + 16 && t % 2 == 1 ? (t - 3 * PH) / 2 : -1; }
  constexpr DkvTicks() {
    int n = 0;
    auto add = [&](int tick, int use, int kind, int i, int part) { r[n++] = Read{tick, use, kind, i, part}; };
    // Operands are waited for in pairs, 7 or 8 ticks (128 cycles) behind the request of the second one.
    add(0, 8, Q, 4, 0);
    add(1, 8, Q, 5, 0);
    add(4, 12, Q, 6, 0);
    add(5, 12, Q, 7, 0);
    add(8, PH, DP_INIT, 0, 0);
    add(10, PH, DP_INIT, 1, 0);
    for (int y = 0; y < KS / 2; ++y) {
      const int at = PH + 8 * y;
      add(y == 0 ? 12 : at - 14, at, V, 2 * y, 0);
      add(y == 0 ? 14 : at - 12, at, V, 2 * y + 1, 0);
      add(y == 0 ? 15 : at - 10, at, DO, 2 * y, 0);
      add(y == 0 ? 16 : at - 8, at, DO, 2 * y + 1, 0);
    }
    for (int ph = 2; ph < 4; ++ph)
      for (int x = 0; x < KS; ++x)
        for (int part = 0; part < 2; ++part) {
          const int at = ph * PH + 8 * (x / 2);
          add(at - 14 + 4 * (x % 2) + 2 * part, at, ph == 2 ? DO_T : Q_T, x, part);
        }
    add(T - 13, T, S_INIT, 0, 0);
    add(T - 12, T, Q_NEXT, 0, 0);
    add(T - 11, T, S_INIT, 1, 0);
    add(T - 10, T, Q_NEXT, 1, 0);
    add(T - 7, T + 4, Q_NEXT, 2, 0);
    add(T - 5, T + 4, Q_NEXT, 3, 0);
    order_reads();
    for (int t = 0; t < T; ++t) {
      if (q_copy(t) >= 0) cycles[t] += kCopy + (q_copy(t) % 4 == 0 ? kScalar : 0);
      if (do_copy(t) >= 0) cycles[t] += kCopy + (do_copy(t) % 4 == 0 ? kScalar : 0);
    }
    // P: an item's first exponential, the products of the next, the second exponential, the conversion of the item before; dS: the
    // products of an item, the conversion of the one before.
    n = 0;
    pw[n++] = {MUL, 0, 0};
    pw[n++] = {MUL, 0, 1};
    for (int g = 0; g < 16; ++g) {
      pw[n++] = {EXP, g, 0};
      if (g < 15) pw[n++] = {MUL, g + 1, 0};
      if (g < 15) pw[n++] = {MUL, g + 1, 1};
      pw[n++] = {EXP, g, 1};
      if (g > 0) pw[n++] = {CVT, g - 1, 0};
    }
    pw[n++] = {CVT, 15, 0};
    n = 0;
    for (int k = 0; k < 17; ++k) {
      if (k < 16) sw[n++] = {MUL, k, 0};
      if (k > 0) sw[n++] = {CVT, k - 1, 0};
      if (k < 16) sw[n++] = {MUL, k, 1};
    }
    // (from two instructions behind the S, the dP they need)
    deal(p, pw, kPOps, PH / 2 + 2, 2 * PH - 1);
    deal(s, sw, kSOps, 2 * PH + 2, 3 * PH - 1);
  }
  // Operations lie two instructions behind what they need and are done one instruction ahead of what needs them: S of the first 32 keys (items
  // 0 .. 7) is there at tick PH / 2, that of the others at PH, dP at 2 PH, where dV begins; dK begins at 3 PH.
  constexpr bool in_order() const {
    if (p[PH / 2 + 2] != 0 || p[2 * PH - 1] != kPOps || s[2 * PH + 2] != 0 || s[3 * PH - 1] != kSOps) return false;
    for (int n = 0; n < p[PH + 2]; ++n)
      if (pw[n].item >= 8) return false;
    return ordered(pw, kPOps) && ordered(sw, kSOps);
  }
};
static_assert(DkvTicks().in_order(), "operations of dK/dV");

// d = 128: which matrix instruction, by the number of blocks of all heads and of 64-token blocks in a query block's list.  The small one saves
// energy and costs issue slots, so the large one wins where a launch leaves SIMDs idle and power does not hold the clock.  Time of the pass with the large
// instruction over that with the small one, both in turn in one process, three sets of inputs, iid lists, top-k (from run to run 0.005; one build against
// another moves kernels of 15 to 50 us by 0.01 to 0.02 by where their code lies):
//   one launch    (with dQ) 32 blocks, k 4 0.984, 8 0.984, 32 0.981 (29.6 / 30.1 us); 64 in heads of 32, 2 0.987, 8 0.987, 32 0.994, of 64, 8 0.988, 16 0.994, 64
//                 0.987; 96, 8 0.982 and 0.987, 12 0.993, 16 0.997 and 0.985, 32 0.999, 96 1.009; 128 in heads of 32, 8 0.989, 16 1.010, of 64, 8 0.994, 16
//                 0.999, 24 1.009, 64 1.020, of 128, 8 0.988, 12 0.996, 16 1.012, 128 1.026; 160, 4 0.994, 8 1.003; 192 in heads of 32, 8 0.994, of 192, 8 1.014, 64
//                 1.034; 256 in heads of 32, 8 0.994, of 64, 8 0.992, 64 1.033, of 256, 8 1.054, 128 1.031
//   two launches  288, 4 0.976, 8 0.986 to 0.997, 12 1.000, 16 1.001, 96 1.018; 320, 4 0.969, 8 0.987 and 1.002, 12 0.995, 16 1.013; 384 in heads of 32 to 192, 4 0.985
//                 to 0.996, 6 0.989 to 0.996, 8 0.989 to 1.001, 10 1.009, 16 1.020; 448, 8 0.998, 64 1.061; 512, 8 1.009 to 1.022; 768, 8 1.018
//   64 x 16       32, top-16 0.988, 64 0.965; 64, 32 0.991, 128 0.961; 128, 32 0.984, 64 0.967, 256 0.961 (81.4 / 84.7 us); 192, 32 1.004; 256, 64 1.004 and 1.009;
//                 288, 16 0.995, 32 0.969, 64 0.964, 256 0.965; 320, 32 0.975; 384, 24 0.991, 32 0.989 and 1.001; 448, 32 0.991, 64 1.013; 512, 64 1.007; 1024, 64 1.040
inline bool dkv_narrow(int blocks, int entries, int key_cubes_16) {
  if (key_cubes_16) return blocks > 384;
  if (blocks <= kDkvFourWaves) return blocks > 64 && blocks * entries > 1536;
  return blocks > 384 || entries > 8;
}

// What the coarse backward of a short sequence is formed from (see coarse_small.h).
struct SmallCoarseArgs {
  const float *qc, *kc, *vc, *doc, *lse_c, *dot;
};

// Two floats that workgroups of other XCDs read, or wrote, in the same launch.
__device__ __forceinline__ void store_shared(float* p, float x, float y) {
  const uint64_t v = (uint64_t)__float_as_uint(x) | ((uint64_t)__float_as_uint(y) << 32);
  __hip_atomic_store((uint64_t*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 load_shared(const float* p) {
  const uint64_t v = __hip_atomic_load((const uint64_t*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}

// `smem`: DkvShape::LDS bytes, aligned to 1024.  COARSE: the pooled-gradient terms are formed here (NW = 4, cubes of one block),
// in `lc`, and dkc, dvc are not read.
template <int D, int NW, bool SUB, bool COARSE, bool NARROW>
__device__ __forceinline__ void dkv_block(unsigned char* smem, int* last_run, unsigned block, int BH, int Nc, int K, float sl2, float scale,
                                          const uint4* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
                                          const uint4* __restrict__ dof, const int32_t* __restrict__ col,
                                          const int32_t* __restrict__ order, int items_per_bh, int32_t* __restrict__ split,
                                          float* parts, int cap, const float* __restrict__ rowd,
                                          const float* __restrict__ dkc, const float* __restrict__ dvc,
                                          const uint64_t* __restrict__ mask, uint4* __restrict__ dk, uint4* __restrict__ dv,
                                          int m_blocks, int stream, const RasterMap& raster, const SmallCoarseArgs& sc,
                                          SmallCoarse<D>* lc) {
  using TL = std::conditional_t<NARROW, NarrowTile<D>, Tile<D>>;
  using SH = DkvShape<D, NW>;
  constexpr int CPR = TL::CPR, KS = D / 16, DVB = D / 32, NT = 64 * NW, LPT = kTile * CPR / NT;
  constexpr int EPR = NW / 2;              // list entries a round of units takes
  constexpr int HALF = SH::HALF, STAGE = SH::STAGE, NST = SH::NST;
  constexpr int NC = HALF / 1024;          // copy instructions per 32 rows
  constexpr int kAhead = NARROW ? DkvTicks::kAhead : 2;  // Q operands that are read ahead of their unit
  constexpr int NCD = 2 * DVB;             // steps of the dV and of the dK phase
  constexpr int OS = D;
  static_assert(HALF % 256 == 0 && STAGE % 256 == 0, "the operand addresses XOR the bits below 256");
  static_assert(KS == NCD && NC == KS && (!NARROW || KS == DkvTicks::KS), "phase interleave");
  static_assert(!NARROW || D == 128, "the small instruction has tables for d = 128");
  static_assert(!COARSE || (NT == kSmallThreads && !SUB), "the coarse backward takes 256 threads");

  // Start-up: one descriptor load (key block, begin and end of its run of the block's list, slot; the
  // items of a (b, h) come longest first), then the list chunk, then the first copies, then the resident
  // K rows.  A list longer than the split length is shared by several workgroups, each of which leaves
  // its fp32 partial sums in its slot (run_word in desc.w) and the last of which to arrive adds all of them, in slot
  // order; unused descriptors carry block -1.
  int bh_, item;
  dkv_item(block, BH, items_per_bh, dkv_heads_at_once(Nc, D), bh_, item);
  if (item >= items_per_bh) return;
  const long long bh = bh_;
  const int4 desc = ((const int4*)order)[bh * items_per_bh + item];
  if (desc.x < 0) return;
  const int j = desc.x, beg = desc.y, n = desc.z - desc.y, slot = run_slot(desc.w);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5, l16 = lane & 15, g16 = lane >> 4;
  const long long rows0 = bh * (long long)Nc * kTile;
  const int32_t* my_col = col + bh * (long long)Nc * K + beg;
  const uint64_t kmask = mask[j];

  // The list sits in a register, 64 entries at a time (lane e holds entry e of the current chunk).
  int chunk = 0;
  int col_v = n > 0 ? my_col[list_slot(0, lane, n)] : 0;
  asm volatile("" : "+v"(col_v));
  const int first = wave >> 1, half = wave & 1;  // this wavefront's entries: first, first + EPR, ...
  const int nu = n > first ? (n - first + EPR - 1) / EPR : 0;
  auto load_chunk = [&](int u) {  // that of unit u (ascending u)
    const int e = first + EPR * u;
    if (__builtin_expect((e >> 6) != chunk, 0)) {
      chunk = e >> 6;
      col_v = my_col[list_slot(chunk, lane, n)];
      asm volatile("" : "+v"(col_v));  // its wait stays inside this branch
    }
  };
  auto entry_of = [&](int u) { return __builtin_amdgcn_readlane(col_v, (first + EPR * u) & 63); };
  auto entry = [&](int u) {  // list entry of unit u
    load_chunk(u);
    return entry_of(u);
  };
  // a unit's bytes: its block's offset from this wavefront's first rows of the (b, h) (at most 4096 blocks of 16 KiB)
  auto unit_off = [&](int raw) { return (unsigned)(SUB ? raw & 0xffff : raw) * (unsigned)TL::BYTES; };
  const unsigned char* qw = (const unsigned char*)uniform_ptr(q + (rows0 + half * 32) * CPR);
  const unsigned char* dw = (const unsigned char*)uniform_ptr(dof + (rows0 + half * 32) * CPR);
  const unsigned char* rw = (const unsigned char*)uniform_ptr(rowd + 2 * (rows0 + half * 32));  // 32 + 32 floats per 32 rows
  constexpr int ROWD_SHIFT = D == 128 ? 5 : 4;  // bytes of a block's Q rows / bytes of its row terms

  // Copies (see UnitCopy): instruction c of 32 rows fills rows c*RPI ..; the swizzle repeats after
  // 16 rows = 4 KiB (d = 128), so four lane offsets serve and the second group moves both bases by 4 KiB.
  constexpr int NOFF = NC < 4 ? NC : 4;
  unsigned goff[NOFF];
#pragma unroll
  for (int i = 0; i < NOFF; ++i) {
    const int r = i * TL::RPI + lane / CPR, pc = lane % CPR;
    goff[i] = (unsigned)((r * CPR + (pc ^ TL::swz(r))) * 16) - (unsigned)i * 1024u;
  }
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem));
  const unsigned wbase = lds0 + HALF + (unsigned)wave * (NST * STAGE);
  auto copy_aim = [&](unsigned lds, int c) {  // (another instruction between it and copy_piece)
    if ((c & 3) == 0) set_m0_ahead(lds + (c >> 2) * 4096);
  };
  auto copy_piece = [&](const void* g, unsigned lds, int c, bool aimed = false) {  // copy c of 32 rows; `g`, `lds` uniform
    const void* gb = (const unsigned char*)g + (c >> 2) * 4096;
    if ((c & 3) == 0 && !aimed) set_m0(lds + (c >> 2) * 4096);
    const int r = c & 3;
    if (r == 0) lds_dma16_at<0>(gb, goff[0]);
    if (r == 1) lds_dma16_at<1024>(gb, goff[1 % NOFF]);
    if (r == 2) lds_dma16_at<2048>(gb, goff[2 % NOFF]);
    if (r == 3) lds_dma16_at<3072>(gb, goff[3 % NOFF]);
  };
  auto copy_rows = [&](unsigned off, unsigned lds) { lds_dma4(rw + (off >> ROWD_SHIFT), (unsigned)lane * 4u, lds); };

  // K and V reach the registers through LDS as well (coalesced copies, one per workgroup): K waits in the Q
  // slots of the first two wavefronts' last stages, V of the first 32 keys in the dO_f slot of the first
  // one's, V of the last 32 keys stays where the dP products read it.
  constexpr int LAST = HALF + (NST - 1) * STAGE;  // the first wavefront's last stage
  auto copy_half = [&](const uint4* src, unsigned lds) {
    const unsigned char* g = (const unsigned char*)uniform_ptr(src);
#pragma unroll
    for (int c = 0; c < NC; ++c) copy_piece(g, lds, c);
  };
  {
    const long long kv0 = (rows0 + (long long)j * kTile) * CPR;
    if (NW == 2 || wave < 2) copy_half(k + kv0 + half * 32 * CPR, lds0 + LAST + half * (NST * STAGE));
    if (NW == 2 || wave >= 2) copy_half(v + kv0 + half * 32 * CPR, lds0 + (half ? 0 : LAST + HALF));
  }
  // the first units; the dO_f rows of the last stage follow once K and V have left it, its Q rows in the
  // first S phase, as in the loop
  int raws[NST];  // SUB: the entries of units u .. u + NST-1
  unsigned next_off = 0;  // offset of the unit whose Q rows are copied next
#pragma unroll
  for (int s = 0; s < NST; ++s) {
    raws[s] = 0;
    if (s < nu) {
      raws[s] = entry(s);
      next_off = unit_off(raws[s]);
      if (s < NST - 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c) copy_piece(dw + next_off, wbase + s * STAGE + HALF, c);
#pragma unroll
        for (int c = 0; c < NC; ++c) copy_piece(qw + next_off, wbase + s * STAGE, c);
        copy_rows(next_off, wbase + s * STAGE + 2 * HALF);
      }
    }
  }
  // [columns of d][keys], in blocks of the matrix instruction's size
  constexpr int MT = NARROW ? 16 : 32, XB = D / MT, KB = kTile / MT, AV = NARROW ? 4 : 16;
  using Acc = std::conditional_t<NARROW, f32x4, f32x16>;
  Acc dka[XB][KB], dva[XB][KB];
#pragma unroll
  for (int x = 0; x < XB; ++x)
#pragma unroll
    for (int b = 0; b < KB; ++b)
#pragma unroll
      for (int i = 0; i < AV; ++i) { dka[x][b][i] = 0.f; dva[x][b][i] = 0.f; }
#pragma unroll
  for (int x = 0; x < XB; ++x)  // (zeroed once, right here, while the first copies are in flight)
#pragma unroll
    for (int b = 0; b < KB; ++b) asm volatile("" : "+a"(dka[x][b]), "+a"(dva[x][b]));
  if (COARSE) small_coarse_bwd<D, true>(*lc, Nc, j, bh * Nc, scale, sc.qc, sc.kc, sc.vc, sc.doc, sc.lse_c, sc.dot, tid);
  constexpr int G = 2 * NC + 1;  // copies of one unit
  if (nu >= NST - 1) wait_vmcnt<(NST - 1) * G>();
  else wait_vmcnt<0>();
  __syncthreads();
  // K, and V of the first 32 keys; NARROW: operand [half][i] is contraction step i / 2 of the keys 32 * half + 16 * (i % 2) ..
  bf16x8 kreg[2][KS], vreg[KS];
  {
    if constexpr (NARROW) {
      const int lane_k = TL::rowmajor_lane(lane) + LAST;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        kreg[0][s] = TL::rowmajor_at(smem, lane_k, s & 1, s >> 1);
        kreg[1][s] = TL::rowmajor_at(smem + NST * STAGE, lane_k, s & 1, s >> 1);
        vreg[s] = TL::rowmajor_at(smem + HALF, lane_k, s & 1, s >> 1);
      }
    } else {
      const int lane_k = TL::rowmajor_lane(0, lane) + LAST;
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        kreg[0][s] = TL::rowmajor_at(smem, lane_k, s);
        kreg[1][s] = TL::rowmajor_at(smem + NST * STAGE, lane_k, s);
        vreg[s] = TL::rowmajor_at(smem + HALF, lane_k, s);
      }
    }
  }
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(kreg[0][s]), "+v"(kreg[1][s]), "+v"(vreg[s]));
  __syncthreads();  // every wavefront has K and V: the last stages may be filled
  if (nu >= NST) {
#pragma unroll
    for (int c = 0; c < NC; ++c) copy_piece(dw + next_off, wbase + (NST - 1) * STAGE + HALF, c);
    wait_vmcnt<(NST - 2) * G + NC>();
  } else {
    wait_vmcnt<0>();
  }

  // all units: `body(steady, u, st)` is one, whose rows lie in the wavefront's stage `st` (a constant in the unrolled loop)
  auto walk = [&](auto body) {
    int u = 0;
    for (; u + 2 * NST - 1 < nu; u += NST) {
#pragma unroll
      for (int st = 0; st < NST; ++st) body(std::true_type{}, u + st, st);
    }
    for (; u + NST < nu; ++u) body(std::true_type{}, u, u % NST);
    for (; u < nu; ++u) body(std::false_type{}, u, u % NST);
  };
  const int wave_rows = (int)(HALF + wave * (NST * STAGE));  // this wavefront's stages
  if constexpr (NARROW) {
  using TK = DkvTicks;
  constexpr TK ticks;
  constexpr int PH = TK::PH;
  const int lane_q = TL::rowmajor_lane(lane) + wave_rows, lane_v = TL::rowmajor_lane(lane), lane_b = TL::transposed_lane(lane) + wave_rows;
  const int lane_r = wave_rows + 2 * HALF + 16 * g16;
  // initial value of an accumulator: the row terms of rows 16*b + 4*g16 ..
  auto row_init = [&](int off, int which, int b) { return *(const f32x4*)(smem + (lane_r + off) + which * 128 + b * 64); };
  bf16x8 qcur[kAhead];
  f32x4 sinit[2];
  if (nu > 0) {
#pragma unroll
    for (int s = 0; s < kAhead; ++s) {  // (in the order of the loop's)
      if (s < 2) sinit[s] = row_init(0, 0, s);
      qcur[s] = TL::rowmajor_at(smem, lane_q, s & 1, s >> 1);
    }
  }
  walk([&](auto steady_tag, int u, int st) {
    constexpr bool STEADY = decltype(steady_tag)::value;  // the units up to u + NST exist
    const bool more_q = STEADY || u + NST - 1 < nu;
    const int st_off = st * STAGE, next_st = st == NST - 1 ? 0 : st_off + STAGE;
    const int prev_st = st == 0 ? (NST - 1) * STAGE : st_off - STAGE;
    // (the addresses of V, and with key cubes of 16 all of them, are rebuilt per unit: registers are short)
    int lv = lane_v, lq = lane_q, lb = lane_b;
    asm volatile("" : "+v"(lv));
    if (SUB) asm volatile("" : "+v"(lq), "+v"(lb));
    const unsigned char *Qs = smem + st_off, *Ds = Qs + HALF, *Qn = smem + next_st;
    // Operand s of Q and dO_f: query rows 16*(s%2) .., contraction step s/2.  S and dP: [query block][key block].
    bf16x8 qa[KS], da[KS], va[KS];
    bf16x4 dt[KS][2], qt[KS][2];
    f32x4 S[2][4], P[2][4], dpinit[2], init[2][2];
#pragma unroll
    for (int s = 0; s < kAhead; ++s) qa[s] = qcur[s];
    auto reads = [&](auto number) {  // those behind tick t
      constexpr int t = decltype(number)::value;
      constexpr int n = ticks.issued[t + 1] - ticks.issued[t];
      static_assert(n <= 1, "at most one");
      if constexpr (n == 1) {
        constexpr TK::Read r = ticks.r[ticks.issued[t]];
        if constexpr (r.kind == TK::Q) qa[r.i] = TL::rowmajor_at(Qs, lq, r.i & 1, r.i >> 1);
        if constexpr (r.kind == TK::DP_INIT) dpinit[r.i] = row_init(st_off, 1, r.i);
        if constexpr (r.kind == TK::DO) da[r.i] = TL::rowmajor_at(Ds, lq, r.i & 1, r.i >> 1);
        if constexpr (r.kind == TK::V) va[r.i] = TL::rowmajor_at(smem, lv, r.i & 1, r.i >> 1);
        if constexpr (r.kind == TK::DO_T) dt[r.i][r.part] = TL::transposed_half(Ds, lb, r.i, r.part);
        if constexpr (r.kind == TK::Q_T) qt[r.i][r.part] = TL::transposed_half(Qs, lb, r.i, r.part);
        if constexpr (r.kind == TK::S_INIT) sinit[r.i] = row_init(next_st, 0, r.i);
        if constexpr (r.kind == TK::Q_NEXT) qcur[r.i] = TL::rowmajor_at(Qn, lq, r.i & 1, r.i >> 1);
      }
    };
    auto wait = [&](auto number) {
      constexpr int n = ticks.newer[decltype(number)::value];
      if constexpr (n >= 0) {
        wait_lgkmcnt<(n < 15 ? n : 15)>();
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto both = [](const bf16x4 (&x)[2]) { return __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7); };
    auto opnd = [](const uint4& x) { return __builtin_bit_cast(bf16x8, x); };
    auto put = [](uint4& u4, int w, uint32_t x) {
      if (w == 0) u4.x = x;
      if (w == 1) u4.y = x;
      if (w == 2) u4.z = x;
      if (w == 3) u4.w = x;
    };
    // P and dS in operations none of which needs the result of the one before it.  Item k of 16: two values of a key column, four
    // items, the operand of a key block, one after the other.
    uint4 pb[4], sb[4];
    float xp[2][2], xd[2][2];  // products of an item, by its parity
    auto p_ops = [&](auto from, auto count) {
      in_steps<decltype(count)::value>([&](auto number) {
        constexpr TK::Work w = ticks.pw[decltype(from)::value + decltype(number)::value];
        constexpr int it = w.item;
        f32x4& x = S[(it >> 1) & 1][it >> 2];
        if constexpr (w.op == TK::MUL) {
          xp[it & 1][w.i] = x[2 * (it & 1) + w.i] * sl2;
          asm volatile("" : : "v"(xp[it & 1][w.i]));  // (pure arithmetic has no place of its own in the order: tie it to this tick)
        } else if constexpr (w.op == TK::EXP) {
          const float e = fast_exp2(xp[it & 1][w.i]);
          asm volatile("" : : "v"(e));
          x[2 * (it & 1) + w.i] = e;
        } else {
          const uint32_t pp = pack_bf16(x[2 * (it & 1)], x[2 * (it & 1) + 1]);
          put(pb[it >> 2], it & 3, pp);
          asm volatile("" : : "v"(pp));
        }
      });
    };
    auto s_ops = [&](auto from, auto count) {
      in_steps<decltype(count)::value>([&](auto number) {
        constexpr TK::Work w = ticks.sw[decltype(from)::value + decltype(number)::value];
        constexpr int it = w.item;
        if constexpr (w.op == TK::MUL) {
          xd[it & 1][w.i] = S[(it >> 1) & 1][it >> 2][2 * (it & 1) + w.i] * P[(it >> 1) & 1][it >> 2][2 * (it & 1) + w.i];
          asm volatile("" : : "v"(xd[it & 1][w.i]));
        } else {
          const uint32_t ss = pack_bf16(xd[it & 1][0], xd[it & 1][1]);
          put(sb[it >> 2], it & 3, ss);
          asm volatile("" : : "v"(ss));
        }
      });
    };
    // ---- S, the keys 0 .. 31 first: their P begins while the others' S is multiplied
    if (SUB) {
      // key row l16 of key block b belongs to key cube 2*(b/2) + (row/2)%2 of the block's four; the rows of the others get a large
      // negative initial value
      const unsigned sel = (unsigned)(raws[0] >> 16) >> ((l16 >> 1) & 1);
      const float bias[2] = {sel & 1u ? 0.f : -30000.f, sel & 4u ? 0.f : -30000.f};
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int hf = 0; hf < 2; ++hf)
#pragma unroll
          for (int i = 0; i < 4; ++i) init[a][hf][i] = sinit[a][i] + bias[hf];
      asm volatile("s_nop 1" : "+v"(init[0][0]), "+v"(init[0][1]), "+v"(init[1][0]), "+v"(init[1][1]));  // (two wait states)
    }
    const unsigned char* gq = qw + next_off;
    int raw = 0;
    unsigned off = 0;
    in_steps<PH>([&](auto number) {
      constexpr int t = decltype(number)::value, hf = t / (PH / 2), s = t % (PH / 2) / 2, b = t & 1, copy = TK::q_copy(t);
      wait(number);
      if (copy >= 0 && more_q) copy_aim(wbase + prev_st, copy);
      f32x4& x = S[s & 1][2 * hf + b];
      const bf16x8 kop = kreg[hf][(s & ~1) | b];
      if (s < 2) mfma_v_from(x, qa[s], kop, SUB ? init[s & 1][hf] : sinit[s & 1]);
      else mfma_v(x, qa[s], kop);
      __builtin_amdgcn_sched_barrier(0);
      if (t % (PH / 2) == 5) {  // (initial values are not written over while the matrix instructions may still read them)
        if (SUB) asm volatile("" : : "v"(init[0][hf]), "v"(init[1][hf]));
        else if (hf == 1) asm volatile("" : : "v"(sinit[0]), "v"(sinit[1]));
      }
      if (copy >= 0 && more_q) copy_piece(gq, wbase + prev_st, copy, true);
      if (t == TK::kRowTerms && more_q) copy_rows(next_off, wbase + prev_st + 2 * HALF);
      // the list entry of unit u + NST, a chain of scalar instructions, in parts
      if (STEADY && t == 7) load_chunk(u + NST);
      if (STEADY && t == 10) raw = entry_of(u + NST);
      if (STEADY && t == 14) off = unit_off(raw);
      reads(number);
      p_ops(std::integral_constant<int, ticks.p[t]>{}, std::integral_constant<int, ticks.p[t + 1] - ticks.p[t]>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dP
    in_steps<PH>([&](auto number) {
      constexpr int t = PH + decltype(number)::value, s = (t - PH) / 4, b = t & 3;
      const std::integral_constant<int, t> tick;
      wait(tick);
      const bf16x8 vop = b < 2 ? vreg[(s & ~1) | (b & 1)] : va[(s & ~1) | (b & 1)];
      if (s < 2) mfma_v_from(P[s & 1][b], da[s], vop, dpinit[s & 1]);
      else mfma_v(P[s & 1][b], da[s], vop);
      __builtin_amdgcn_sched_barrier(0);
      if (t == PH + 9) asm volatile("" : : "v"(dpinit[0]), "v"(dpinit[1]));
      reads(tick);
      p_ops(std::integral_constant<int, ticks.p[t]>{}, std::integral_constant<int, ticks.p[t + 1] - ticks.p[t]>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dV
    in_steps<PH>([&](auto number) {
      constexpr int t = 2 * PH + decltype(number)::value, x = (t - 2 * PH) / 4, b = t & 3;
      const std::integral_constant<int, t> tick;
      wait(tick);
      mfma_a(dva[x][b], both(dt[x]), opnd(pb[b]));
      __builtin_amdgcn_sched_barrier(0);
      reads(tick);
      s_ops(std::integral_constant<int, ticks.s[t]>{}, std::integral_constant<int, ticks.s[t + 1] - ticks.s[t]>{});
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dK; the dO_f rows of this stage are done with: refill them (unit u + NST), then wait for the Q
    // rows of the next unit -- everything issued before this phase's copies but the dO_f, Q groups after them
#pragma unroll
    for (int s = 0; s + 1 < NST; ++s) raws[s] = raws[s + 1];
    if (STEADY) {
      raws[NST - 1] = raw;
      next_off = off;
    }
    const unsigned char* gd = dw + next_off;
    in_steps<PH>([&](auto number) {
      constexpr int t = 3 * PH + decltype(number)::value, x = (t - 3 * PH) / 4, b = t & 3, copy = TK::do_copy(t);
      static_assert(copy < 0 || t < TK::kRowsReady, "the wait counts this phase's copies");
      const std::integral_constant<int, t> tick;
      wait(tick);
      if (STEADY && copy >= 0) copy_aim(wbase + st_off + HALF, copy);
      mfma_a(dka[x][b], both(qt[x]), opnd(sb[b]));
      __builtin_amdgcn_sched_barrier(0);
      if (STEADY && copy >= 0) copy_piece(gd, wbase + st_off + HALF, copy, true);
      if (t == TK::kRowsReady) {
        const int left = nu - 1 - (u + 1);  // units after the next one
        if (STEADY) wait_vmcnt<(NST - 2) * G + NC>();
        else if (NST > 2 && left == 2) wait_vmcnt<2 * G>();
        else if (NST > 2 && left == 1) wait_vmcnt<G>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
      }
      reads(tick);
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  } else {
  // SUB: A operand (1 in contraction slot 0) and the bit of the entry that selects this lane's key cube
  bf16x8 ones_a = {0, 0, 0, 0, 0, 0, 0, 0};
  if (SUB && h == 0) ones_a[0] = (__bf16)1.f;

  const int lane_q = TL::rowmajor_lane(0, lane) + wave_rows;
  const int lane_v = TL::rowmajor_lane(0, lane);
  int lane_b0, lane_b1;
  TL::transposed_lane(0, lane, lane_b0, lane_b1);
  lane_b0 += wave_rows;
  lane_b1 += wave_rows;
  const int lane_r = wave_rows + 2 * HALF + 16 * h;

  // initial value of an accumulator: the row term of rows 8*(i/4) + 4*h + i%4
  auto row_init = [&](int off, int which) {
    f32x16 r;
    const unsigned char* p = smem + (lane_r + off) + which * 128;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const f32x4 x = *(const f32x4*)(p + 32 * g);
      r[4 * g] = x[0]; r[4 * g + 1] = x[1]; r[4 * g + 2] = x[2]; r[4 * g + 3] = x[3];
    }
    return r;
  };

  bf16x8 qcur[kAhead];  // Q operands of a unit's first steps, read during the unit before
  f32x16 sinit;
  if (nu > 0) {
    sinit = row_init(0, 0);
#pragma unroll
    for (int s = 0; s < kAhead; ++s) qcur[s] = TL::rowmajor_at(smem, lane_q, s);
  }

  walk([&](auto steady_tag, int u, int st) {
    constexpr bool STEADY = decltype(steady_tag)::value;  // the units up to u + NST exist
    const bool more_q = STEADY || u + NST - 1 < nu;
    const int st_off = st * STAGE, next_st = st == NST - 1 ? 0 : st_off + STAGE;
    const int prev_st = st == 0 ? (NST - 1) * STAGE : st_off - STAGE;
    // (the addresses of V, and with key cubes of 16 all of them, are rebuilt per unit: registers are short)
    int lv = lane_v, lq = lane_q, lb0 = lane_b0, lb1 = lane_b1;
    asm volatile("" : "+v"(lv));
    if (SUB) asm volatile("" : "+v"(lq), "+v"(lb0), "+v"(lb1));
    const unsigned char* Qs = smem + st_off;
    const unsigned char* Ds = smem + st_off + HALF;
    const unsigned char* Qn = smem + next_st;
    bf16x8 qa[KS], da[KS], va[KS];
    bf16x4 dt[NCD][2], qt[NCD][2];
    f32x16 dpinit;
#pragma unroll
    for (int s = 0; s < kAhead; ++s) qa[s] = qcur[s];
    // operand reads of step m: S steps, dP steps, dV steps, dK steps, then the S steps of the next unit; `part` 0, 1: behind the
    // first or the second matrix instruction of a step.  Row terms come with the first operands of their phase.
    auto read_part = [&](int m, int part) {
      if (m < KS) {
        if (part == 0) qa[m] = TL::rowmajor_at(Qs, lq, m);
      } else if (m < 2 * KS) {
        const int s = m - KS;
        if (s == 0 && part == 0) dpinit = row_init(st_off, 1);
        if (part == 0) da[s] = TL::rowmajor_at(Ds, lq, s);
        if (part == 1) va[s] = TL::rowmajor_at(smem, lv, s);
      } else if (m < 2 * KS + 2 * NCD) {
        const bool of_dv = m < 2 * KS + NCD;
        const int c = m - 2 * KS - (of_dv ? 0 : NCD);
        (of_dv ? dt : qt)[c][part] = TL::transposed_half(of_dv ? Ds : Qs, part ? lb1 : lb0, c / DVB, c % DVB);
      } else if (part == 0) {
        const int s = m - 2 * KS - 2 * NCD;
        if (s == 0) sinit = row_init(next_st, 0);
        qcur[s] = TL::rowmajor_at(Qn, lq, s);
      }
    };
    auto both = [](const bf16x4 (&x)[2]) { return __builtin_shufflevector(x[0], x[1], 0, 1, 2, 3, 4, 5, 6, 7); };
    // at the first matrix instruction of step m: its operands, requested two steps before, are there; newer: those of the next
    constexpr auto reads_in = [](int m) {  // reads requested in step m
      const int steps = 2 * KS + 2 * NCD, to = (m + 2 + steps) % steps;
      return (to < KS ? 1 : 2) + (to == 0 || to == KS ? 4 : 0);
    };
    // ---- S
    f32x16 s0, s1, p0, p1;
    bf16x8 bias0 = {0, 0, 0, 0, 0, 0, 0, 0}, bias1 = bias0;
    if (SUB) {
      // key row l32 of key half b belongs to key cube 2b + (row/2)%2 of the block's four
      const unsigned sel = (unsigned)(raws[0] >> 16) >> ((l32 >> 1) & 1);
      bias0[0] = (h == 0 && !(sel & 1u)) ? (__bf16)-30000.f : (__bf16)0.f;
      bias1[0] = (h == 0 && !(sel & 4u)) ? (__bf16)-30000.f : (__bf16)0.f;
    }
    const unsigned char* gq = qw + next_off;
    in_steps<KS>([&](auto number) {
      constexpr int s = decltype(number)::value;
      wait_lgkmcnt<reads_in(s - 1)>();
      __builtin_amdgcn_sched_barrier(0);
      if (more_q) copy_aim(wbase + prev_st, s);
      if (s == 0) mfma_v_from(s0, qa[0], kreg[0][0], sinit);
      else mfma_v(s0, qa[s], kreg[0][s]);
      if (more_q) copy_piece(gq, wbase + prev_st, s, true);
      read_part(s + 2, 0);
      __builtin_amdgcn_sched_barrier(0);
      if (s == 0) s1 = sinit;
      mfma_v(s1, qa[s], kreg[1][s]);
      if (s == KS - 1 && more_q) copy_rows(next_off, wbase + prev_st + 2 * HALF);
      read_part(s + 2, 1);
      __builtin_amdgcn_sched_barrier(0);
    });
    if (SUB) {
      asm volatile("s_nop 1");  // (two wait states between the moves to the bias operands and the matrix instruction)
      mfma_v(s0, ones_a, bias0);
      mfma_v(s1, ones_a, bias1);
      __builtin_amdgcn_sched_barrier(0);
    }
    // ---- dP, with P = exp2(S' sl2) of both key halves behind it.  Item k of 16: one pair of values, first
    // those of contraction step 0 of the dV products (accumulator values 0..7), then those of step 1.  The items go through
    // stages inside which neighbours do not depend on one another (see fine_fwd.hip), dealt to the matrix instructions.  P: stage 0 the products of
    // item 0; 2g + 1 the first exponential of item g and the products of the next; 2g + 2 its second, and the conversion of the
    // item before; 33 that of the last.  dS: stage k the products of item k and the conversion of the item before.
    uint4 pb[2][2], sb[2][2];
    auto put = [](uint4& u4, int w, uint32_t x) {
      if (w == 0) u4.x = x;
      if (w == 1) u4.y = x;
      if (w == 2) u4.z = x;
      if (w == 3) u4.w = x;
    };
    float xp[2][2], xd[2][2];  // products of an item, by its parity
    auto first_of = [](int it) { return 8 * (it >> 3) + 2 * (it & 3); };
    auto p_multiply = [&](int it) {
      const f32x16& S = (it >> 2) & 1 ? s1 : s0;
      const int e = first_of(it);
      xp[it & 1][0] = S[e] * sl2;
      xp[it & 1][1] = S[e + 1] * sl2;
      asm volatile("" : : "v"(xp[it & 1][0]), "v"(xp[it & 1][1]));  // (pure arithmetic has no place of its own in the order: tie it to this step)
    };
    auto p_exp = [&](int it, int i) {
      f32x16& S = (it >> 2) & 1 ? s1 : s0;
      const float x = fast_exp2(xp[it & 1][i]);
      asm volatile("" : : "v"(x));
      S[first_of(it) + i] = x;
    };
    auto p_convert = [&](int it) {
      const f32x16& S = (it >> 2) & 1 ? s1 : s0;
      const uint32_t pp = pack_bf16(S[first_of(it)], S[first_of(it) + 1]);
      put(pb[(it >> 2) & 1][it >> 3], it & 3, pp);
      asm volatile("" : : "v"(pp));
    };
    auto p_stages = [&](int from, int to) {
#pragma unroll
      for (int n = from; n < to; ++n) {
        const int g = (n - 1) >> 1;
        if (n == 0) p_multiply(0);
        else if (n == 33) p_convert(15);
        else p_exp(g, (n - 1) & 1);
        if (n > 0 && n < 33) {
          if (n & 1) {
            if (g < 15) p_multiply(g + 1);
          } else if (g > 0) {
            p_convert(g - 1);
          }
        }
      }
    };
    auto s_stages = [&](int from, int to) {
#pragma unroll
      for (int k = from; k < to; ++k) {
        if (k > 0) {
          const int it = k - 1;
          const uint32_t ss = pack_bf16(xd[it & 1][0], xd[it & 1][1]);
          put(sb[(it >> 2) & 1][it >> 3], it & 3, ss);
          asm volatile("" : : "v"(ss));
        }
        if (k < 16) {
          const f32x16& S = (k >> 2) & 1 ? s1 : s0;
          const f32x16& P = (k >> 2) & 1 ? p1 : p0;
          const int e = first_of(k);
          xd[k & 1][0] = S[e] * P[e];
          xd[k & 1][1] = S[e + 1] * P[e + 1];
          asm volatile("" : : "v"(xd[k & 1][0]), "v"(xd[k & 1][1]));
        }
      }
    };
    using DS = DkvStages<D>;
    in_steps<KS>([&](auto number) {
      constexpr int s = decltype(number)::value, m = KS + s;
      wait_lgkmcnt<reads_in(m - 1)>();
      __builtin_amdgcn_sched_barrier(0);
      if (s == 0) mfma_v_from(p0, da[0], vreg[0], dpinit);
      else mfma_v(p0, da[s], vreg[s]);
      read_part(m + 2, 0);
      p_stages(DS::p(2 * s), DS::p(2 * s + 1));
      __builtin_amdgcn_sched_barrier(0);
      if (s == 0) p1 = dpinit;
      mfma_v(p1, da[s], va[s]);
      read_part(m + 2, 1);
      p_stages(DS::p(2 * s + 1), DS::p(2 * s + 2));
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dV, contraction step 0 first; the remaining P items have to be done before step 1 begins, the dS items of
    // step 0 before the dK phase begins
    auto opnd = [](const uint4& x) { return __builtin_bit_cast(bf16x8, x); };
    constexpr int SLOTS = 2 * NCD;  // matrix instructions of a phase
    in_steps<NCD>([&](auto number) {
      constexpr int c = decltype(number)::value, m = 2 * KS + c, j = 2 * c;
      wait_lgkmcnt<reads_in(m - 1)>();
      __builtin_amdgcn_sched_barrier(0);
      mfma_a(dva[c % DVB][0], both(dt[c]), opnd(pb[0][c / DVB]));
      read_part(m + 2, 0);
      p_stages(DS::p(SLOTS + j), DS::p(SLOTS + j + 1));
      s_stages(DS::s(j), DS::s(j + 1));
      __builtin_amdgcn_sched_barrier(0);
      mfma_a(dva[c % DVB][1], both(dt[c]), opnd(pb[1][c / DVB]));
      read_part(m + 2, 1);
      p_stages(DS::p(SLOTS + j + 1), DS::p(SLOTS + j + 2));
      s_stages(DS::s(j + 1), DS::s(j + 2));
      __builtin_amdgcn_sched_barrier(0);
    });
    // ---- dK; the dO_f rows of this stage are done with: refill them (unit u + NST), then wait for the Q
    // rows of the next unit -- everything issued before this phase's copies but the dO_f, Q groups after them
#pragma unroll
    for (int s = 0; s + 1 < NST; ++s) raws[s] = raws[s + 1];
    if (STEADY) {
      raws[NST - 1] = entry(u + NST);
      next_off = unit_off(raws[NST - 1]);
    }
    const unsigned char* gd = dw + next_off;
    in_steps<SLOTS>([&](auto number) {
      constexpr int j = decltype(number)::value, c = j / 2, m = 2 * KS + NCD + c;
      if (j % 2 == 0) {
        wait_lgkmcnt<reads_in(m - 1)>();
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int copy = DS::copy(j);  // (they end before the wait for the next unit's rows)
      if (STEADY && copy >= 0) copy_aim(wbase + st_off + HALF, copy);
      mfma_a(dka[c % DVB][j % 2], both(qt[c]), opnd(sb[j % 2][c / DVB]));
      if (STEADY && copy >= 0) copy_piece(gd, wbase + st_off + HALF, copy, true);
      if (j == 2 * (NCD - kAhead)) {
        // newer than the next unit's Q group: the dO_f and Q groups of the units after it requested so far
        const int left = nu - 1 - (u + 1);  // units after the next one
        if (STEADY) wait_vmcnt<(NST - 2) * G + NC>();
        else if (NST > 2 && left == 2) wait_vmcnt<2 * G>();
        else if (NST > 2 && left == 1) wait_vmcnt<G>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
      }
      read_part(m + 2, j % 2);
      s_stages(DS::s(SLOTS + j), DS::s(SLOTS + j + 1));
      __builtin_amdgcn_sched_barrier(0);
    });
  });
  }
  asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");  // the last matrix results land before they are read
  __builtin_amdgcn_sched_barrier(0);

  // the pooled-gradient terms of this thread's column chunk (the same chunk for all of its items),
  // requested before the partial results go through LDS
  static_assert(NT % CPR == 0, "a thread keeps its column chunk");
  float4 pk[2] = {}, pv[2] = {};
  if (COARSE) {
    const float *a = lc->sum[0] + (tid % CPR) * 8, *b = lc->sum[1] + (tid % CPR) * 8;
    pk[0] = *(const float4*)a, pk[1] = *(const float4*)(a + 4);
    pv[0] = *(const float4*)b, pv[1] = *(const float4*)(b + 4);
  } else if (!SUB) {
    const float* a = dkc + ((bh * Nc + j) / m_blocks) * D + (tid % CPR) * 8;  // per cube = m_blocks blocks
    const float* b = dvc + ((bh * Nc + j) / m_blocks) * D + (tid % CPR) * 8;
    pk[0] = *(const float4*)a, pk[1] = *(const float4*)(a + 4);
    pv[0] = *(const float4*)b, pv[1] = *(const float4*)(b + 4);
  }
  const float inv_cnt = 1.0f / (float)cube_count(mask, j, m_blocks);

  // Add the partial results in wavefront order through LDS: dK, then dV.
  static_assert(NW * 64 * OS * 4 <= SH::LDS, "merge buffers must fit");
  // KIND 0, 1: dK and dV tiled, 1 past the caches; 2: raster
  auto finish = [&](auto kind_tag) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool ONCE = KIND == 1;
    const RasterRows rows_r(raster, bh, j, CPR);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      __syncthreads();
      float* bufs = (float*)smem;  // [wavefront][64][OS]
      {
        float* Op = bufs + wave * 64 * OS;
#pragma unroll
        for (int x = 0; x < XB; ++x)
#pragma unroll
          for (int b = 0; b < KB; ++b)
#pragma unroll
            for (int g4 = 0; g4 < AV / 4; ++g4) {
              const Acc& a = pass == 0 ? dka[x][b] : dva[x][b];
              const int at = NARROW ? merge_offset(b * 16 + l16, x * 16 + 4 * g16, OS) : merge_offset(b * 32 + l32, x * 32 + 8 * g4 + 4 * h, OS);
              *(float4*)&Op[at] = make_float4(a[4 * g4], a[4 * g4 + 1], a[4 * g4 + 2], a[4 * g4 + 3]);
            }
      }
      __syncthreads();
      const float4 q0 = pass == 0 ? pk[0] : pv[0], q1 = pass == 0 ? pk[1] : pv[1];
      const float pooled[8] = {q0.x * inv_cnt, q0.y * inv_cnt, q0.z * inv_cnt, q0.w * inv_cnt,
                               q1.x * inv_cnt, q1.y * inv_cnt, q1.z * inv_cnt, q1.w * inv_cnt};
      const float mul = pass == 0 ? scale : 1.0f;
      uint4* dst = pass == 0 ? dk : dv;
      float* slot_dst = parts + ((bh * cap + slot) * 2 + pass) * (long long)(64 * D);
#pragma unroll
      for (int it = 0; it < LPT; ++it) {
        const int item = it * NT + tid, r = item / CPR, ch = item % CPR;
        const int m0 = merge_offset(r, ch * 8, OS), m1 = merge_offset(r, ch * 8 + 4, OS);
        float4 a = *(const float4*)(bufs + m0), b = *(const float4*)(bufs + m1);
#pragma unroll
        for (int w = 1; w < NW; ++w) {
          const float4 x = *(const float4*)(bufs + w * 64 * OS + m0), y = *(const float4*)(bufs + w * 64 * OS + m1);
          a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
          b.x += y.x; b.y += y.y; b.z += y.z; b.w += y.w;
        }
        if (slot >= 0) {  // one run of a split list: raw fp32 sums [dK | dV][64][D], added up below
          float* o = slot_dst + r * D + ch * 8;
          store_shared(o, a.x, a.y);
          store_shared(o + 2, a.z, a.w);
          store_shared(o + 4, b.x, b.y);
          store_shared(o + 6, b.z, b.w);
          continue;
        }
        const float sum[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
        uint4 ov = make_uint4(0, 0, 0, 0);
        if ((kmask >> r) & 1) {
          float res[8];
          if (SUB) {
            float pl[8];
            subcube_pooled_term(pass == 0 ? dkc : dvc, (bh * Nc + j) * 4, kmask, r, D, ch, pl);
#pragma unroll
            for (int e = 0; e < 8; ++e) res[e] = fmaf(sum[e], mul, pl[e]);
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) res[e] = fmaf(sum[e], mul, pooled[e]);
          }
          ov = pack8(res);
        }
        if (KIND < 2) store16<ONCE>(dst + (rows0 + j * kTile + r) * CPR + ch, ov);
        else if ((kmask >> r) & 1) dst[rows_r.at(r) + ch] = ov;
      }
    }
  };
  if (raster.on) finish(std::integral_constant<int, 2>{});
  else if (stream) finish(std::integral_constant<int, 1>{});
  else finish(std::integral_constant<int, 0>{});
  if (slot < 0) return;

  // A run of a split list.  The last of them to arrive (the count starts at zero, written with the list's descriptor: cube,
  // first slot, runs, arrived) adds the partial results in slot order -- whichever run that is, the sum is the same
  // -- and finishes them like a whole list: scale, pooled-gradient term, zero pad rows, one rounding to bf16.
  // The parts go past the L2s of the XCDs both ways (store_shared, load_shared), so that nothing has to be written back or
  // invalidated: a part is there for the others once its stores are done.
  wait_vmcnt<0>();
  __syncthreads();
  int4* const sp = (int4*)split + bh * (cap / 2 + 1) + 1 + run_list(desc.w);
  if (tid == 0) *last_run = atomicAdd(&sp->w, 1) == sp->z - 1;
  __syncthreads();
  if (!*last_run) return;
  const int slot0 = sp->y, runs = sp->z;
  float sums[2][LPT][8];
#pragma unroll
  for (int pass = 0; pass < 2; ++pass)
#pragma unroll
    for (int it = 0; it < LPT; ++it)
#pragma unroll
      for (int e = 0; e < 8; ++e) sums[pass][it][e] = 0.f;
  for (int s = 0; s < runs; ++s) {  // (all loads of a part in flight together: each is a trip past the L2)
    const float* src = parts + (bh * cap + slot0 + s) * (long long)(128 * D) + tid * 8;
    float2 x[2][LPT][4];
#pragma unroll
    for (int pass = 0; pass < 2; ++pass)
#pragma unroll
      for (int it = 0; it < LPT; ++it)
#pragma unroll
        for (int e = 0; e < 4; ++e) x[pass][it][e] = load_shared(src + pass * 64 * D + it * NT * 8 + 2 * e);
#pragma unroll
    for (int pass = 0; pass < 2; ++pass)
#pragma unroll
      for (int it = 0; it < LPT; ++it)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          sums[pass][it][2 * e] += x[pass][it][e].x;
          sums[pass][it][2 * e + 1] += x[pass][it][e].y;
        }
  }
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const float4 p0 = pass == 0 ? pk[0] : pv[0], p1 = pass == 0 ? pk[1] : pv[1];
    const float pooled[8] = {p0.x * inv_cnt, p0.y * inv_cnt, p0.z * inv_cnt, p0.w * inv_cnt,
                             p1.x * inv_cnt, p1.y * inv_cnt, p1.z * inv_cnt, p1.w * inv_cnt};
    const float mul = pass == 0 ? scale : 1.0f;
    uint4* dst = pass == 0 ? dk : dv;
#pragma unroll
    for (int it = 0; it < LPT; ++it) {
      const int item_ = it * NT + tid, r = item_ / CPR, ch = item_ % CPR;
      const float(&sum)[8] = sums[pass][it];
      uint4 ov = make_uint4(0, 0, 0, 0);
      if ((kmask >> r) & 1) {
        float res[8];
        if (SUB) {
          float pl[8];
          subcube_pooled_term(pass == 0 ? dkc : dvc, (bh * Nc + j) * 4, kmask, r, D, ch, pl);
#pragma unroll
          for (int e = 0; e < 8; ++e) res[e] = fmaf(sum[e], mul, pl[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) res[e] = fmaf(sum[e], mul, pooled[e]);
        }
        ov = pack8(res);
      }
      if (!raster.on) dst[(rows0 + j * kTile + r) * CPR + ch] = ov;
      else if ((kmask >> r) & 1) dst[RasterRows(raster, bh, j, CPR).at(r) + ch] = ov;
    }
  }
}

}  // namespace vsa
