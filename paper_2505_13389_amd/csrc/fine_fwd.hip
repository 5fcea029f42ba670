// Fine stage forward (Sec. 2.2 fine stage; Sec. 2.1 attention equation under the block mask)
// fused with the gated combine O = O_c * G_c + O_f * G_f.
//
// "Cube" below means a 64-row query block (a cube of 64*m tokens is m consecutive blocks, and the lists the kernel
// gets name blocks).  A workgroup is two wavefronts (four where the launch is too small to fill the chip), each with a
// list walk, LDS stages and an online softmax of its own: it multiplies UNITS of 32 keys with all 64 query rows
// (unit_stream.h), so that every operand it reads from LDS feeds two matrix instructions, and since nobody else reads
// its rows the loop has no barrier.  A workgroup takes one block, whose units its wavefronts share and whose partial
// results they merge through LDS, or (d = 128) two blocks, one per wavefront: see paired_workgroups.  The two round differently: a
// shared block's P is relative to a reference per wavefront and query, so that two weights of a row are 1 exactly, not one.
// O_f against float64: off by 2.335e-3 of its 2-norm with all blocks shared, 2.340e-3 with all paired (16384 tokens, top-32; its own
// rounding to bf16 is 1.7e-3 of that).
//
// Everything is computed transposed so that softmax statistics are per-lane scalars:
//   S^T[key, q]  = K rows (A operand, row-major LDS reads) x Q^T (B operand, registers)
//   O^T[dv,  q] += V^T (A operand, transposing LDS reads) x P^T (B operand = the S^T accumulator
//                  registers converted to bf16 in place)
// In the 32x32 accumulator layout lane l holds query column l%32 and 16 key (or dv) rows.
//
// d = 128: one wavefront per SIMD (Q 64 registers, S of two units 64, O in 128 accumulation registers), so
// nothing but the wavefront's own order overlaps vector work with matrix work: P(u) is formed while S(u+1) is
// multiplied and begun while PV(u-1) is, in steps pinned by scheduling barriers; K is copied three units ahead, V
// one.  d = 64 takes two wavefronts per SIMD.
//
// What bounds it: instruction issue, at the clock that power leaves.  A unit is 32 matrix instructions and 188 others, 192 where all blocks
// are shared (112 of softmax: fma, exp2, sum, half a conversion per value; 24 LDS reads, 16 copies, 20 to 24 scalar ones): 1330 cycles by the
// costs below where the matrix pipe needs 1024, at a
// clock that falls as the chip fills (1.6 to 1.75 GHz; 2.1 while the last workgroups of a launch run).  What an instruction costs a
// wavefront that is alone on its SIMD, measured behind matrix instructions: 5 cycles in vector arithmetic, 8 if the next one
// needs its result, exp2 9, an LDS read 8, scalar ones and waits 4; five or six plain ones fit behind a matrix instruction,
// and none is made up for by fewer behind the next.  So the softmax is cut into operations that are dealt, like the reads, copies and the
// scalar chain of the next list entry, to the 32 matrix instructions one by one (FwdTicks: 32 to 55 cycles each as emitted, 87 at the check of the references), pinned by a
// scheduling barrier right behind each of them, and what is rare (a moved
// reference, pad keys, a new chunk of the list) lies out of the loop's line.  A wavefront with a block of its own walks in a loop of its own,
// where the half of a unit is known and every second one is in the same tile; the tile is counted on, not worked out; the check for a moved
// reference is one comparison.  Against stages of the softmax in place of operations, a list entry at once and 210 others a unit: 1490 -> 1330
// cycles by the costs, 2.03 -> 1.87 M in a whole launch (39936 tokens, 12 heads, top-78), of which the clock leaves a third of the time: 1217 ->
// 1184 us for the forward, 252 -> 247 at 16384 tokens, top-32 (two generations' start-up and end in it), results the same bits.  16x16x32 matrix
// instructions take less energy and, for the same work, 8 cycles of issue more per large one (fine_bwd_dkv.h): with these operations dealt to them a unit
// would be about 1590 cycles; not measured.
// Around the walk a wavefront
// spends 2 to 3 us until its first K is there, 1.4 on the first products, 3 on the merge and 2 (shared block) to 4 on
// normalising, gating and storing, which nothing overlaps on its SIMD: halved per block where a wavefront has a block of
// its own.  That, one factor per lane instead of per row and item on the way out, and a start that waits for K alone:
// 39936 tokens, 12 heads, d = 128, top-78 of 624 1257 -> 1225 us (i.i.d.); 16384 tokens, top-32 of 256 246 -> 233 us, without
// a fine gate 288 -> 264 for the whole forward; 9 % to 17 % where lists are shorter (rules below).
// Measured against 32 keys x 32 queries per wavefront, four wavefronts in step, two per SIMD (every operand fed one
// matrix instruction; the vector work of one wavefront behind the matrix work of another): 39936 tokens, 12
// heads, d = 128, top-78 of 624: 1.47 -> 1.28 ms (i.i.d. selections), 1.43 -> 1.22 ms (local ones); 16384 tokens,
// top-32 of 256: 263 -> 241 us; B = 2, 16 heads, top-128 of 256: 2.38 -> 2.09 ms; d = 64, B = 2, 8 heads, top-32:
// 193 -> 172 us.
#include <type_traits>

#include "coarse_small.h"
#include "ticks.h"
#include "unit_stream.h"
#include "vsa_kernels.h"

namespace vsa {

// A lane's sum of 16 values of a unit above this moves the reference of its column.  Values far above the reference
// cost nothing unless V is large: then O may overflow before it is normalised.  A block in which it does is done again
// with the second bound, under which O stays below 2^8 times the sum of the values of V it is made of.
// Moving a reference costs about 770 cycles per 32 query columns (O through ordinary registers and back).  2^80: with
// N(0, s^2) logits, s in nats, top-32 of 256 blocks / top-78 of 624, 12 heads, d = 128: s = 12 244 / 1262 us, 30 264 / 1380,
// 60 309 / 1500, 100 331 / 1520 (2^60 and both halves of the queries at once: 245 / 1265, 332 / 1665, 374 / 1735, 394 /
// 1766; the kernel for short lists, whose O is in ordinary registers: 283 / 1516, 263 / 1517, 255 / 1496, 252 / 1495).
// Not higher: where one wavefront's sum is 2^80 times the number of keys, another's share is scaled by 2^-126 and no less.
constexpr float kMaxSum = 1208925819614629174706176.f;  // 2^80
constexpr float kTightSum = 256.f;
constexpr float kNoRef = -1e30f;        // below every reference

// Gangs.  The workgroups that run side by side on an XCD fetch their tiles through one 4 MiB L2, and a tile
// is in it for the second one that wants it only if both are at about the same place of their (ascending) lists.
// They start together, but every workgroup starts when an earlier one ends, and after many generations their places
// are spread over the whole walk.  So in long launches the workgroups that fill an XCD once form a gang, and those
// of every `every`-th gang wait until all of it is there.  A wait is bounded and changes no result.  Where a gang
// cannot be on the chip all at once -- another stream's kernel holds part of it, or the device is not 8 XCDs of 32 CUs
// -- every such gang waits out its bound of about 25 us, at most a tenth of the time its 256 tiles take.  Workgroups are dealt to the 8 XCDs round-robin
// by blockIdx.
constexpr unsigned kGang = 64;  // 32 CUs x the workgroups of two wavefronts a CU holds at d = 128
constexpr int kGangSpins = 40;

__global__ void k_gang_clear(unsigned* __restrict__ arrived, unsigned n) {
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) arrived[i] = 0;
}

__device__ __forceinline__ void gang_start(unsigned* arrived, unsigned every) {
  const unsigned x = blockIdx.x & 7u, i = blockIdx.x >> 3, gang = i / kGang;
  if (gang % every) return;  // (uniform)
  if (threadIdx.x == 0) {
    unsigned* mine = arrived + gang * 8 + x;
    const unsigned of_xcd = (gridDim.x + 7 - x) >> 3, size = min(kGang, of_xcd - gang * kGang);
    __hip_atomic_fetch_add(mine, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int spin = 0; spin < kGangSpins; ++spin) {
      if (__hip_atomic_load(mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= size) break;
      __builtin_amdgcn_s_sleep(4);
    }
  }
  __syncthreads();
}

// What lies behind which matrix instruction of a unit, S of the next unit | PV, and where the softmax of a unit, in operations (p_ops), is done:
// from the second instruction of the PV phase before it to the last but one of the S phase of the next.
template <int D>
struct FwdTicks : TickCycles<D / 2> {  // (two units)
  using Table = TickCycles<D / 2>;
  using typename Table::Work;
  using Table::cycles;
  using Table::T;
  static constexpr int KS = D / 16, PH = 2 * KS, U = T / 2;  // LDS operands of a phase; matrix instructions of a phase, of a unit
  static constexpr int kEvery = D == 128 ? 2 : 1;  // a copy behind every other, or every, one of a phase until all are requested
  // LDS operands are waited for in pairs of steps, and read kAhead steps before the first of them is used, spread over kSpread instructions
  static constexpr int kAhead = D == 128 ? 4 : 2, kSpread = D == 128 ? 4 : 2;
  static constexpr int kTile = 1, kChunk = D == 128 ? 3 : 2, kRows = D == 128 ? 5 : 3, kValid = D == 128 ? 7 : 4;  // the list entry of the unit after the next two, in parts
  static constexpr int kOps = 112;
  Work w[kOps] = {};
  int ahead[T + 1] = {};
  static constexpr int in_pv(int j) { return PH + j; }
  static constexpr int in_s(int j) { return U + j; }
  constexpr FwdTicks() {
    for (int t = 0; t < T; ++t) {
      const int u = t % U, j = u % PH, q = j & 3, to = j / 4 * 2 + kAhead;
      const bool of_v = u < PH ? to >= KS : to < KS;  // operands of V are two reads
      if (j % kEvery == 0 && j < kEvery * KS) cycles[t] += Table::kCopy + (j / kEvery % (KS / 2) == 0 ? 3 * Table::kScalar : 0);
      if (q == 0) cycles[t] += Table::kWait;
      if (j == 2 * (KS - kAhead)) cycles[t] += Table::kWait;
      if (of_v && q < kSpread) cycles[t] += Table::kRead * 4 / kSpread;
      if (!of_v && (q == 0 || q == kSpread / 2)) cycles[t] += Table::kRead;
      if (u < PH) {
        if (j == kTile || j == kChunk) cycles[t] += 4 * Table::kScalar;
        if (j == kRows || j == kValid) cycles[t] += 9;
        if (j == PH - 2) cycles[t] += 38;  // the check of the references
        if (j == PH - 1) cycles[t] += 2 * Table::kScalar;
      }
    }
    // an item's first exponential, the arguments of the next, its second exponential, the sums and the conversion of the item before
    int n = 0;
    w[n++] = {Table::MUL, 0, 0};
    w[n++] = {Table::MUL, 0, 1};
    for (int g = 0; g < 17; ++g) {
      if (g < 16) w[n++] = {Table::EXP, g, 0};
      if (g < 15) w[n++] = {Table::MUL, g + 1, 0};
      if (g < 15) w[n++] = {Table::MUL, g + 1, 1};
      if (g < 16) w[n++] = {Table::EXP, g, 1};
      if (g > 0) w[n++] = {Table::ADD, g - 1, 0};
      if (g > 0) w[n++] = {Table::CVT, g - 1, 0};
      if (g > 0) w[n++] = {Table::ADD, g - 1, 1};
    }
    this->deal(ahead, w, kOps, in_pv(1), in_s(PH - 1));
  }
  // A unit's operations begin behind the second matrix instruction that follows its S, and all of them lie ahead of the check of the references,
  // behind the last but one of the next unit's S.
  constexpr bool in_order() const { return ahead[in_pv(1)] == 0 && ahead[in_s(PH - 1)] == kOps && this->ordered(w, kOps); }
};
static_assert(FwdTicks<128>().in_order() && FwdTicks<64>().in_order(), "operations of the softmax");

// PAIRS: the first `pairs` workgroups take two blocks, one per wavefront (d = 128, NW = 2; at d = 64 two wavefronts per SIMD hide one
// another's start-up).  Launches without pairs have instances of their own, which know each wavefront's key half: 288 blocks,
// top-26 32.7 -> 32.1 us, top-50 49.2 -> 48.1.
// COARSE: short sequences, whose coarse stage a workgroup does for its block on the way (NW = 4, see coarse_small.h).
// RASTER: RasterMap or NoRaster (as a runtime choice it cost the smallest launches 0.8 us of 13).
template <int D, int NW, template <class> class UNITS, bool PAIRS, bool COARSE, class RASTER>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 2) void k_fine_fwd(
    int Nc_, int K_, float sl2, const uint4* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
    const uint4* __restrict__ gc, const uint4* __restrict__ gf, const int32_t* __restrict__ idx,
    const float* __restrict__ oc, const uint64_t* __restrict__ mask, uint4* __restrict__ out,
    uint4* __restrict__ out_fine, float* __restrict__ lse_f, int H, long long out_head_stride, long long out_row_stride,
    int m_blocks, unsigned blocks, unsigned pairs, int stream, unsigned* __restrict__ gang_arrived, unsigned gang_every, SmallForwardArgs small, RASTER raster) {
  constexpr bool kRaster = std::is_same_v<RASTER, RasterMap>;
  using TL = Tile<D>;
  using UL = UNITS<TL>;
  using UC = UnitCopy<TL, UL>;
  constexpr int CPR = TL::CPR, KS = D / 16, DVB = D / 32;
  constexpr int HALF = TL::BYTES / 2;   // 32 rows
  constexpr int NC = UC::NC;            // copy instructions per 32 rows
  constexpr int NPV = 2 * DVB;          // steps of the PV phase
  using TK = FwdTicks<D>;
  constexpr TK ticks;
  constexpr int kAhead = TK::kAhead, kEvery = TK::kEvery;
  constexpr int OS = D;
  // per wavefront: K of two units, V of two units
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * 4 * HALF];
  __shared__ float ml[NW * 64 * 2];
  __shared__ SmallCoarse<COARSE ? D : 4> lc;
  __shared__ int32_t lc_list[COARSE ? kSmallCubes : 1];
  static_assert(HALF % 256 == 0, "the operand addresses XOR the bits below 256");
  // copies of a phase that precede its wait for earlier ones
  constexpr int kPart = 2 * (KS - kAhead) / kEvery < NC ? 2 * (KS - kAhead) / kEvery : NC;
  static_assert(KS == NPV && KS == NC && KS > kAhead && KS == TK::KS, "phase interleave");

  // With K = Nc every workgroup of a head walks the same list: then all XCDs work on the same head
  // (plain blockIdx order), which keeps that list's tiles shared chip-wide, and the workgroups that
  // run side by side on an XCD (cubes c, c+8, ...) start their walk a few entries apart and wrap
  // around -- otherwise they ask for the same cache lines in the same cycles.
  if (D == 128 && NW == 2 && gang_arrived) gang_start(gang_arrived, gang_every);
  __shared__ int again;  // O of a valid row overflowed under kMaxSum
  if (threadIdx.x == 0) again = 0;  // (read behind several barriers)
  for (bool tight = false;; tight = true) {
  const float limit = tight ? kTightSum : kMaxSum;
  // (nothing is kept in registers from one round to the next)
  unsigned block = blockIdx.x;
  int tid = threadIdx.x, Nc = Nc_, K = K_;
  asm volatile("" : "+s"(block), "+v"(tid), "+s"(Nc), "+s"(K));
  const int tiles = (K + UL::kEntriesPerTile - 1) / UL::kEntriesPerTile;
  const bool same_lists = K == Nc * UL::kEntriesPerTile;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  // the first `pairs` workgroups take two blocks, one per wavefront; the others one, whose units they share
  const bool paired = PAIRS && block < pairs;
  const unsigned from = paired ? 0u : pairs, those = paired ? pairs : gridDim.x - pairs;
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
  const long long rows0 = bh * (long long)Nc * kTile;  // first row of this (b,h)
  const unsigned char* kb = (const unsigned char*)uniform_ptr(k + rows0 * CPR);
  const unsigned char* vb = (const unsigned char*)uniform_ptr(v + rows0 * CPR);

  // Start-up: the list and Q (one round trip), then the key masks and the copies of the first units, of which the
  // first products need K of the first alone.  Q waits in second stages: a wavefront of its own block has both halves
  // of it, of V and then of K; where a block is shared the first two wavefronts have one each, of V.
  // O: accumulation registers where the kernel has them (one wavefront per SIMD)
  auto mfma_o = [](f32x16& acc, bf16x8 a, bf16x8 b) {
    if (D == 128) mfma_a(acc, a, b);
    else mfma_v(acc, a, b);
  };
  auto pin_o = [](f32x16& acc) {
    if (D == 128) asm volatile("" : "+a"(acc));
    else asm volatile("" : "+v"(acc));
  };
  f32x16 o[DVB][2];
  UC copy;
  copy.init(lane);
  const unsigned lds0 = __builtin_amdgcn_readfirstlane(lds_address(smem)) + (unsigned)wave * (4 * HALF);
  UL list;
  if (!PAIRS) list.only = wave & 1;
  Unit un[3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // the units after the current one
  Unit u0 = {0, 0, 0};
  if constexpr (!COARSE) list.request(idx + (bh * Nc + c) * (long long)K, mask, K, lane, Nc, nu > 0 ? tile_of(0) : 0);
  {
    UnitCopy<TL, CubeUnits<TL>> cq;
    cq.init(lane);
    const unsigned char* qb = (const unsigned char*)uniform_ptr(q + (rows0 + (long long)c * kTile) * CPR);
    const Unit q0 = {0, HALF / 2, 0}, q1 = {HALF, HALF + HALF / 2, 0};
    if (paired) {
      cq.all(qb, q0, lds0 + 3 * HALF);
      cq.all(qb, q1, lds0 + HALF);
    } else if (NW == 2 || wave < 2) {
      cq.all(qb, wave & 1 ? q1 : q0, lds0 + 3 * HALF);
    }
  }
  SmallRows<COARSE ? D : 4> vrows;
  if constexpr (COARSE) {
    if (!tight) small_select<D>(lc, lc_list, Nc, K, c, bh * Nc, small, vrows, tid);
    list.take(lc_list, mask, K, lane, Nc);
  } else {
    wait_vmcnt<0>();  // the list and Q have landed (COARSE: Q is waited for below)
  }
  list.arrived();
  const unsigned ml0 = __builtin_amdgcn_readfirstlane(lds_address(ml)) + (unsigned)wave * 512u;
  const bool second = !paired && nu > 1 && list.loaded(tile_of(1));  // unit 1 is requested already
  if (nu > 0) {  // (a wavefront without units has nothing in flight behind this: `ml` is written again, without a wait)
    request_masks(list, ml0);
    list.rows(tile_of(0), half_of(0), u0);
    copy.all(kb, u0, lds0);
    if (second) {
      list.rows(tile_of(1), half_of(1), un[0]);
      copy.all(kb, un[0], lds0 + HALF);
    }
    copy.all(vb, u0, lds0 + 2 * HALF);
  }
  float nil = 0.f;
  asm volatile("" : "+v"(nil));  // (made anew in every round: a vector of zeros kept from the first would be spilled)
#pragma unroll
  for (int x = 0; x < DVB; ++x)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[x][b][i] = nil;
#pragma unroll
  for (int x = 0; x < DVB; ++x)  // (zeroed once, right here, while the first copies are in flight)
#pragma unroll
    for (int b = 0; b < 2; ++b) pin_o(o[x][b]);
  if constexpr (COARSE) {
    wait_vmcnt<0>();  // Q has landed (and with it the copies, which the loads of the next step would wait for anyway)
    if (!tight) small_output<D>(lc, Nc, c, bh * Nc, small, vrows, tid);
    else __syncthreads();
  } else if (!paired) {
    __syncthreads();
  }
  bf16x8 qreg[2][KS];
  {
    const unsigned char* first_half = smem + (paired ? wave * (4 * HALF) : 0) + 3 * HALF;
    const unsigned char* second_half = smem + (paired ? wave * (4 * HALF) + HALF : 7 * HALF);
    const int lane_q = TL::rowmajor_lane(0, lane);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qreg[0][s] = TL::rowmajor_at(first_half, lane_q, s);
      qreg[1][s] = TL::rowmajor_at(second_half, lane_q, s);
    }
  }
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qreg[0][s]), "+v"(qreg[1][s]));
  if (!paired) __syncthreads();  // every wavefront has Q: the second V stages may be filled
  // the masks and K of the first unit have landed; newer: V of the first and, ahead of it, K of the second
  wait_vmcnt<2 * NC>();
  if (!second) wait_vmcnt<NC>();
  __builtin_amdgcn_sched_barrier(0);
  take_masks(list, ml + wave * 128);
  if (nu > 0) list.get(tile_of(0), half_of(0), u0);
  if (nu > 1) {
    list.get(tile_of(1), half_of(1), un[0]);
    if (!second) copy.all(kb, un[0], lds0 + HALF);
  }
  if (nu > 2) list.get(tile_of(2), half_of(2), un[1]);

  const int my = wave * (4 * HALF);
  const int lane_a = TL::rowmajor_lane(0, lane) + my;
  int lane_b0, lane_b1;
  TL::transposed_lane(0, lane, lane_b0, lane_b1);
  lane_b0 += my;
  lane_b1 += my;

  const bf16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  bf16x8 ones_b = zero8;
  ones_b[0] = (h == 0) ? (__bf16)1.f : (__bf16)0.f;
  // Pad keys never take part: one extra matrix step adds a large negative bias to their rows of S^T (A = bias
  // of key l%32 in contraction slot 0, B = ones in slot 0).
  auto add_bias = [&](f32x16 (&S)[2], uint32_t valid) {
    bf16x8 ab = zero8;
    ab[0] = (h == 0 && !((valid >> l32) & 1)) ? (__bf16)kMaskBias : (__bf16)0.f;
    S[0] = mfma32(ab, ones_b, S[0]);
    S[1] = mfma32(ab, ones_b, S[1]);
  };

  // references of the lane's two query columns; zero, and `have` false, until the first unit with a valid key
  float ref[2] = {0.f, 0.f};
  bool have = false;
  float bar = -1.f;
  float lsum[2] = {0.f, 0.f};
  float ta[2] = {0.f, 0.f}, tb[2] = {0.f, 0.f};  // the unit's sums of a column, even and odd values
  uint4 pb[2][2];  // P^T of the current unit as operands: [query half][contraction step]
  auto put = [](uint4& u4, int w, uint32_t x) {
    if (w == 0) u4.x = x;
    if (w == 1) u4.y = x;
    if (w == 2) u4.z = x;
    if (w == 3) u4.w = x;
  };
  // Softmax item `it` of 16: two values of one query half; the first eight make up contraction step 0.  Its arithmetic is done in operations, dealt
  // to the matrix instructions one by one (FwdTicks), none of which needs the result of the one before it (that costs 8 cycles instead of 5).
  float xf[2][2] = {}, xe[2][2] = {};  // arguments and exponentials of an item, by its parity
  auto p_fma = [&](const f32x16 (&S)[2], int it, int i, const float* rf) {
    const int b = (it >> 2) & 1, e = 8 * (it >> 3) + 2 * (it & 3);
    xf[it & 1][i] = fmaf(S[b][e + i], sl2, -rf[b]);
    asm volatile("" : : "v"(xf[it & 1][i]));  // (pure arithmetic has no place of its own in the order: tie it to this step)
  };
  auto p_exp = [&](int it, int i) {
    xe[it & 1][i] = fast_exp2(xf[it & 1][i]);
    asm volatile("" : : "v"(xe[it & 1][i]));
  };
  auto p_sum = [&](int it, int i) {
    float& t = (i ? tb : ta)[(it >> 2) & 1];
    const float x = xe[it & 1][i];
    t = (it & 11) == 0 ? x : t + x;
    asm volatile("" : : "v"(t));
  };
  auto p_convert = [&](int it) {
    const uint32_t pp = pack_bf16(xe[it & 1][0], xe[it & 1][1]);
    put(pb[(it >> 2) & 1][it >> 3], it & 3, pp);
    asm volatile("" : : "v"(pp));
  };
  auto p_ops = [&](const f32x16 (&S)[2], auto from, auto to, const float* rf) {
    in_steps<decltype(to)::value - decltype(from)::value>([&](auto number) {
      constexpr typename TK::Work w = ticks.w[decltype(from)::value + decltype(number)::value];
      if constexpr (w.op == TK::MUL) p_fma(S, w.item, w.i, rf);
      if constexpr (w.op == TK::EXP) p_exp(w.item, w.i);
      if constexpr (w.op == TK::ADD) p_sum(w.item, w.i);
      if constexpr (w.op == TK::CVT) p_convert(w.item);
    });
  };
  // the larger of `old` and the largest (scaled) logit of the unit in the lane's query column
  // (pad keys do not count: a column all of whose logits are -inf keeps kNoRef and ends as one without a valid key)
  auto unit_max = [&](const f32x16& S, uint32_t keys, float old) {
    float mx = fmaxf(fmaxf(S[0], S[1]), S[2]);
#pragma unroll
    for (int i = 3; i < 15; i += 2) mx = fmaxf(fmaxf(mx, S[i]), S[i + 1]);
    mx = max_across_halves(fmaxf(mx, S[15]));
    if (keys != 0xffffffffu && mx < 0.5f * kMaskBias) mx = -INFINITY;
    return fmaxf(mx * sl2, old);
  };
  uint32_t valid = 0;  // valid keys of the current unit

  f32x16 zero16;
#pragma unroll
  for (int i = 0; i < 16; ++i) zero16[i] = 0.f;
  f32x16 s0[2], s1[2];
  bf16x8 kcur[kAhead];  // K operands of a unit's first steps, read during the phase before
  if (nu > 0) {  // S of the first unit, its reference, and the softmax items that precede its PV phase's own
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bf16x8 a = TL::rowmajor_at(smem, lane_a, s);
      s0[0] = mfma32(a, qreg[0][s], s == 0 ? zero16 : s0[0]);
      s0[1] = mfma32(a, qreg[1][s], s == 0 ? zero16 : s0[1]);
    }
    if (u0.valid != 0xffffffffu) add_bias(s0, u0.valid);
    __builtin_amdgcn_sched_barrier(0);  // (the matrix instructions above have waited for the reads of this stage)
    if (nu > 2) copy.all(kb, un[1], lds0);
    // K(1) has landed; newer: K(2) and, where K(1) was requested early, V(0)
    if (second && nu > 2) wait_vmcnt<2 * NC>();
    else if (nu > 2) wait_vmcnt<NC>();
    else wait_vmcnt<0>();
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < kAhead; ++s) kcur[s] = TL::rowmajor_at(smem + HALF, lane_a, s);
    valid = u0.valid;
    if (valid) {
      ref[0] = unit_max(s0[0], valid, kNoRef);
      ref[1] = unit_max(s0[1], valid, kNoRef);
      have = true;
      bar = limit;
    }
    p_ops(s0, std::integral_constant<int, 0>{}, std::integral_constant<int, ticks.ahead[TK::U]>{}, ref);
  }

  // The unit that is fetched next in the steady walk: its tile and half.  Two blocks per workgroup: both halves of a tile one after the other.
  int next_tile = nu > 3 ? tile_of(2) : 0;
  // One unit u (its S is there, in S): P(u) while S(u+1) is multiplied into T, then PV(u) while P(u+1) begins.
  // KIND 2: the units up to u + 3 exist; 1: u + 1 exists; 0: u is the last one.  `par` = u & 1.
  // OWN: the wavefront has a block of its own (then the half of a unit of the steady walk is known: `par`).
  auto body = [&](auto kind_tag, auto own_tag, int par, f32x16 (&S)[2], f32x16 (&T)[2], int u) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool OWN = decltype(own_tag)::value;
    constexpr bool more1 = KIND >= 1;
    const bool more2 = KIND == 2 || (KIND == 1 && u + 2 < nu), more3 = KIND == 2 || (KIND == 1 && u + 3 < nu);
    const unsigned char* kn = smem + (1 - par) * HALF;  // K(u+1)
    const unsigned char* vc = smem + (2 + par) * HALF;  // V(u)
    bf16x8 ka[KS + kAhead];
    bf16x4 va[NPV + kAhead][2];
    auto v_half = [&](int i, int part) { return TL::transposed_half(vc, part ? lane_b1 : lane_b0, i / DVB, i % DVB); };
    // The operand reads for the two steps kAhead further on, spread over the four matrix instructions (q = 0 .. 3) of two steps, d = 64: over the
    // first two.  A V operand is two reads: read_v issues the share of q of those of steps i and i + 1.  A K operand is one read: reads_row says
    // whether that of the w-th of the two steps is issued at q.
    constexpr int kSpread = TK::kSpread;
    auto read_v = [&](int i, int q) {  // of steps i and i + 1
#pragma unroll
      for (int r = q * 4 / kSpread; r < (q + 1) * 4 / kSpread; ++r)
        if (q < kSpread) va[i + (r >> 1)][r & 1] = v_half(i + (r >> 1), r & 1);
    };
    // reads requested behind those of the pair of steps (s, s + 1), of a phase of n steps: `now` for a pair of this phase, `next` of the next
    constexpr auto reads_between = [](int s, int n, int now, int next) {
      int r = 0;
      for (int t = s + 2; t < s + kAhead; t += 2) r += t < n ? now : next;
      return r;
    };
    auto reads_row = [&](int q, int w) { return q == 2 * w * kSpread / 4; };
    auto v_op = [&](int i) { return __builtin_shufflevector(va[i][0], va[i][1], 0, 1, 2, 3, 4, 5, 6, 7); };
    if (more1) {
#pragma unroll
      for (int s = 0; s < kAhead; ++s) ka[s] = kcur[s];
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- S(u+1) | the rest of P(u), the copy of V(u+1), the first V operands
    in_steps<2 * KS>([&](auto number) {
      constexpr int j = decltype(number)::value, s = j >> 1, q = j & 3;
      if (more1 && q == 0 && j < kEvery * NC) copy.aim(lds0 + (3 - par) * HALF, j / kEvery);
      if (more1 && q == 0) {  // this pair of steps is there; newer: the next one
        wait_lgkmcnt<reads_between(s, KS, 2, 4)>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more1) T[j & 1] = mfma32(ka[s], qreg[j & 1][s], s == 0 ? zero16 : T[j & 1]);
      __builtin_amdgcn_sched_barrier(0);
      if (j == 2 * (KS - kAhead)) {  // V(u) has landed; newer: K(u+2) and a part of V(u+1)
        if (more2) wait_vmcnt<NC + kPart>();
        else if (more1) wait_vmcnt<kPart>();
        else wait_vmcnt<0>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more1 && j % kEvery == 0 && j < kEvery * NC) copy.piece(vb, un[0], lds0 + (3 - par) * HALF, j / kEvery, q == 0);
      constexpr int to = s - s % 2 + kAhead;  // the two steps whose operands are requested now
      if constexpr (to >= KS) {
        read_v(to - KS, q);
      } else if (more1) {
        if (reads_row(q, 0)) ka[to] = TL::rowmajor_at(kn, lane_a, to);
        if (reads_row(q, 1)) ka[to + 1] = TL::rowmajor_at(kn, lane_a, to + 1);
      }
      if (KIND == 2) {
        const int half = OWN ? 1 - par : wave & 1;
        if (j == TK::kTile && !(OWN && half)) {
          next_tile += OWN ? 1 : NW / 2;
          if (next_tile >= tiles) next_tile -= tiles;
        }
        if (j == TK::kChunk && !(OWN && half)) list.load(next_tile);
        if (j == TK::kRows) list.rows(next_tile, half, un[2]);
        if (j == TK::kValid) list.valid(next_tile, half, un[2]);
      } else if (j == 3 && more3) {
        list.get(tile_of(u + 3), half_of(u + 3), un[2]);
      }
      p_ops(S, std::integral_constant<int, ticks.ahead[TK::in_s(j)]>{}, std::integral_constant<int, ticks.ahead[TK::in_s(j + 1)]>{}, ref);
      __builtin_amdgcn_sched_barrier(0);
      if (j == 2 * KS - 2) {
        // The reference of a column stays as long as neither lane's sum of 16 values exceeds `limit`: then no value does, and
        // the rescaling of O is skipped for almost every unit.  The result is exact either way, and a lane's arithmetic
        // never depends on what other query columns (pad rows included) hold.
        // (A unit without a valid key leaves every value at zero; the first one that has some sets the reference.)
        // (`bar`: `limit`, or as long as there is no reference less than any sum)
        float tsum[2] = {ta[0] + tb[0], ta[1] + tb[1]};
        if (__builtin_expect(__any(!(fmaxf(tsum[0], tsum[1]) <= bar)), 0) && (have || valid)) {
          // (the last products that wrote O lie almost a whole S phase back, so it can be read at once)
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const bool moves = !have || max_across_halves(tsum[b]) > limit;
            if (!__any(moves)) continue;
            const float old = have ? ref[b] : kNoRef, mnew = moves ? unit_max(S[b], valid, old) : old;
            const float alpha = fast_exp2(old - mnew);  // (nothing accumulated yet: 0 times 0; unchanged: 1)
            lsum[b] *= alpha;
#pragma unroll
            for (int x = 0; x < DVB; ++x) {
              pin_o(o[x][b]);  // (moved to ordinary registers from here on and not before the branch)
#pragma unroll
              for (int i = 0; i < 16; ++i) o[x][b][i] *= alpha;
              pin_o(o[x][b]);
              __builtin_amdgcn_sched_barrier(0);  // (one block of O in ordinary registers at a time)
            }
            ref[b] = mnew;
            // (no reference yet: -inf in every key, and nothing of the pad keys either)
            const float use[2] = {ref[0] > kNoRef ? ref[0] : -kNoRef, ref[1] > kNoRef ? ref[1] : -kNoRef};
#pragma unroll
            for (int st = 0; st < 2; ++st)
#pragma unroll
              for (int w = 0; w < 4; ++w) {
                const int it = 8 * st + 4 * b + w;
                for (int i = 0; i < 2; ++i) {
                  p_fma(S, it, i, use);
                  p_exp(it, i);
                  p_sum(it, i);
                }
                p_convert(it);
              }
            tsum[b] = ta[b] + tb[b];
          }
          have = true;
          bar = limit;
        }
        lsum[0] += tsum[0];
        lsum[1] += tsum[1];
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    if (more1) {
      if (__builtin_expect(un[0].valid != 0xffffffffu, 0)) add_bias(T, un[0].valid);
    }
    // ---- PV(u) | the first of P(u+1), the copy of K(u+3), the first K operands of u+2
    const uint4 pc[2][2] = {{pb[0][0], pb[0][1]}, {pb[1][0], pb[1][1]}};
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");  // (two wait states between the moves to pc and the first matrix instruction)
    in_steps<2 * NPV>([&](auto number) {
      constexpr int j = decltype(number)::value, i = j >> 1, q = j & 3;
      if (KIND == 2 && q == 0 && j < kEvery * NC) copy.aim(lds0 + (1 - par) * HALF, j / kEvery);
      if (q == 0) {
        wait_lgkmcnt<reads_between(i, NPV, 4, 2)>();
        __builtin_amdgcn_sched_barrier(0);
      }
      mfma_o(o[i % DVB][j & 1], v_op(i), __builtin_bit_cast(bf16x8, pc[j & 1][i / DVB]));
      __builtin_amdgcn_sched_barrier(0);
      if (more1 && j == 2 * (NPV - kAhead)) {  // K(u+2) has landed; newer: V(u+1) and a part of K(u+3)
        if (more3) wait_vmcnt<NC + (KIND == 2 ? kPart : NC)>();
        else if (more2) wait_vmcnt<NC>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (KIND == 1 && j == 0 && more3) copy.all(kb, un[2], lds0 + (1 - par) * HALF);  // (one branch, not one per copy)
      if (KIND == 2 && j % kEvery == 0 && j < kEvery * NC) copy.piece(kb, un[2], lds0 + (1 - par) * HALF, j / kEvery, q == 0);
      constexpr int to = i - i % 2 + kAhead;
      if constexpr (to < NPV) {
        read_v(to, q);
      } else if (more1) {  // (unused if u + 2 does not exist)
        if (reads_row(q, 0)) kcur[to - NPV] = TL::rowmajor_at(smem + par * HALF, lane_a, to - NPV);
        if (reads_row(q, 1)) kcur[to - NPV + 1] = TL::rowmajor_at(smem + par * HALF, lane_a, to - NPV + 1);
      }
      if (more1) p_ops(T, std::integral_constant<int, ticks.ahead[TK::in_pv(j)]>{}, std::integral_constant<int, ticks.ahead[TK::in_pv(j + 1)]>{}, ref);
      __builtin_amdgcn_sched_barrier(0);
    });
    valid = un[0].valid;
    un[0] = un[1];
    un[1] = un[2];
  };
  if (nu > 0) {
    const std::integral_constant<int, 2> steady;
    const std::integral_constant<int, 1> inner;
    const std::integral_constant<int, 0> last;
    const std::true_type own;
    const std::false_type shared;
    int u = 0;
    if constexpr (PAIRS) {
      if (paired)
        for (; u + 4 < nu; u += 2) {
          body(steady, own, 0, s0, s1, u);
          body(steady, own, 1, s1, s0, u + 1);
        }
    }
    if (!paired)
      for (; u + 4 < nu; u += 2) {
        body(steady, shared, 0, s0, s1, u);
        body(steady, shared, 1, s1, s0, u + 1);
      }
    for (; u + 1 < nu; ++u) {
      body(inner, shared, u & 1, s0, s1, u);
      s0[0] = s1[0];
      s0[1] = s1[1];
    }
    body(last, shared, u & 1, s0, s1, u);
  }
  mfma_fence();  // the last matrix results land before they are read
#pragma unroll
  for (int x = 0; x < DVB; ++x)
#pragma unroll
    for (int b = 0; b < 2; ++b) pin_o(o[x][b]);
  __builtin_amdgcn_sched_barrier(0);

  // `out` may be head-major [B,H,Np,D] or token-major [B,Np,H,D] (same batch stride): chunk ch of
  // tiled row n of head h of batch b sits at b*H*Np*CPR + h*out_head_stride + n*out_row_stride + ch
  const long long out0 = (bh / H) * ((long long)H * Nc * kTile * CPR) + (bh % H) * out_head_stride;
  // ---- merge the partial results of the block's wavefronts (P of them), normalise, gate, store
  const uint64_t qmask = mask[c];
  // KIND 0, 1: `out` tiled, 1 past the caches; 2: raster, through them (past them is left to do: op at 48 to 96 MiB 0.4 to 2 % faster)
  auto finish = [&](auto parts_tag, auto kind_tag) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool ONCE = KIND == 1;
    constexpr int P = decltype(parts_tag)::value, NT = 64 * P, LPT = kTile * CPR / NT, AT_ONCE = LPT < 8 ? LPT : 8;
    static_assert(NT % CPR == 0, "a thread keeps its column chunk");
    const int t = P == 1 ? lane : tid, ch = t % CPR;
    float* const bufs = (float*)smem + (P == 1 ? wave * 64 * OS : 0);
    // The gates and the coarse output of this thread's first items are requested first: they arrive while
    // the partial results go through LDS.  Pad rows are loaded too (they exist in memory) and ignored.
    const long long g0 = (rows0 + c * kTile + t / CPR) * CPR + ch;
    uint4 gc_raw[AT_ONCE], gf_raw[AT_ONCE];
    auto request = [&](int it) {
      gc_raw[it % AT_ONCE] = load16<ONCE>(gc + g0 + it * NT);
      gf_raw[it % AT_ONCE] = gf ? load16<ONCE>(gf + g0 + it * NT) : make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);  // bf16 ones
    };
#pragma unroll
    for (int it = 0; it < AT_ONCE; ++it) request(it);
    const float* ocr = oc + ((bh * Nc + c) / m_blocks) * D + ch * 8;  // O_c is per cube = m_blocks blocks
    if constexpr (COARSE) ocr = lc.sum[0] + ch * 8;
    const float4 c0 = *(const float4*)ocr, c1 = *(const float4*)(ocr + 4);

    // M, L: reference and sum of a column.  (M = -inf: the list named no valid key at all -- only a caller-supplied
    // list can, e.g. one made of dead key cubes -- or every logit of the column was -inf; the row then gets O_f = 0
    // and lse = 0 instead of NaN)
    auto logsum = [&](float M, float L) { return M == -INFINITY ? 0.f : (M + fast_log2(L)) * kLn2; };
    auto merge = [&](int r, float& M, float& L, float& biggest) {
      float m[P], l[P];
#pragma unroll
      for (int w = 0; w < P; ++w) {
        m[w] = ml[(w * 64 + r) * 2];
        l[w] = ml[(w * 64 + r) * 2 + 1];
        biggest = fmaxf(biggest, l[w]);
      }
      M = m[0];
#pragma unroll
      for (int w = 1; w < P; ++w) M = fmaxf(M, m[w]);
      L = 0.f;
#pragma unroll
      for (int w = 0; w < P; ++w) L += M == -INFINITY ? 0.f : l[w] * fast_exp2(m[w] - M);
    };
    // Up to two wavefronts normalise O on the way to LDS, one factor per lane and query half; four, whose threads have
    // few rows each, save the barrier before it and weigh the parts row by row.
    constexpr bool kByRow = P > 2;
    float M[2], L[2], f[2] = {1.f, 1.f}, most = 0.f;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      M[b] = have && ref[b] > kNoRef ? ref[b] : -INFINITY;
      L[b] = lsum[b] + __shfl_xor(lsum[b], 32);
      most = fmaxf(most, L[b]);
      if (P > 1 && h == 0) *(float2*)&ml[(wave * 64 + b * 32 + l32) * 2] = make_float2(M[b], L[b]);
    }
    if (P > 1) __syncthreads();  // (every wavefront is done with its stages, too)
    if (!kByRow) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const int r = b * 32 + l32;
        const float mine = M[b];
        if (P > 1) merge(r, M[b], L[b], most);
        f[b] = M[b] == -INFINITY ? 0.f : (P > 1 ? fast_exp2(mine - M[b]) : 1.0f) / L[b];
        if (lse_f && h == 0 && (P == 1 || wave == 0)) lse_f[rows0 + c * kTile + r] = (qmask >> r) & 1 ? logsum(M[b], L[b]) : 0.f;
      }
    }
    {
      float* Op = bufs + (P == 1 ? 0 : wave) * 64 * OS;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int x = 0; x < DVB; ++x)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4)
            *(float4*)&Op[merge_offset(b * 32 + l32, x * 32 + 8 * g4 + 4 * h, OS)] =
                make_float4(o[x][b][4 * g4] * f[b], o[x][b][4 * g4 + 1] * f[b], o[x][b][4 * g4 + 2] * f[b], o[x][b][4 * g4 + 3] * f[b]);
    }
    if (P > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();  // (a wavefront's LDS accesses stay in order)

    const bool check = kByRow || __any(most > kTightSum);  // (only then can O have overflowed before it was normalised)
    bool overflow = false;
    uint4* const orow = out + out0 + (long long)(c * kTile + t / CPR) * out_row_stride + ch;
    auto raster_row = [&](int r) {
      if constexpr (kRaster) return RasterRows(raster, bh, c, CPR).at(r);
      else return 0ll;
    };
    const float ocv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
    for (int it = 0; it < LPT; ++it) {
      const int r = (it * NT + t) / CPR;
      const int m0 = merge_offset(r, ch * 8, OS), m1 = merge_offset(r, ch * 8 + 4, OS);
      float of[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, Mr = 0.f, Lr = 1.f, seen = 0.f;
      if (kByRow) merge(r, Mr, Lr, seen);
      const float inv = Mr == -INFINITY ? 0.f : 1.0f / Lr;
#pragma unroll
      for (int w = 0; w < P; ++w) {
        const float4 x = *(const float4*)(bufs + w * 64 * OS + m0), y = *(const float4*)(bufs + w * 64 * OS + m1);
        const float part_of[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
        const float fw = !kByRow ? 1.f : (Mr == -INFINITY ? 0.f : fast_exp2(ml[(w * 64 + r) * 2] - Mr) * inv);
#pragma unroll
        for (int e = 0; e < 8; ++e) of[e] = kByRow ? fmaf(part_of[e], fw, of[e]) : w == 0 ? part_of[e] : of[e] + part_of[e];
      }
      float gcv[8], gfv[8], res[8];
      unpack8(gc_raw[it % AT_ONCE], gcv);
      unpack8(gf_raw[it % AT_ONCE], gfv);
      if (it + AT_ONCE < LPT) request(it + AT_ONCE);
#pragma unroll
      for (int e = 0; e < 8; ++e) res[e] = fmaf(ocv[e], gcv[e], of[e] * gfv[e]);
      const bool live = (qmask >> r) & 1;
      uint4 ov = pack8(res), fv = pack8(of);
      if (!live) ov = fv = make_uint4(0, 0, 0, 0);
      if (check) {
        float nought = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) nought = fmaf(of[e], 0.f, nought);  // NaN unless all of them are finite
        overflow |= live && nought != 0.f && (!kByRow || seen > kTightSum);
      }
      if (KIND < 2) store16<ONCE>(orow + (long long)(it * (NT / CPR)) * out_row_stride, ov);
      else if (live) out[raster_row(r) + ch] = ov;
      if (out_fine) out_fine[g0 + it * NT] = fv;
      if (kByRow && lse_f && ch == 0) lse_f[rows0 + c * kTile + r] = live ? logsum(Mr, Lr) : 0.f;
      if (LPT > AT_ONCE) __builtin_amdgcn_sched_barrier(0);  // (item by item: the loads of later ones stay ahead of the stores)
    }
    return overflow;
  };
  if constexpr (PAIRS) {
    if (paired) {
      const std::integral_constant<int, 1> one;
      bool overflow;
      if constexpr (kRaster) overflow = finish(one, std::integral_constant<int, 2>{});
      else overflow = stream ? finish(one, one) : finish(one, std::integral_constant<int, 0>{});
      if (tight || !__any(overflow)) return;
      continue;
    }
  }
  const std::integral_constant<int, NW> all;
  bool overflow;
  if constexpr (kRaster) overflow = finish(all, std::integral_constant<int, 2>{});
  else if constexpr (NW == 2) overflow = stream ? finish(all, std::integral_constant<int, 1>{}) : finish(all, std::integral_constant<int, 0>{});
  else overflow = finish(all, std::integral_constant<int, 0>{});  // (such launches never stream)
  if (tight) return;
  if (overflow) again = 1;
  __syncthreads();
  if (!again) return;
  }
}

// Which kernel, by the number of query blocks and of 64-key tiles in a list.  The one for short lists hides its workgroups' start-up and wind-down
// behind one another and takes longer per tile.  Figures: time of a whole forward with the general kernel over that with the other, both in turn in one
// process, back to back, N(0,1) inputs, mean of two machines (which differ by 0.01 to 0.03 where a last generation is nearly empty).
//   d = 128  1024 blocks are a generation of the general kernel (two per workgroup), 512 of the other.  Where blocks are shared: 360, 3 tiles 1.005, 4
//            0.995, 5 0.985; 384, 3 1.005, 4 1.00, 5 0.985; 448, 3 1.02, 4 1.005, 6 1.02; 468, 6 1.005, 8 1.005; 480, 8 1.005, 10 1.02; 504, 8 1.015, 10 1.02, 12
//            1.02; 512, 8 1.01, 10 1.02, 12 1.025.  Where the last generation of pairs is nearly empty: 1026, 8 0.995, 12 0.985, 20 0.97; 1056, 8
//            0.98, 16 0.97, 24 0.955; 1100, 6 0.975, 12 0.96; 1152 in heads of 96, 4 0.99, 8 0.98, 16 0.97, of 288, 4 0.99, 8 0.98; 1200, 4 1.00, 8 0.98;
//            1280, 4 0.995, 8 0.99, 10 0.97; 2112, 4 1.03, 8 0.965, 12 0.955; 2200, 4 1.02, 6 1.005, 8 0.975; 2205, 4 1.00, 8 0.98; 2304 in heads of 96, 4
//            1.015, 6 1.01, 8 0.98, of 288, 6 1.01, 8 0.995, 12 0.965; 2400, 3 1.04, 5 1.00, in heads of 400, 5 1.01, 6 0.97; 2560 of 256, 3 1.00, 5 0.995, of
//            512, 3 1.04, 5 0.995, 6 1.00; 2600, 3 1.055, 4 1.00, 5 1.00; 2688, 3 1.025, 4 1.015; 2800, 3 1.04, 4 1.025; 2880, 3 1.035, 4 0.99; 3000, 3 1.03, 4
//            0.995; 3072, 2 1.015, 3 1.01; 3200, 3 1.045, 4 1.00, 6 0.99; 4200, 3 1.005, 4 0.955; 4500, 2 0.97, 3 0.965.
//            The lines of 1025 to 1280, 2049 to 2304 and 4097 to 4608 blocks lie where the two kernels met when the general one took 1490 cycles a unit
//            (now 1330): from 6 to 8 tiles on, and at 4500 blocks, it wins by 1 to 5 % there.
//   d = 64   a generation of the general kernel is 1024 blocks: 384, 1 1.035, 2 1.00, 3 1.02, 4 1.01; 560, 8 0.995, 16 0.98, 20 0.95; 720, 8 1.02, 12 1.005, 16
//            0.97; 1056, 8 1.03, 12 1.00, 14 1.00, 16 0.98; 1536, 12 1.05, 14 1.05, 16 0.97; 1920, 2 1.01, 4 1.00, 6 1.00, 8 0.99; 2240, 8 1.03, 10 1.00, 12
//            0.97; 2660, 8 1.01, 9 1.005, 10 0.985; 3500, 4 1.00, 6 0.995, 8 0.99; 4500, 1 1.025, 2 1.005, 3 1.00, 4 0.99; 6144, 4 0.91.
//   Large heads (d = 128), whose K and V outgrow an L2 several times: a second wavefront per SIMD also hides the trips beyond it, so
//            the lines lie further out. 22 to 64 MiB: 2200 blocks in 2 heads, 6 tiles 1.005, 8 0.995, 12 0.985, 16 0.955; 2304 in 2, 8 0.98, 12 0.98, 16 0.955; 2400 in
//            3, 5 1.00, 6 0.995, 8 1.005; 2560 in 2, 4 1.02, 6 1.00, 8 0.985; 2640 in 3, 3 1.005, 5 0.995; 2880 in 3, 3 1.005, 4 0.995, 5 0.985; 3200 in 4, 3 1.02, 5
//            1.01, 7 1.00, 8 0.99; 4320 in 4, 3 1.04, 4 1.035, 6 1.02. From 64 MiB, where the general kernel's workgroups also wait for one another (gangs):
//            2304, 8 1.04, 16 1.02, 20 1.015, 24 1.01; 2560, 8 1.03, 16 1.02, 20 1.005; 3072, 4 1.045, 8 1.02, 12 1.005, 16 1.00; 4096, 4 1.045, 8 1.01, 16 1.005;
//            4224 in 2, 4 1.08, 8 1.04, 10 1.025.
constexpr size_t kLargeHead = (size_t)22 << 20, kVastHead = (size_t)64 << 20;
inline size_t kv_bytes(int Nc, int d) { return (size_t)Nc * kTile * d * 4; }
inline bool fwd_short(int d, int Nc, unsigned grid, int tiles) {
  if (d == 64) {
    if (grid <= 512) return tiles <= 2;
    if (grid <= 768) return tiles <= 16;
    if (grid <= 1024) return false;
    if (grid <= 1792) return tiles <= 14;
    if (grid < 2048) return tiles <= 4;
    if (grid <= 2560) return tiles <= 12;
    return tiles <= (grid < 2816 ? 9 : grid <= 4096 ? 6 : grid <= 5120 ? 2 : 0);
  }
  if (grid <= 512) return tiles <= (grid > 448 ? 10 : 4);
  if (grid <= 1024) return false;
  if (grid <= 1280) return tiles <= (grid <= 1152 ? 20 : 10);
  if (grid <= 2048) return false;
  const size_t head = kv_bytes(Nc, d);
  if (head >= kVastHead) return tiles <= (grid <= 2304 ? 20 : grid <= 4096 ? 16 : grid <= 4608 ? 8 : 0);
  const bool large = head >= kLargeHead;
  if (grid <= 3072) return tiles <= (grid <= 2304 ? 12 : grid <= 2560 ? (large ? 8 : 5) : grid < 2816 ? 4 + large : grid < 3072 ? 3 + large : 0);
  return tiles <= (grid <= 3264 ? 6 + large : grid > 4096 && grid <= 4608 ? 3 + large : 0);
}
// The general kernel with four wavefronts per workgroup: half as long a walk counts where the launch does not fill the chip
// with two-wavefront workgroups.  d = 64, 64 blocks, 8 tiles 10.0 against 12.0; 512 blocks, 33 tiles 27.6 / 37.2; 640 blocks
// 0.93 of it, 1536 0.87; 1024 blocks 1.05, 2560 0.95 to 1.01.  d = 128, 256 blocks, 33 tiles 26.2 / 34.8, 384 blocks 44.0 / 37.2.
inline bool fwd_four_waves(int d, unsigned grid, int tiles) {
  if (d == 128) return grid <= 256;
  return grid <= 512 || (tiles > 14 && grid <= 2560 && !(grid > 768 && grid <= 1024));
}
// (and such launches do not bypass the caches: an epilogue that may costs them 0.1 to 0.2 us; 96 blocks, d = 64, 4 tiles 9.1 -> 8.9 us,
// 288 11.2 -> 10.9)
static_assert(2560ll * kTile * 64 * 2 < kStreamBytes && 256ll * kTile * 128 * 2 < kStreamBytes, "four wavefronts: no large tensors");

bool fine_fwd_with_coarse(int BH, int Nc, int d, int m_blocks) {
  return m_blocks == 1 && Nc <= kSmallCubes && BH * Nc <= (d == 128 ? 256 : 512);
}

static int fwd_tiles(int K, int key_cubes_16) { return key_cubes_16 ? (K + 3) / 4 : K; }
FineRoute fine_fwd_route(int BH, int Nc, int d, int K, int key_cubes_16, bool coarse) {
  const unsigned grid = (unsigned)(BH * Nc);
  const int tiles = fwd_tiles(K, key_cubes_16);
  if (coarse) return {4, 0};
  if (fwd_short(d, Nc, grid, tiles)) return {0, 0};
  if (fwd_four_waves(d, grid, tiles)) return {4, 0};
  return {2, d == 128 ? paired_workgroups(grid, 512) : 0};
}

hipError_t launch_fine_fwd(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                           const void* gate_c, const void* gate_f, const int32_t* idx, const float* oc,
                           const uint64_t* mask, void* out, void* out_fine, float* lse_f, int H, int out_token_major,
                           int m_blocks, int key_cubes_16, unsigned* gang_scratch, const SmallForwardArgs* coarse, const RasterMap& raster, hipStream_t s) {
  const float sl2 = scale * kLog2e;
  const unsigned grid = (unsigned)(BH * Nc);
  const int tiles = fwd_tiles(K, key_cubes_16);
  const int stream = (long long)grid * kTile * d * 2 >= kStreamBytes;
  const FineRoute route = fine_fwd_route(BH, Nc, d, K, key_cubes_16, coarse != nullptr);
  if (route.waves == 0)
    return launch_fine_fwd_short(BH, Nc, d, K, scale, q, k, v, gate_c, gate_f, idx, oc, mask, out, out_fine, lse_f, H,
                                 out_token_major, m_blocks, key_cubes_16, raster, s);
  const unsigned pairs = route.pairs;
  // Gangs, one in about every 256 tiles walked, at d = 128 where the K and V of a head are many times an L2, the lists differ
  // and there are 16 generations (heads of 64 MiB: two).  Without / with, lists of N(0,1) inputs, then local ones: 1440
  // blocks (45 MiB), 40 heads, lists of 96 14.3 / 13.1, 13.4 / 13.0 ms, of 180 32.9 / 23.3 (L2 hits 0.38 without); 16 heads,
  // 180 9.66 / 9.06, 9.06 / 8.87 ms, 60 3.25 / 3.29, 3.31 / 3.36; 1152 blocks (36 MiB), 12 heads, 32 1.55 / 1.42, 1.10 / 1.13;
  // 2160 blocks (68 MiB), 2 heads, 180 2.72 / 2.62, 1.60 / 1.59, 4 heads 5.10 / 3.43, 3.17 / 3.20.  Elsewhere the waits
  // cost more than the hits return: 1440 blocks, 2 heads, 32 228 / 240 us; 624 blocks (19.5 MiB) 1.23 / 1.26 ms; d = 64,
  // 1440 blocks, 16 heads, 180 4.62 / 4.83, 4.55 / 4.72 ms, 2 heads, 24 105 / 123 us.
  const size_t head = kv_bytes(Nc, d);
  const bool gangs = d == 128 && tiles < Nc && ((head >= kLargeHead && grid >= 8192) || (head >= kVastHead && grid >= 1024));
  const unsigned every = gangs ? (unsigned)(127 / tiles + 1) : 1u;
  unsigned* arrived = gangs ? gang_scratch : nullptr;
  if (gangs) {
    const unsigned n = 8 * ((grid / 8 + kGang) / kGang + 1);  // (at most BH*Nc/32 + 24 counters)
    k_gang_clear<<<(n + 255) / 256, 256, 0, s>>>(arrived, n);
  }
  const long long cpr = d / 8, Np = (long long)Nc * kTile;
  const long long ohs = out_token_major ? cpr : Np * cpr, ors = out_token_major ? H * cpr : cpr;
  const SmallForwardArgs small = coarse ? *coarse : SmallForwardArgs{};
#define VSA_FWD_AS(D_, NW_, LIST_, PAIRS_, COARSE_, RASTER_, MAP_)                                                    \
  k_fine_fwd<D_, NW_, LIST_, PAIRS_, COARSE_, RASTER_><<<workgroups(grid, pairs), 64 * NW_, 0, s>>>(                   \
      Nc, K, sl2, (const uint4*)q, (const uint4*)k, (const uint4*)v, (const uint4*)gate_c, (const uint4*)gate_f, idx, oc, mask, \
      (uint4*)out, (uint4*)out_fine, lse_f, H, ohs, ors, m_blocks, grid, pairs, stream, arrived, every, small, MAP_)
#define VSA_FWD_IO(D_, NW_, LIST_, PAIRS_, COARSE_)                                    \
  do {                                                                                 \
    if (raster.on) VSA_FWD_AS(D_, NW_, LIST_, PAIRS_, COARSE_, RasterMap, raster);     \
    else VSA_FWD_AS(D_, NW_, LIST_, PAIRS_, COARSE_, NoRaster, NoRaster{});            \
  } while (0)
#define VSA_FWD(D_, NW_, LIST_, COARSE_)                                               \
  do {                                                                                 \
    if (pairs) VSA_FWD_IO(D_, NW_, LIST_, (D_ == 128 && NW_ == 2), COARSE_);           \
    else VSA_FWD_IO(D_, NW_, LIST_, false, COARSE_);                                   \
  } while (0)
  const bool four = route.waves == 4;
  if (coarse) {
    if (d == 128) VSA_FWD(128, 4, CubeUnits, true);
    else VSA_FWD(64, 4, CubeUnits, true);
  } else if (key_cubes_16) {  // K counts key cubes of 16 tokens
    if (d == 128 && four) VSA_FWD(128, 4, SubCubeUnits, false);
    else if (d == 128) VSA_FWD(128, 2, SubCubeUnits, false);
    else if (four) VSA_FWD(64, 4, SubCubeUnits, false);
    else VSA_FWD(64, 2, SubCubeUnits, false);
  } else {
    if (d == 128 && four) VSA_FWD(128, 4, CubeUnits, false);
    else if (d == 128) VSA_FWD(128, 2, CubeUnits, false);
    else if (four) VSA_FWD(64, 4, CubeUnits, false);
    else VSA_FWD(64, 2, CubeUnits, false);
  }
#undef VSA_FWD
#undef VSA_FWD_AS
#undef VSA_FWD_IO
  return hipGetLastError();
}

}  // namespace vsa
