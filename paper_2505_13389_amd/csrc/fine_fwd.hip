// Fine stage forward (Sec. 2.2 fine stage; Sec. 2.1 attention equation under the block mask)
// fused with the gated combine O = O_c * G_c + O_f * G_f.
//
// One workgroup per (b, h, 64-row query block); "cube" below means such a block (a cube of 64*m tokens is m
// consecutive blocks, and the lists the kernel gets name blocks).  A workgroup is two wavefronts (four where the
// launch is too small to fill the chip), each with a list walk, LDS stages and an online softmax of its own:
// it multiplies UNITS of 32 keys with all 64 query rows (unit_stream.h), so that every operand it reads from
// LDS feeds two matrix instructions, and since nobody else reads its rows the loop has no barrier.  The partial
// results are merged once, through LDS, at the end.
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
// What bounds it: instruction issue.  A unit is 32 matrix instructions and 190 others (112 of softmax: fma, exp2, sum,
// half a conversion per value; 24 LDS reads, 16 copies): 1650 cycles at 1.77 GHz where the matrix pipe needs 1024;
// without waiting for any copy it is as fast, and without the copies 6 to 15 % faster.  About 7 us of a workgroup's
// 80 are start-up, merge and stores, which nothing overlaps on its SIMD.
// Measured against 32 keys x 32 queries per wavefront, four wavefronts in step, two per SIMD (every operand fed one
// matrix instruction; the vector work of one wavefront behind the matrix work of another): 39936 tokens, 12
// heads, d = 128, top-78 of 624: 1.47 -> 1.28 ms (i.i.d. selections), 1.43 -> 1.22 ms (local ones); 16384 tokens,
// top-32 of 256: 263 -> 241 us; B = 2, 16 heads, top-128 of 256: 2.38 -> 2.09 ms; d = 64, B = 2, 8 heads, top-32:
// 193 -> 172 us.
#include <type_traits>

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

template <int D, int NW, template <class> class UNITS>
__global__ __launch_bounds__(64 * NW, D == 128 ? 1 : 2) void k_fine_fwd(
    int Nc_, int K_, float sl2, const uint4* __restrict__ q, const uint4* __restrict__ k, const uint4* __restrict__ v,
    const uint4* __restrict__ gc, const uint4* __restrict__ gf, const int32_t* __restrict__ idx,
    const float* __restrict__ oc, const uint64_t* __restrict__ mask, uint4* __restrict__ out,
    uint4* __restrict__ out_fine, float* __restrict__ lse_f, int H, long long out_head_stride, long long out_row_stride,
    int m_blocks, unsigned* __restrict__ gang_arrived, unsigned gang_every) {
  using TL = Tile<D>;
  using UL = UNITS<TL>;
  using UC = UnitCopy<TL, UL>;
  constexpr int CPR = TL::CPR, KS = D / 16, DVB = D / 32, NT = 64 * NW, LPT = kTile * CPR / NT;
  constexpr int EPR = NW / 2;           // tiles a round of units takes
  constexpr int HALF = TL::BYTES / 2;   // 32 rows
  constexpr int NC = UC::NC;            // copy instructions per 32 rows
  constexpr int NPV = 2 * DVB;          // steps of the PV phase
  // LDS operands are read in pairs (one wait for both), kAhead steps before the first of them is used
  constexpr int kAhead = D == 128 ? 4 : 2;
  constexpr int kEarly = 7;             // of the 16 softmax items of a unit, those behind the PV phase before it
  constexpr int OS = D;
  // per wavefront: K of two units, V of two units
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NW * 4 * HALF];
  __shared__ float ml[NW * 64 * 2];
  static_assert(HALF % 256 == 0, "the operand addresses XOR the bits below 256");
  static_assert(KS == NPV && KS > kAhead, "phase interleave");

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
  const unsigned wg = same_lists ? block : xcd_chunked_id(block, gridDim.x);
  const int c = wg % Nc;
  const long long bh = wg / Nc;
  const int rot = same_lists ? ((c >> 3) & 15) % tiles : 0;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, h = lane >> 5;
  const int first = wave >> 1, half = wave & 1;  // this wavefront's tiles: first, first + EPR, ...
  const int nu = tiles > first ? (tiles - first + EPR - 1) / EPR : 0;
  auto tile_of = [&](int u) { const int t = first + EPR * u + rot; return t >= tiles ? t - tiles : t; };
  const long long rows0 = bh * (long long)Nc * kTile;  // first row of this (b,h)
  const unsigned char* kb = (const unsigned char*)uniform_ptr(k + rows0 * CPR);
  const unsigned char* vb = (const unsigned char*)uniform_ptr(v + rows0 * CPR);

  // Start-up: the list first (one round trip), then the copies of the first units and of Q (which waits in
  // the second V stages of the first two wavefronts), then the key masks, all in flight together.
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
  list.init(idx + (bh * Nc + c) * (long long)K, mask, K, half, lane, Nc, nu > 0 ? tile_of(0) : 0);
  Unit un[3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};  // the units after the current one
  Unit u0 = {0, 0, 0};
  bool second = false;  // unit 1 is requested already
  if (nu > 0) {
    list.rows(tile_of(0), u0);
    copy.all(kb, u0, lds0);
  }
  if (NW == 2 || wave < 2) {  // half w of Q by wavefront w
    UnitCopy<TL, CubeUnits<TL>> cq;
    cq.init(lane);
    const Unit uq = {(unsigned)half * HALF, (unsigned)half * HALF + HALF / 2, 0};
    cq.all((const unsigned char*)uniform_ptr(q + (rows0 + (long long)c * kTile) * CPR), uq, lds0 + 3 * HALF);
  }
  if (nu > 0) copy.all(vb, u0, lds0 + 2 * HALF);
  if (nu > 1 && list.loaded(tile_of(1))) {
    list.rows(tile_of(1), un[0]);
    copy.all(kb, un[0], lds0 + HALF);
    second = true;
  }
  list.load_masks();
  asm volatile("" : "+v"(list.km_v));
#pragma unroll
  for (int x = 0; x < DVB; ++x)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[x][b][i] = 0.f;
#pragma unroll
  for (int x = 0; x < DVB; ++x)  // (zeroed once, right here, while the first copies are in flight)
#pragma unroll
    for (int b = 0; b < 2; ++b) pin_o(o[x][b]);
  if (nu > 0) list.get(tile_of(0), u0);
  if (nu > 1) {
    list.get(tile_of(1), un[0]);
    if (!second) copy.all(kb, un[0], lds0 + HALF);
  }
  if (nu > 2) list.get(tile_of(2), un[1]);
  wait_vmcnt<0>();
  __syncthreads();
  bf16x8 qreg[2][KS];
  {
    const int lane_q = TL::rowmajor_lane(0, lane) + 3 * HALF;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qreg[0][s] = TL::rowmajor_at(smem, lane_q, s);
      qreg[1][s] = TL::rowmajor_at(smem + 4 * HALF, lane_q, s);
    }
  }
#pragma unroll
  for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qreg[0][s]), "+v"(qreg[1][s]));
  __syncthreads();  // every wavefront has Q: the second V stages may be filled

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
  float lsum[2] = {0.f, 0.f}, tsum[2] = {0.f, 0.f};
  uint4 pb[2][2];  // P^T of the current unit as operands: [query half][contraction step]
  auto put = [](uint4& u4, int w, uint32_t x) {
    if (w == 0) u4.x = x;
    if (w == 1) u4.y = x;
    if (w == 2) u4.z = x;
    if (w == 3) u4.w = x;
  };
  // softmax item `it` of 16: two values of one query half; the first eight make up contraction step 0
  auto p_item = [&](const f32x16 (&S)[2], int it, const float* rf) {
    const int st = it >> 3, b = (it >> 2) & 1, w = it & 3, e = 8 * st + 2 * w;
    const float x0 = fast_exp2(fmaf(S[b][e], sl2, -rf[b])), x1 = fast_exp2(fmaf(S[b][e + 1], sl2, -rf[b]));
    tsum[b] = (it & 11) == 0 ? x0 + x1 : tsum[b] + x0 + x1;
    const uint32_t pp = pack_bf16(x0, x1);
    put(pb[b][st], w, pp);
    asm volatile("" : "+v"(tsum[b]) : "v"(pp));  // (pure arithmetic has no place of its own in the order: tie it to this step)
  };
  auto p_items = [&](const f32x16 (&S)[2], int from, int to, const float* rf) {
#pragma unroll
    for (int it = from; it < to; ++it) p_item(S, it, rf);
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
#pragma unroll
    for (int s = 0; s < kAhead; ++s) kcur[s] = TL::rowmajor_at(smem + HALF, lane_a, s);
    valid = u0.valid;
    if (valid) {
      ref[0] = unit_max(s0[0], valid, kNoRef);
      ref[1] = unit_max(s0[1], valid, kNoRef);
      have = true;
    }
    p_items(s0, 0, kEarly, ref);
  }

  // One unit u (its S is there, in S): P(u) while S(u+1) is multiplied into T, then PV(u) while P(u+1) begins.
  // KIND 2: the units up to u + 3 exist; 1: u + 1 exists; 0: u is the last one.  `par` = u & 1.
  auto body = [&](auto kind_tag, int par, f32x16 (&S)[2], f32x16 (&T)[2], int u) {
    constexpr int KIND = decltype(kind_tag)::value;
    constexpr bool more1 = KIND >= 1;
    const bool more2 = KIND == 2 || (KIND == 1 && u + 2 < nu), more3 = KIND == 2 || (KIND == 1 && u + 3 < nu);
    const unsigned char* kn = smem + (1 - par) * HALF;  // K(u+1)
    const unsigned char* vc = smem + (2 + par) * HALF;  // V(u)
    bf16x8 ka[KS + kAhead], va[NPV + kAhead];
    auto v_op = [&](int i) { return TL::transposed_at(vc, lane_b0, lane_b1, i / DVB, i % DVB); };
    if (more1) {
#pragma unroll
      for (int s = 0; s < kAhead; ++s) ka[s] = kcur[s];
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---- S(u+1) | the rest of P(u), the copy of V(u+1), the first V operands
    constexpr int LATE = 16 - kEarly;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int i0 = kEarly + s * LATE / KS, i2 = kEarly + (s + 1) * LATE / KS, i1 = (i0 + i2) / 2;
      if (more1 && s % 2 == 0) {  // this pair is there; newer: the next one
        if (kAhead == 2) wait_lgkmcnt<0>();
        else if (s + 2 < KS) wait_lgkmcnt<2>();
        else wait_lgkmcnt<4>();
        __builtin_amdgcn_sched_barrier(0);
      }
      if (more1) {
        T[0] = mfma32(ka[s], qreg[0][s], s == 0 ? zero16 : T[0]);
        if (s < KS - kAhead) {
#pragma unroll
          for (int e = s * NC / (KS - kAhead); e < (s + 1) * NC / (KS - kAhead); ++e)
            copy.piece(vb, un[0], lds0 + (3 - par) * HALF, e);
        }
      }
      p_items(S, i0, i1, ref);
      if (s == KS - kAhead) {  // V(u) has landed; newer: K(u+2) and V(u+1)
        if (more2) wait_vmcnt<2 * NC>();
        else if (more1) wait_vmcnt<NC>();
        else wait_vmcnt<0>();
      }
      __builtin_amdgcn_sched_barrier(0);
      if (more1) {
        T[1] = mfma32(ka[s], qreg[1][s], s == 0 ? zero16 : T[1]);
      }
      if (s % 2 == 0) {
#pragma unroll
        for (int j = s + kAhead; j < s + kAhead + 2; ++j) {
          if (j >= KS) va[j - KS] = v_op(j - KS);
          else if (more1) ka[j] = TL::rowmajor_at(kn, lane_a, j);
        }
      }
      p_items(S, i1, i2, ref);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more1) {
      if (un[0].valid != 0xffffffffu) add_bias(T, un[0].valid);
    }
    // The reference of a column stays as long as neither lane's sum of 16 values exceeds `limit`: then no value does, and
    // the rescaling of O is skipped for almost every unit.  The result is exact either way, and a lane's arithmetic
    // never depends on what other query columns (pad rows included) hold.
    // (A unit without a valid key leaves every value at zero; the first one that has some sets the reference.)
    if (__builtin_expect((!have && valid) || __any(fmaxf(tsum[0], tsum[1]) > limit), 0)) {
      // (the last products that wrote O lie a whole S phase back, so it can be read at once)
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
        for (int st = 0; st < 2; ++st) p_items(S, 8 * st + 4 * b, 8 * st + 4 * b + 4, use);
      }
      have = true;
    }
    lsum[0] += tsum[0];
    lsum[1] += tsum[1];
    // ---- PV(u) | the first of P(u+1), the copy of K(u+3), the first K operands of u+2
    const uint4 pc[2][2] = {{pb[0][0], pb[0][1]}, {pb[1][0], pb[1][1]}};
    if (more3) list.get(tile_of(u + 3), un[2]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 1");  // (two wait states between the moves to pc and the first matrix instruction)
#pragma unroll
    for (int i = 0; i < NPV; ++i) {
      const int i0 = i == 0 ? 0 : (i - 1) * kEarly / (NPV - 1), i2 = i * kEarly / (NPV - 1), i1 = (i0 + i2) / 2;
      if (i % 2 == 0) {
        if (kAhead == 2) wait_lgkmcnt<0>();
        else if (i + 2 < NPV) wait_lgkmcnt<4>();
        else wait_lgkmcnt<2>();
        __builtin_amdgcn_sched_barrier(0);
      }
      mfma_o(o[i % DVB][0], va[i], __builtin_bit_cast(bf16x8, pc[0][i / DVB]));
      if (more3 && i < NPV - kAhead) {
#pragma unroll
        for (int e = i * NC / (NPV - kAhead); e < (i + 1) * NC / (NPV - kAhead); ++e)
          copy.piece(kb, un[2], lds0 + (1 - par) * HALF, e);
      }
      if (more1) p_items(T, i0, i1, ref);
      if (more1 && i == NPV - kAhead) {  // K(u+2) has landed; newer: V(u+1) and K(u+3)
        if (more3) wait_vmcnt<2 * NC>();
        else if (more2) wait_vmcnt<NC>();
      }
      __builtin_amdgcn_sched_barrier(0);
      mfma_o(o[i % DVB][1], va[i], __builtin_bit_cast(bf16x8, pc[1][i / DVB]));
      if (i % 2 == 0) {
#pragma unroll
        for (int j = i + kAhead; j < i + kAhead + 2; ++j) {
          if (j < NPV) va[j] = v_op(j);
          else if (more1) kcur[j - NPV] = TL::rowmajor_at(smem + par * HALF, lane_a, j - NPV);  // (unused if u + 2 does not exist)
        }
      }
      if (more1) p_items(T, i1, i2, ref);
      __builtin_amdgcn_sched_barrier(0);
    }
    valid = un[0].valid;
    un[0] = un[1];
    un[1] = un[2];
  };
  if (nu > 0) {
    const std::integral_constant<int, 2> steady;
    const std::integral_constant<int, 1> inner;
    const std::integral_constant<int, 0> last;
    int u = 0;
    for (; u + 4 < nu; u += 2) {
      body(steady, 0, s0, s1, u);
      body(steady, 1, s1, s0, u + 1);
    }
    for (; u + 1 < nu; ++u) {
      body(inner, u & 1, s0, s1, u);
      s0[0] = s1[0];
      s0[1] = s1[1];
    }
    body(last, u & 1, s0, s1, u);
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
  // ---- merge the wavefronts' partial results, normalise, gate, store
  // The gates and the coarse output of this thread's items are requested first: they arrive while
  // the partial results go through LDS.  Pad rows are loaded too (they exist in memory) and ignored.
  static_assert(NT % CPR == 0, "a thread keeps its column chunk");
  const uint64_t qmask = mask[c];
  const int ch = tid % CPR;
  uint4 gc_raw[LPT], gf_raw[LPT];
  const float* ocr = oc + ((bh * Nc + c) / m_blocks) * D + ch * 8;  // O_c is per cube = m_blocks blocks
  const float4 c0 = *(const float4*)ocr, c1 = *(const float4*)(ocr + 4);
#pragma unroll
  for (int it = 0; it < LPT; ++it) {
    const long long g = (rows0 + c * kTile + (it * NT + tid) / CPR) * CPR + ch;
    gc_raw[it] = gc[g];
    gf_raw[it] = gf ? gf[g] : make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);  // bf16 ones
  }
  __syncthreads();  // every wavefront is done with its stages
  {
    float* Op = (float*)smem + wave * 64 * OS;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
#pragma unroll
      for (int x = 0; x < DVB; ++x)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
          *(float4*)&Op[merge_offset(b * 32 + l32, x * 32 + 8 * g4 + 4 * h, OS)] =
              make_float4(o[x][b][4 * g4], o[x][b][4 * g4 + 1], o[x][b][4 * g4 + 2], o[x][b][4 * g4 + 3]);
      const float l = lsum[b] + __shfl_xor(lsum[b], 32);
      if (h == 0) {
        // (kNoRef: every logit of the column was -inf)
        ml[(wave * 64 + b * 32 + l32) * 2] = have && ref[b] > kNoRef ? ref[b] : -INFINITY;
        ml[(wave * 64 + b * 32 + l32) * 2 + 1] = l;
      }
    }
  }
  __syncthreads();

  bool overflow = false;
#pragma unroll
  for (int it = 0; it < LPT; ++it) {
    const int r = (it * NT + tid) / CPR;
    float M = ml[r * 2], L = 0.f, most = 0.f, f[NW];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, ml[(w * 64 + r) * 2]);
    // (M = -inf: the list named no valid key at all -- only a caller-supplied list can, e.g. one made of
    // dead key cubes; the row then gets O_f = 0 and lse = 0 instead of NaN)
    const bool none = M == -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      f[w] = none ? 0.f : fast_exp2(ml[(w * 64 + r) * 2] - M);
      L += ml[(w * 64 + r) * 2 + 1] * f[w];
      most = fmaxf(most, ml[(w * 64 + r) * 2 + 1]);
    }
    const float inv = none ? 0.f : 1.0f / L;
    const int m0 = merge_offset(r, ch * 8, OS), m1 = merge_offset(r, ch * 8 + 4, OS);
    float of[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f}, res[8];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* Op = (const float*)smem + w * 64 * OS;
      const float4 a0 = *(const float4*)(Op + m0), a1 = *(const float4*)(Op + m1);
      const float fw = f[w] * inv;
      of[0] = fmaf(a0.x, fw, of[0]); of[1] = fmaf(a0.y, fw, of[1]); of[2] = fmaf(a0.z, fw, of[2]); of[3] = fmaf(a0.w, fw, of[3]);
      of[4] = fmaf(a1.x, fw, of[4]); of[5] = fmaf(a1.y, fw, of[5]); of[6] = fmaf(a1.z, fw, of[6]); of[7] = fmaf(a1.w, fw, of[7]);
    }
    const long long g = (rows0 + c * kTile + r) * CPR + ch;
    uint4 ov = make_uint4(0, 0, 0, 0), fv = make_uint4(0, 0, 0, 0);
    if ((qmask >> r) & 1) {
      float gcv[8], gfv[8];
      unpack8(gc_raw[it], gcv);
      unpack8(gf_raw[it], gfv);
      const float ocv[8] = {c0.x, c0.y, c0.z, c0.w, c1.x, c1.y, c1.z, c1.w};
#pragma unroll
      for (int e = 0; e < 8; ++e) res[e] = fmaf(ocv[e], gcv[e], of[e] * gfv[e]);
      ov = pack8(res);
      fv = pack8(of);
      float nought = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) nought = fmaf(of[e], 0.f, nought);  // NaN unless all of them are finite
      overflow |= most > kTightSum && nought != 0.f;
    }
    out[out0 + (long long)(c * kTile + r) * out_row_stride + ch] = ov;
    if (out_fine) out_fine[g] = fv;
    if (lse_f && ch == 0) lse_f[rows0 + c * kTile + r] = (((qmask >> r) & 1) && !none) ? (M + fast_log2(L)) * kLn2 : 0.f;
  }
  if (tight) return;
  if (overflow) again = 1;
  __syncthreads();
  if (!again) return;
  }
}

// Which kernel, by the number of query blocks and of 64-key tiles in a list (times in us: one head size, lists of N(0,1)
// inputs, B*H*Nb from 64 to 7488).  512 workgroups of the d = 128 kernels are on the chip at a time, 1024 of the d = 64
// kernel with two wavefronts, 512 of the one with four.
//
// The kernel for short lists, whose workgroups hide one another's start-up and wind-down but which takes longer per tile:
//   d = 128  full generations: 384 blocks, 6 tiles 17.7 against 17.4; 512, 8 tiles 21.0 / 22.4, 12 tiles 25.0 / 24.4; 1024, 20 tiles 59.5 / 60.1, 24
//            tiles 69.5 / 67.2; 3072, 20 tiles 165 / 166, 33 tiles 246 / 237.  A last generation that is at most half
//            full costs the general kernel more, the less the more generations there are: 576 blocks, 16 tiles 40.3 / 43.9,
//            56 tiles 104 / 108; 1152, 16 tiles 62.2 / 69.5, 48 tiles 145 / 149; 1600, 28 tiles 127 / 134; 4160, 24 tiles 1.02.
//   d = 64   up to 14 tiles, unless the blocks just fill the chip with two-wavefront workgroups (1024 blocks, 12 tiles 27.4 /
//            23.8) or there are generations enough (4160, 12 tiles 0.95).
//   one or two tiles: 256 blocks 7.3 / 7.8, 9.2 / 9.6.
inline bool fwd_short(int d, unsigned grid, int tiles) {
  if (tiles <= 2) return true;
  if (d == 128) {
    const unsigned full = grid / 512, last = grid % 512;
    if (grid <= 256) return false;
    if (grid <= 512) return tiles <= (grid > 448 ? 12 : 8);
    return tiles <= (last > 0 && last <= 256 ? 20 + 40 / (int)full : 20);
  }
  if (grid <= 512 || (grid > 768 && grid <= 1024) || grid > 4096) return false;
  return tiles <= (grid <= 2560 ? 14 : 8);
}
// The general kernel with four wavefronts per workgroup: half as long a walk counts where the launch does not fill the chip
// with two-wavefront workgroups.  d = 64, 64 blocks, 8 tiles 10.0 against 12.0; 512 blocks, 33 tiles 27.6 / 37.2; 640 blocks
// 0.93 of it, 1536 0.87; 1024 blocks 1.05, 2560 0.95 to 1.01.  d = 128, 256 blocks, 33 tiles 26.2 / 34.8, 384 blocks 44.0 / 37.2.
inline bool fwd_four_waves(int d, unsigned grid, int tiles) {
  if (d == 128) return grid <= 256;
  return grid <= 512 || (tiles > 14 && grid <= 2560 && !(grid > 768 && grid <= 1024));
}

hipError_t launch_fine_fwd(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                           const void* gate_c, const void* gate_f, const int32_t* idx, const float* oc,
                           const uint64_t* mask, void* out, void* out_fine, float* lse_f, int H, int out_token_major,
                           int m_blocks, int key_cubes_16, unsigned* gang_scratch, hipStream_t s) {
  const float sl2 = scale * kLog2e;
  const unsigned grid = (unsigned)(BH * Nc);
  const int tiles = key_cubes_16 ? (K + 3) / 4 : K;
  if (fwd_short(d, grid, tiles))
    return launch_fine_fwd_short(BH, Nc, d, K, scale, q, k, v, gate_c, gate_f, idx, oc, mask, out, out_fine, lse_f, H,
                                 out_token_major, m_blocks, key_cubes_16, s);
  // Gangs, one in about every 256 tiles walked, at d = 128 where the K and V of a head are many times an L2, the lists differ
  // and there are 16 generations (heads of 64 MiB: two).  Without / with, lists of N(0,1) inputs, then local ones: 1440
  // blocks (45 MiB), 40 heads, lists of 96 14.3 / 13.1, 13.4 / 13.0 ms, of 180 32.9 / 23.3 (L2 hits 0.38 without); 16 heads,
  // 180 9.66 / 9.06, 9.06 / 8.87 ms, 60 3.25 / 3.29, 3.31 / 3.36; 1152 blocks (36 MiB), 12 heads, 32 1.55 / 1.42, 1.10 / 1.13;
  // 2160 blocks (68 MiB), 2 heads, 180 2.72 / 2.62, 1.60 / 1.59, 4 heads 5.10 / 3.43, 3.17 / 3.20.  Elsewhere the waits
  // cost more than the hits return: 1440 blocks, 2 heads, 32 228 / 240 us; 624 blocks (19.5 MiB) 1.23 / 1.26 ms; d = 64,
  // 1440 blocks, 16 heads, 180 4.62 / 4.83, 4.55 / 4.72 ms, 2 heads, 24 105 / 123 us.
  const size_t head = (size_t)Nc * kTile * d * 4;  // bytes of its K and V
  const bool gangs = d == 128 && tiles < Nc &&
                     ((head >= ((size_t)22 << 20) && grid >= 8192) || (head >= ((size_t)64 << 20) && grid >= 1024));
  const unsigned every = gangs ? (unsigned)(255 / tiles + 1) : 1u;
  unsigned* arrived = gangs ? gang_scratch : nullptr;
  if (gangs) {
    const unsigned n = 8 * ((grid / 8 + kGang) / kGang + 1);  // (at most BH*Nc/32 + 24 counters)
    k_gang_clear<<<(n + 255) / 256, 256, 0, s>>>(arrived, n);
  }
  const long long cpr = d / 8, Np = (long long)Nc * kTile;
  const long long ohs = out_token_major ? cpr : Np * cpr, ors = out_token_major ? H * cpr : cpr;
#define VSA_FWD(D_, NW_, LIST_)                                                                                      \
  k_fine_fwd<D_, NW_, LIST_><<<grid, 64 * NW_, 0, s>>>(Nc, K, sl2, (const uint4*)q, (const uint4*)k, (const uint4*)v,  \
                                             (const uint4*)gate_c, (const uint4*)gate_f, idx, oc, mask, (uint4*)out, \
                                             (uint4*)out_fine, lse_f, H, ohs, ors, m_blocks, arrived, every)
#define VSA_FWD_NW(D_, LIST_)                     \
  do {                                            \
    if (fwd_four_waves(D_, grid, tiles)) VSA_FWD(D_, 4, LIST_); \
    else VSA_FWD(D_, 2, LIST_);                   \
  } while (0)
  if (key_cubes_16) {  // K counts key cubes of 16 tokens
    if (d == 128) VSA_FWD_NW(128, SubCubeUnits);
    else VSA_FWD_NW(64, SubCubeUnits);
  } else {
    if (d == 128) VSA_FWD_NW(128, CubeUnits);
    else VSA_FWD_NW(64, CubeUnits);
  }
#undef VSA_FWD_NW
#undef VSA_FWD
  return hipGetLastError();
}

}  // namespace vsa
