// The stream of the forward and the dQ kernel: UNITS of 32 key rows, each copied by the one wavefront that
// multiplies it, global -> LDS, into stages of that wavefront's own.  A list is walked in tiles of 64 keys = two
// units each; of P wavefronts that share a list wavefront w takes the units w, w + P, ...
//
// A unit is two groups of 16 consecutive LDS rows whose sources may lie apart (lists that name key cubes of
// 16 tokens gather a tile from four entries).  The list sits in a register, 64 entries at a time (lane e
// holds entry e of the current chunk) with the valid-key bits of the entries, and is read with v_readlane:
// no load and no wait on one sits in the loops except where a chunk ends.
#pragma once
#include "fine_tile.h"

namespace vsa {

constexpr float kMaskBias = -30000.f;  // added to the raw logits of pad keys (|q.k| is assumed < 15000)

// Byte offsets of a unit's two 16-row groups from the first row of the (b, h), and its 32 valid-key bits.
struct Unit {
  unsigned a, b;
  uint32_t valid;
};

// Lists that name 64-row blocks: one tile per entry.
template <class TL>
struct CubeUnits {
  const int32_t* list;
  const uint64_t* mask;
  int n, lane, chunk, idx_v, ncubes;
  int only = -1;     // the half that all units of this wavefront are (-1: both)
  uint32_t km_v[2];  // valid-key bits of the two halves of the lane's entry
  static constexpr int kEntriesPerTile = 1, kTilesPerChunk = 64;
  static constexpr bool kContiguous = true;  // a unit's 32 rows lie one behind the other
  __device__ __forceinline__ void arrived() {
    asm volatile("" : "+v"(idx_v));  // consumed here: the compiler's wait for the load is placed right here
    idx_v = clamp_cube(idx_v, ncubes);  // (a caller-supplied list is not trusted)
  }
  __device__ __forceinline__ void load_indices(int c) {
    chunk = c;
    idx_v = list[list_slot(c, lane, n)];
    arrived();
  }
  __device__ __forceinline__ int mask_block() const { return idx_v; }
  __device__ __forceinline__ void set_masks(uint64_t m) {
    km_v[0] = (uint32_t)m;
    km_v[1] = (uint32_t)(m >> 32);
    if (only >= 0) km_v[0] = km_v[only ? 1 : 0];
  }
  // (after arrived() the offsets of the units of tile t's chunk are there; the valid-key bits come with set_masks)
  __device__ __forceinline__ void request(const int32_t* list_, const uint64_t* mask_, int n_, int lane_, int ncubes_, int t) {
    list = list_, mask = mask_, n = n_, lane = lane_, ncubes = ncubes_;
    chunk = t / kTilesPerChunk;
    idx_v = list[list_slot(chunk, lane, n)];
  }
  // a list of up to 64 entries, in LDS
  __device__ __forceinline__ void take(const int32_t* lds_list, const uint64_t* mask_, int n_, int lane_, int ncubes_) {
    list = nullptr, mask = mask_, n = n_, lane = lane_, ncubes = ncubes_, chunk = 0;
    idx_v = lds_list[list_slot(0, lane, n)];
  }
  __device__ __forceinline__ bool loaded(int t) const { return (unsigned)t / kTilesPerChunk == (unsigned)chunk; }
  __device__ __forceinline__ void rows(int t, int half, Unit& u) const {
    u.a = (unsigned)__builtin_amdgcn_readlane(idx_v, t & 63) * (unsigned)TL::BYTES + (unsigned)half * (TL::BYTES / 2);
    u.b = u.a + TL::BYTES / 4;
  }
  // a unit in parts: the chunk of its tile, its rows, its valid-key bits
  __device__ __forceinline__ void load(int t) {
    if (__builtin_expect(!loaded(t), 0)) {
      load_indices(t / kTilesPerChunk);
      set_masks(mask[mask_block()]);
      asm volatile("" : "+v"(km_v[0]), "+v"(km_v[1]));
    }
  }
  __device__ __forceinline__ void valid(int t, int half, Unit& u) const {
    u.valid = (uint32_t)__builtin_amdgcn_readlane((int)km_v[0], t & 63);
    if (only < 0) {
      const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)km_v[1], t & 63);
      u.valid = half ? hi : u.valid;
    }
  }
  __device__ __forceinline__ void get(int t, int half, Unit& u) {
    load(t);
    rows(t, half, u);
    valid(t, half, u);
  }
  __device__ static __forceinline__ int source_row(int x) { return x; }
};

// Lists that name key cubes of 16 tokens (see subcube_* in list_rules.h): a tile is four entries, and row x of
// a 16-row group is token x of its key cube.  Entries past the end repeat the last one with no valid key.
template <class TL>
struct SubCubeUnits {
  const int32_t* list;
  const uint64_t* mask;
  int n, lane, chunk, idx_v, ncubes;
  int only = -1;  // (as in CubeUnits; of no use here)
  uint32_t km_v;  // 16 valid-key bits of the lane's entry
  static constexpr int kEntriesPerTile = 4, kTilesPerChunk = 16;
  static constexpr bool kContiguous = false;
  __device__ __forceinline__ void arrived() {
    asm volatile("" : "+v"(idx_v));
    idx_v = clamp_cube(idx_v, 4 * ncubes);
  }
  __device__ __forceinline__ void load_indices(int c) {
    chunk = c;
    idx_v = list[list_slot(c, lane, n)];
    arrived();
  }
  __device__ __forceinline__ int mask_block() const { return idx_v >> 2; }
  __device__ __forceinline__ void set_masks(uint64_t m) { km_v = subcube_mask16(m, idx_v & 3); }
  __device__ __forceinline__ void request(const int32_t* list_, const uint64_t* mask_, int n_, int lane_, int ncubes_, int t) {
    list = list_, mask = mask_, n = n_, lane = lane_, ncubes = ncubes_;
    chunk = t / kTilesPerChunk;
    idx_v = list[list_slot(chunk, lane, n)];
  }
  __device__ __forceinline__ bool loaded(int t) const { return (unsigned)t / kTilesPerChunk == (unsigned)chunk; }
  __device__ __forceinline__ unsigned entry_offset(int e) const {  // e in the current chunk
    const int id = __builtin_amdgcn_readlane(idx_v, min(e, n - 1) & 63);
    return (unsigned)(id >> 2) * (unsigned)TL::BYTES + (unsigned)subcube_first_slot(id & 3) * (unsigned)TL::ROW_BYTES;
  }
  __device__ __forceinline__ void rows(int t, int half, Unit& u) const {
    u.a = entry_offset(4 * t + 2 * half);
    u.b = entry_offset(4 * t + 2 * half + 1);
  }
  __device__ __forceinline__ void load(int t) {
    if (__builtin_expect(!loaded(t), 0)) {
      load_indices(t / kTilesPerChunk);
      set_masks(mask[mask_block()]);
      asm volatile("" : "+v"(km_v));
    }
  }
  __device__ __forceinline__ void valid(int t, int half, Unit& u) const {
    const int ea = 4 * t + 2 * half, eb = ea + 1;
    const uint32_t ma = (uint32_t)__builtin_amdgcn_readlane((int)km_v, ea & 63);
    const uint32_t mb = (uint32_t)__builtin_amdgcn_readlane((int)km_v, eb & 63);
    u.valid = (ea < n ? ma : 0u) | ((eb < n ? mb : 0u) << 16);
  }
  __device__ __forceinline__ void get(int t, int half, Unit& u) {
    load(t);
    rows(t, half, u);
    valid(t, half, u);
  }
  __device__ static __forceinline__ int source_row(int x) { return subcube_slot(x); }
};

// Forward and dQ: a workgroup of two wavefronts takes one block, whose units they share, or two blocks, one each.  The
// second form has half as many starts and nothing to merge, but its workgroups run twice as long; so all blocks are
// paired where that takes no more generations of `places` workgroups, else those of the generations that are full.
// With two workgroups' wavefronts on a SIMD, whose speed depends on the other (dQ, d = 64: 1024 places), all are paired where the last
// generation is three quarters full, and none where it is between an eighth and that.  None / those of full generations, us, top-9
// and top-32: 2304 blocks 48.6 / 46.3, 124.8 / 124.0; 2400 51.8 / 53.5, 130 / 137; 2520, top-8 and 30 44.9 / 47.5, 122 / 136; 3360 56.0 /
// 58.4, 163 / 167.  None / all: 1536 37.6 / 35.3, 97.2 / 93.9; 2048 46.7 / 40.5, 108.9 / 107.7; 8192 142.7 / 141.8, 407 / 401.
inline unsigned paired_workgroups(unsigned blocks, unsigned places) {
  const bool two = places > 512;
  const unsigned rest = blocks % (2 * places), enough = two ? places + places / 2 - 1 : places;
  if (rest == 0 || rest > enough) return (blocks + 1) / 2;
  return two && rest > places / 4 ? 0 : blocks / (2 * places) * places;
}
inline unsigned workgroups(unsigned blocks, unsigned pairs) { return 2 * pairs >= blocks ? pairs : blocks - pairs; }

// The masks of the first chunk's entries by way of LDS (512 bytes at `lds`), like the copies they precede: a load to
// registers among the copies would make the compiler wait for all of them.
template <class UNITS>
__device__ __forceinline__ void request_masks(const UNITS& list, unsigned lds) {
  const unsigned char* base = (const unsigned char*)list.mask;  // (a kernel argument)
  const unsigned off = (unsigned)list.mask_block() * 8u;
  lds_dma4<4>(base, off, lds);
  lds_dma4<4>(base + 4, off, lds + 256);
}
template <class UNITS>
__device__ __forceinline__ void take_masks(UNITS& list, const void* lds) {
  const uint32_t* m = (const uint32_t*)lds + list.lane;
  list.set_masks(m[0] | ((uint64_t)m[64] << 32));
}

// Copies of 32 rows by one wavefront (global_load_lds_dwordx4, see lds_dma16_at): instruction c fills rows c*RPI ..,
// the swizzle is applied on the SOURCE side (the lane that writes physical chunk pc of row r fetches logical chunk
// pc ^ swz(r)) and repeats after 16 rows.  Every 16-row group has an M0 value of its own; where
// the 32 rows are contiguous one base address serves both, the distance is in the second group's lane offsets.
template <class TL, class UNITS>
struct UnitCopy {
  static constexpr int NC = 32 / TL::RPI;  // instructions
  static constexpr int GROUP = NC / 2;     // per 16-row group
  unsigned off[UNITS::kContiguous ? NC : GROUP];
  __device__ __forceinline__ void init(int lane) {
#pragma unroll
    for (int i = 0; i < (UNITS::kContiguous ? NC : GROUP); ++i) {
      const int x = i * TL::RPI + lane / TL::CPR, pc = lane % TL::CPR;
      off[i] = (unsigned)((UNITS::source_row(x) * TL::CPR + (pc ^ TL::swz(x))) * 16) - (unsigned)(i % GROUP) * 1024u;
    }
  }
  // instruction c (a constant after unrolling); `base` = first row of the (b, h), `lds` = the stage's address
  // (`aimed`: aim(lds, c) and another instruction came before it)
  __device__ __forceinline__ void aim(unsigned lds, int c) const {
    if (c % GROUP == 0) set_m0_ahead(lds + (unsigned)(c / GROUP) * (16u * TL::ROW_BYTES));
  }
  __device__ __forceinline__ void piece(const unsigned char* base, const Unit& u, unsigned lds, int c, bool aimed = false) const {
    const void* g = base + (UNITS::kContiguous || c < GROUP ? u.a : u.b);
    const int r = c % GROUP, o = UNITS::kContiguous ? c : r;
    if (r == 0 && !aimed) set_m0(lds + (unsigned)(c / GROUP) * (16u * TL::ROW_BYTES));
    if (r == 0) lds_dma16_at<0>(g, off[o]);
    if (r == 1) lds_dma16_at<1024>(g, off[o]);
    if (r == 2) lds_dma16_at<2048>(g, off[o]);
    if (r == 3) lds_dma16_at<3072>(g, off[o]);
  }
  __device__ __forceinline__ void all(const unsigned char* base, const Unit& u, unsigned lds) const {
#pragma unroll
    for (int c = 0; c < NC; ++c) piece(base, u, lds, c);
  }
};

// Matrix instructions written as assembly, so that the register class of every accumulator is fixed: `_v`
// accumulates in ordinary registers, `_a` in the accumulation registers (left to the compiler, all
// accumulators of a kernel with more than 256 registers are accumulation registers, and every vector use of
// one costs a move).  The compiler does not see matrix instructions here and inserts none of the wait states
// they need; the kernels' fixed order provides them: a vector result is consumed by a matrix instruction
// no earlier than two instructions after it was written, and a matrix result is read by vector instructions
// no earlier than two matrix instructions after the one that completed it (tests/test_wait_states.py checks the
// emitted code of every instance).
__device__ __forceinline__ void mfma_v(f32x16& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_v_from(f32x16& d, bf16x8 a, bf16x8 b, const f32x16& c) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "v"(b), "v"(c));
}
__device__ __forceinline__ void mfma_a(f32x16& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
// 16x16x32 forms: half the passes, so what is far enough from a 32x32x16 instruction is far enough from one of these
__device__ __forceinline__ void mfma_v(f32x4& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_v_from(f32x4& d, bf16x8 a, bf16x8 b, const f32x4& c) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "v"(b), "v"(c));
}
__device__ __forceinline__ void mfma_a(f32x4& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(d) : "v"(a), "v"(b));
}
// (B operand in the accumulation registers)
__device__ __forceinline__ void mfma_v_from_qa(f32x4& d, bf16x8 a, bf16x8 b, const f32x4& c) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" : "=&v"(d) : "v"(a), "a"(b), "v"(c));
}
__device__ __forceinline__ void mfma_v_qa(f32x4& d, bf16x8 a, bf16x8 b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}
// matrix results land before the vector instructions behind this read them, and the other way round
__device__ __forceinline__ void mfma_fence() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

}  // namespace vsa
