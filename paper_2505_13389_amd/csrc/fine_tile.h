// LDS tile layout and MFMA operand access shared by the fine-stage kernels.
//
// A tile is 64 token rows x D bf16, row-major, stored in LDS WITHOUT padding; the 16-byte
// chunk c of row r lives at chunk position c ^ swz(r).  The swizzle is chosen so that both
// access patterns of the 32x32x16 MFMA operands are spread over distinct 16-byte bank groups:
//   - row-major reads (lane = row, same chunk): 16 consecutive rows hit 16 distinct slots;
//   - transposed reads (ds_read_b64_tr_b16: 4 consecutive rows x 64 contiguous bytes): the
//     4 rows land in 4 different 64-byte groups of the 256-byte bank line.
#pragma once
#include <type_traits>
#include <utility>

#include "list_rules.h"
#include "vsa_common.h"

namespace vsa {

typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef __attribute__((address_space(1))) const void* global_void_ptr;

// Byte address of an LDS object inside the workgroup's LDS allocation.
__device__ __forceinline__ unsigned lds_address(const void* p) {
  return (unsigned)(size_t)(__attribute__((address_space(3))) const unsigned char*)p;
}

// 64 lanes x 16 bytes, global -> LDS at M0 + IMM + lane*16; `base` and M0 wave-uniform.  The immediate byte offset is
// added to BOTH addresses (global and LDS): a run of copies whose LDS targets are IMM apart shares one M0
// value, the callers compensating in the per-lane global offsets.  0 <= IMM < 4096.
//
// The copies are issued from inline assembly on purpose: the compiler then keeps no record of them, so it never
// drains them early, and the kernels order them by hand -- completion is counted by vmcnt in issue order.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int IMM>
__device__ __forceinline__ void lds_dma16_at(const void* base, unsigned voff) {
  static_assert(IMM >= 0 && IMM < 4096, "13-bit signed instruction offset");
  asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" : : "v"(voff), "s"(base), "n"(IMM) : "memory");
}
// M0 is written here and read by the copies that follow in program order (volatile asm statements
// keep their order).  Nothing else in these kernels uses M0: no dynamically indexed register arrays
// (v_movrel), no GWS or message instructions.  One wait state has to lie between the write and the copy that reads it;
// the compiler inserts none for inline assembly.
__device__ __forceinline__ void set_m0(unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0" : : "s"(lds_addr) : "m0", "memory");
}
// (with another instruction between it and the copies)
__device__ __forceinline__ void set_m0_ahead(unsigned lds_addr) { asm volatile("s_mov_b32 m0, %0" : : "s"(lds_addr) : "m0", "memory"); }
// (NOPS 4: for a base that the compiler may fetch from a vector register right before, which takes 5 wait states)
template <int NOPS = 0>
__device__ __forceinline__ void lds_dma4(const void* base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop %3\n\tglobal_load_lds_dword %0, %1"
               :
               : "v"(voff), "s"(base), "s"(lds_addr), "n"(NOPS)
               : "memory", "m0");
}
#pragma clang diagnostic pop

// s_waitcnt immediates (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
// A pointer the caller knows to be wave-uniform, forced into scalar registers.
__device__ __forceinline__ const void* uniform_ptr(const void* p) {
  const unsigned long long a = (unsigned long long)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a), hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
  return (const void*)(((unsigned long long)hi << 32) | lo);
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}
template <int N>
__device__ __forceinline__ void wait_lgkmcnt() {
  __builtin_amdgcn_s_waitcnt(0xC07F | (N << 8));
}

// f(0), f(1), ..., f(N - 1), each with its number as a constant
template <class F, int... M>
__device__ __forceinline__ void in_steps_of(const F& f, std::integer_sequence<int, M...>) {
  (f(std::integral_constant<int, M>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void in_steps(const F& f) { in_steps_of(f, std::make_integer_sequence<int, N>{}); }

template <int D>
struct Tile {
  static constexpr int CPR = D / 8;               // 16-byte chunks per row
  static constexpr int ROW_BYTES = D * 2;
  static constexpr int BYTES = kTile * ROW_BYTES;

  __device__ static __forceinline__ int swz(int r) {
    if (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
    return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
  }
  __device__ static __forceinline__ int off(int r, int c) { return r * ROW_BYTES + ((c ^ swz(r)) << 4); }

  static constexpr int RPI = 1024 / ROW_BYTES;   // rows per wave copy instruction (1 KiB of consecutive LDS)

  // MFMA 32x32x16 operand whose 32-index is the tile ROW and whose contraction index runs
  // along D: lane l supplies tile[row0 + l%32][16*s + 8*(l/32) .. +7]  (one 16-byte read).
  // The lane-dependent part of the address is split off: the swizzle is an XOR on the chunk bits, so the
  // k-step s enters as an XOR with a constant, everything else as a constant byte offset.
  __device__ static __forceinline__ int rowmajor_lane(int row0, int lane) { return off(row0 + (lane & 31), lane >> 5); }
  __device__ static __forceinline__ bf16x8 rowmajor_at(const unsigned char* tile, int lane_part, int s) {
    return *(const bf16x8*)(tile + (lane_part ^ (s << 5)));
  }

  // MFMA 32x32x16 operand whose 32-index runs along D (columns 32 x ..) and whose
  // contraction index is the tile ROW, in the order the 32x32 accumulator layout produces:
  // for k-step s, lane half h = l/32 and j = 0..7 the row is row0 + 16*s + 8*(j/4) + 4*h + j%4.
  // Two transposing 8-byte LDS reads; in each 16-lane block, lanes 4e..4e+3 read row e.  The column block
  // enters the address as an XOR with a constant;
  // valid for row0 a multiple of 32 (swz(r + 8) == swz(r) ^ 2 and swz(r + 16) == swz(r) then hold)
  __device__ static __forceinline__ void transposed_lane(int row0, int lane, int& b0, int& b1) {
    const int L = lane & 15;
    const int r1 = row0 + 4 * (lane >> 5) + (L >> 2);
    const int col = ((lane >> 4) & 1) * 16 + 4 * (L & 3);
    b0 = off(r1, col >> 3) + (col & 7) * 2;
    b1 = off(r1 + 8, col >> 3) + (col & 7) * 2;
  }
  __device__ static __forceinline__ bf16x4 transposed_half(const unsigned char* tile, int b, int s, int x) {  // b: b0 or b1
    const unsigned char* p = tile + s * 16 * ROW_BYTES;
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + (b ^ (x << 6))));
  }
  __device__ static __forceinline__ bf16x8 transposed_at(const unsigned char* tile, int b0, int b1, int s, int x) {
    const bf16x4 a0 = transposed_half(tile, b0, s, x), a1 = transposed_half(tile, b1, s, x);
    return __builtin_shufflevector(a0, a1, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

// The same rows for the operands of 16x16x32 matrix instructions, with a swizzle of its own:
//   - row-major reads: a phase of the LDS takes 16 lanes, of rows {0..3, 12..15} and {4..11} with neighbouring chunks (2j, 2j + 1
//     or the other way round): all 16 slots are hit if swz ^ 1 maps either half of the rows onto the slots of the other one's;
//   - transposed reads: a phase takes 32 lanes, 8 consecutive rows x 32 contiguous bytes: swz / 2 differs in rows 0..7 and in 8..15.
template <int D>
struct NarrowTile {
  static constexpr int CPR = Tile<D>::CPR, ROW_BYTES = Tile<D>::ROW_BYTES, BYTES = Tile<D>::BYTES, RPI = Tile<D>::RPI;

  __device__ static __forceinline__ int swz(int r) {
    static_assert(D == 128, "16 slots a row");
    const int low = (r >> 3) & 1;
    return (((r & 7) ^ (low << 2)) << 1) | low;
  }
  __device__ static __forceinline__ int off(int r, int c) { return r * ROW_BYTES + ((c ^ swz(r)) << 4); }

  // Operand whose 16-index is the tile ROW (16*b ..) and whose contraction index runs along D: for contraction step s lane l
  // supplies tile[16*b + l%16][32*s + 8*(l/16) .. +7]  (one 16-byte read; the lane's part of the address is split off as above).
  __device__ static __forceinline__ int rowmajor_lane(int lane) { return off(lane & 15, lane >> 4); }
  __device__ static __forceinline__ bf16x8 rowmajor_at(const unsigned char* tile, int lane_part, int b, int s) {
    return *(const bf16x8*)(tile + b * 16 * ROW_BYTES + (lane_part ^ (s << 6)));
  }

  // Operand whose 16-index runs along D (columns 16*x ..) and whose contraction index is the tile ROW (32 of them), in the order in
  // which two 16x16 accumulators, one below the other, hold their rows: element j of lane l is row 16*(j/4) + 4*(l/16) + j%4.
  // Two transposing 8-byte reads, one per 16 rows; in each 16-lane block, lanes 4e..4e+3 read row e.
  __device__ static __forceinline__ int transposed_lane(int lane) {
    const int L = lane & 15;
    return off(4 * (lane >> 4) + (L >> 2), (L & 3) >> 1) + (L & 1) * 8;
  }
  __device__ static __forceinline__ bf16x4 transposed_half(const unsigned char* tile, int lane_part, int x, int part) {
    const unsigned char* p = tile + part * 16 * ROW_BYTES;  // (swz(r + 16) == swz(r))
    return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p + (lane_part ^ (x << 5))));
  }
};

// fp32 merge buffers [64][D] in LDS (partial results of the wavefronts that share output rows).
// A row is D*4 bytes, a multiple of the 256 bytes the 64 banks span, so the 32 lanes of an
// accumulator column (one row each) would all hit the same banks; the 16-byte chunks of a row are
// therefore XOR-ed with the row number (mod 16).  `col` is a multiple of 4.
__device__ __forceinline__ int merge_offset(int row, int col, int row_stride) {
  return row * row_stride + ((((col >> 2) ^ (row & 15)) << 2));
}

// max over both lane halves (lanes l and l^32) with one cross-lane VALU instruction instead of a
// round trip through the LDS permute path
__device__ __forceinline__ float max_across_halves(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

}  // namespace vsa
