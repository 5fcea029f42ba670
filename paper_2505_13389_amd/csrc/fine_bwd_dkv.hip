// The dK/dV kernels of larger launches (the body of a workgroup is in fine_bwd_dkv.h).
#include "fine_bwd_dkv.h"

namespace vsa {

template <int D, int NW, bool SUB, bool NARROW>
__global__ __launch_bounds__(64 * NW, 1) void k_fine_bwd_dkv(int BH, int Nc, int K, float sl2, float scale, const uint4* __restrict__ q,
                                                             const uint4* __restrict__ k, const uint4* __restrict__ v,
                                                             const uint4* __restrict__ dof, const int32_t* __restrict__ col,
                                                             const int32_t* __restrict__ order, int items_per_bh,
                                                             int32_t* __restrict__ split, float* parts, int cap,
                                                             const float* __restrict__ rowd, const float* __restrict__ dkc,
                                                             const float* __restrict__ dvc, const uint64_t* __restrict__ mask,
                                                             uint4* __restrict__ dk, uint4* __restrict__ dv, int m_blocks, int stream,
                                                             RasterMap raster) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[DkvShape<D, NW>::LDS];
  __shared__ int last_run;
  dkv_block<D, NW, SUB, false, NARROW>(smem, &last_run, blockIdx.x, BH, Nc, K, sl2, scale, q, k, v, dof, col, order, items_per_bh, split,
                               parts, cap, rowd, dkc, dvc, mask, dk, dv, m_blocks, stream, raster, SmallCoarseArgs{}, nullptr);
}

hipError_t launch_fine_bwd_dkv(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                               const void* dof, const int32_t* col, const int32_t* order, int32_t* split,
                               float* parts, int cap, const float* rowd, const float* dkc, const float* dvc,
                               const uint64_t* mask, void* dk, void* dv, int m_blocks, int key_cubes_16, const RasterMap& raster,
                               hipStream_t s) {
  const float sl2 = scale * kLog2e;
  const int items = Nc + cap;
  const int stream = (long long)BH * Nc * kTile * d * 2 >= kStreamBytes;
  const unsigned grid = dkv_grid(BH, items, dkv_heads_at_once(Nc, d));
#define VSA_DKV(D_, NW_, SUB_, NARROW_)                                                                                              \
  k_fine_bwd_dkv<D_, NW_, SUB_, NARROW_><<<grid, 64 * NW_, 0, s>>>(BH, Nc, K, sl2, scale, (const uint4*)q, (const uint4*)k, (const uint4*)v, \
                                                          (const uint4*)dof, col, order, items, split, parts, cap, rowd, dkc, dvc, \
                                                          mask, (uint4*)dk, (uint4*)dv, m_blocks, stream, raster)
  const bool narrow = d == 128 && dkv_narrow(BH * Nc, K, key_cubes_16);
  if (key_cubes_16) {  // lists of key cubes of 16 tokens: the pooled terms dkc, dvc are [BH, 4 Nc, d]
    const bool four = BH * Nc <= kDkvFourWaves;  // (lists of blocks: launch_fine_bwd_one)
    if (narrow) VSA_DKV(128, 2, true, true);
    else if (d == 128 && four) VSA_DKV(128, 4, true, false);
    else if (d == 128) VSA_DKV(128, 2, true, false);
    else if (four) VSA_DKV(64, 4, true, false);
    else VSA_DKV(64, 2, true, false);
  } else {
    if (narrow) VSA_DKV(128, 2, false, true);
    else if (d == 128) VSA_DKV(128, 2, false, false);
    else VSA_DKV(64, 2, false, false);
  }
#undef VSA_DKV
  return hipGetLastError();
}

}  // namespace vsa
