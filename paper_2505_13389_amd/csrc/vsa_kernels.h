// Host-side launchers of the gfx950 kernels (one per step of the forward/backward path).
// Each enqueues on `s` and returns hipGetLastError(); none allocates or synchronises.
#pragma once
#include "vsa_common.h"

namespace vsa {

// `raster` (raster_map or tiled_map): where `out`, `dout` and the gradients lie
constexpr int kPermuteTensors = 8;  // of one launch, by value
struct PermuteTensors {
  const void* src[kPermuteTensors];
  void* dst[kPermuteTensors];
};
hipError_t launch_tile_permute(const Geo& g, int BH, int H_blhd, int d, int count, const PermuteTensors& tensors, bool inverse,
                               hipStream_t s);
hipError_t launch_mfma_rate(const void* operands, float* sink, int workgroups, int iters, hipStream_t s);
// tensors = 3: Q, K, V pooled per cube; 1: Q only (with launch_pool_keys16 for K and V)
hipError_t launch_pool(const Geo& g, int BH, int d, uint64_t* mask, const void* q, const void* k, const void* v,
                       float* qc, float* kc, float* vc, int tensors, hipStream_t s);
// key cubes of 16 tokens: kc, vc [BH, 4 Nc, d], kcnt [4 Nc] valid tokens per key cube (needs `mask`)
hipError_t launch_pool_keys16(int BH, int Nc, int d, const uint64_t* mask, int32_t* kcnt, const void* k, const void* v,
                              float* kc, float* vc, hipStream_t s);
// Nq query cubes, Nk key cubes; kcnt (or NULL): valid tokens per key cube, 0 = dead
hipError_t launch_coarse(int BH, int Nq, int Nk, int d, int K, float scale, const float* qc, const float* kc,
                         const float* vc, float* sc, float* oc, float* lse_c, int32_t* idx, int emit_idx, int fused,
                         const int32_t* kcnt, hipStream_t s);
hipError_t launch_fine_fwd_short(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                                 const void* gate_c, const void* gate_f, const int32_t* idx, const float* oc,
                                 const uint64_t* mask, void* out, void* out_fine, float* lse_f, int H, int out_token_major,
                                 int m_blocks, int key_cubes_16, const RasterMap& raster, hipStream_t s);
// Which instance of a fine kernel a launch takes: wavefronts per workgroup (0: the forward's kernel for short lists) and how many
// workgroups take two blocks.  `Nc`: blocks; `coarse`: the coarse stage is done on the way.
struct FineRoute {
  int waves;
  unsigned pairs;
};
FineRoute fine_fwd_route(int BH, int Nc, int d, int K, int key_cubes_16, bool coarse);
FineRoute fine_bwd_dq_route(int BH, int Nc, int d);
// What the forward of a short sequence forms its coarse stage from, row by row in the fine kernel, and where it leaves it.
struct SmallForwardArgs {
  const float *qc, *kc, *vc;
  float *oc, *lse_c;
  int32_t* idx;
  float scale;
};
bool fine_fwd_with_coarse(int BH, int Nc, int d, int m_blocks);
// gang_scratch: BH*Nc/32 + 24 counters' worth of memory that nothing else uses during the launch.  `coarse` (or NULL): the coarse
// stage is done on the way, idx and oc are its results.
hipError_t launch_fine_fwd(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                           const void* gate_c, const void* gate_f, const int32_t* idx, const float* oc,
                           const uint64_t* mask, void* out, void* out_fine, float* lse_f, int H, int out_token_major,
                           int m_blocks, int key_cubes_16, unsigned* gang_scratch, const SmallForwardArgs* coarse, const RasterMap& raster, hipStream_t s);
// lists of cubes -> lists of 64-row blocks, for cubes of m blocks: every block of query cube c gets
// the m blocks of each of the cube's K key cubes, ascending ([BH,Nc,K] -> [BH,Nc*m,K*m])
// mismatched granularity: top-K on the coarse map pooled over (1,2,2) cubes, and its lists of tiles
// turned into lists of cubes for every query cube ([BH,Ns,K] -> [BH,Nc,4K])
hipError_t launch_pooled_select(int BH, int Nt, int Nh, int Nw, int K, const float* P, float* ps, int32_t* tile_idx,
                                hipStream_t s);
hipError_t launch_expand_tiles(int BH, int Nt, int Nh, int Nw, int K, const int32_t* tile_idx, int32_t* idx_blocks,
                               hipStream_t s);
hipError_t launch_expand_lists(int BH, int Nc, int K, int m, const int32_t* idx, int32_t* idx_blocks, hipStream_t s);

// backward
// The transposed block map of lists of K blocks (or, with key cubes of 16 tokens, key cubes) per query block:
// Nc blocks per (b, h); see split_plan for seg and cap.
struct MapArgs {
  int Nc, K, seg, cap;
  const int32_t* idx;
  int32_t *row_ptr, *col, *order, *split;
};
// whether launch_bwd_pre transposes the map on the side (`map` given) or launch_transpose_map has to
bool map_with_bwd_pre(int Nc, int key_cubes_16);
hipError_t launch_bwd_pre(int BH, int Nc, int m_blocks, int d, const uint64_t* mask, const void* dout, const void* gate_c,
                          const void* gate_f, const void* out_fine, const float* oc, void* dgate_c, void* dgate_f,
                          void* dof, float* rowd, float scale, float* doc, float* dot, const float* lse_f, int H,
                          int dout_token_major, const MapArgs* map, const RasterMap& raster, hipStream_t s);
hipError_t launch_coarse_bwd(int BH, int Nq, int Nk, int d, float scale, const float* qc, const float* kc,
                             const float* vc, const float* lse_c, const float* doc, const float* dot, float* ac,
                             float* dsc, float* dqc, float* dkc, float* dvc, const int32_t* kcnt, hipStream_t s);
hipError_t launch_transpose_map(int BH, const MapArgs& a, uint32_t* bits, int key_cubes_16, hipStream_t s);
hipError_t launch_fine_bwd_dq(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                              const void* dof, const int32_t* idx, const float* rowd,
                              const float* dqc, const uint64_t* mask, void* dq, int m_blocks, int key_cubes_16,
                              const RasterMap& raster, hipStream_t s);
hipError_t launch_fine_bwd_dkv(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                               const void* dof, const int32_t* col, const int32_t* order, int32_t* split,
                               float* parts, int cap, const float* rowd, const float* dkc, const float* dvc,
                               const uint64_t* mask, void* dk, void* dv, int m_blocks, int key_cubes_16, const RasterMap& raster,
                               hipStream_t s);
// Up to this many blocks dK/dV and, at d = 128, dQ take four wavefronts per workgroup: the launch does not fill the 512
// places of two-wavefront workgroups, and half as long a list walk counts (64 blocks, d = 64, top-8: 10.7 against 13.7 us).
constexpr int kDkvFourWaves = 256;
// Both passes of a small problem in one launch (BH*Nc up to kDkvFourWaves blocks, lists of blocks).  `coarse` (cubes of one block,
// Nc up to kSmallCubes): the coarse backward too; qc .. dot are read then, dqc, dkc, dvc are not.
bool fine_bwd_in_one(int BH, int Nc, int key_cubes_16);
bool fine_bwd_with_coarse(int Nc, int m_blocks);
hipError_t launch_fine_bwd_one(int BH, int Nc, int d, int K, float scale, const void* q, const void* k, const void* v,
                               const void* dof, const int32_t* idx, const int32_t* col, const int32_t* order, int32_t* split,
                               float* parts, int cap, const float* rowd, const float* dqc, const float* dkc, const float* dvc,
                               const uint64_t* mask, void* dq, void* dk, void* dv, int m_blocks, const float* qc, const float* kc,
                               const float* vc, const float* doc, const float* lse_c, const float* dot, const RasterMap& raster, hipStream_t s);

}  // namespace vsa
