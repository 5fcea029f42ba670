"""Video Sparse Attention as a differentiable PyTorch op (App. B: tile -> sparse attention -> untile).

Marshalling only: the token permutation, the forward and the backward all run in libvsa.so's
kernels; torch supplies device memory, the current stream and the autograd graph.  Tensors are in
the layout a video DiT holds them in, token-major raster order: bf16 [B, L, H, d] with
L = T*Hh*W and n = t*Hh*W + h*W + w (Sec. 2.1).

    out = video_sparse_attention(q, k, v, gate_c, gate_f, grid=(T, Hh, W), topk=K)

gate_f may be None (a fine gate of ones, Sec. 2.3).  No gradient flows through the top-K selection.
A model that keeps its activations in tiled order across layers (App. B caption) should call the
vsa_* entry points directly and skip the permutations.
"""
import torch

from . import vsa


class _VideoSparseAttention(torch.autograd.Function):
    @staticmethod
    def forward(ctx, q, k, v, gate_c, gate_f, grid, topk, cube, softmax_scale, flags):
        B, L, H, d = q.shape
        T, Hh, W = grid
        assert L == T * Hh * W, "q is [B, T*Hh*W, H, d]"
        pb = vsa.Problem(B, H, T, Hh, W, d, topk, tuple(cube), float(softmax_scale or 0.0), int(flags))
        Np, Nc = vsa.vsa_padded_tokens(pb)
        shape = (B, H, Np, d)
        bf = dict(dtype=torch.bfloat16, device=q.device)
        f32 = dict(dtype=torch.float32, device=q.device)

        raster = [x.contiguous() for x in (q, k, v, gate_c, gate_f) if x is not None]
        tiled = [torch.empty(shape, **bf) for _ in raster]
        vsa.vsa_tile_permute_many(pb, raster, tiled, inverse=False, blhd=True)
        tq, tk, tv, tgc, tgf = tiled if gate_f is not None else tiled + [None]
        # the attention writes raster tokens and, in the backward, reads and writes them: no permutation on that side
        pb = vsa.Problem(B, H, T, Hh, W, d, topk, tuple(cube), float(softmax_scale or 0.0),
                         int(flags) | vsa.VSA_FLAG_RASTER_IO)
        out = torch.empty_like(q, memory_format=torch.contiguous_format)
        rows = Nc // 4 if pb.flags & vsa.VSA_FLAG_SELECT_POOLED_2X2 else Nc
        idx = torch.empty((B, H, rows, pb.topk), dtype=torch.int32, device=q.device)
        out_fine, lse_fine = torch.empty(shape, **bf), torch.empty((B, H, Np), **f32)
        out_coarse, lse_coarse = torch.empty((B, H, Nc, d), **f32), torch.empty((B, H, Nc), **f32)
        workspace = torch.empty(vsa.vsa_workspace_bytes(pb, False), dtype=torch.uint8, device=q.device)
        vsa.vsa_forward(pb, tq, tk, tv, tgc, tgf, out, idx, out_fine, lse_fine, out_coarse, lse_coarse, workspace)
        ctx.pb, ctx.kept = pb, (idx, out_fine, lse_fine, out_coarse, lse_coarse)
        ctx.save_for_backward(tq, tk, tv, tgc, tgf)
        return out

    @staticmethod
    def backward(ctx, dout):
        pb = ctx.pb
        tq, tk, tv, tgc, tgf = ctx.saved_tensors
        idx, out_fine, lse_fine, out_coarse, lse_coarse = ctx.kept
        dout = dout.contiguous()
        dq, dk, dv, dgc = (torch.empty_like(dout) for _ in range(4))
        dgf = None if tgf is None else torch.empty_like(dout)
        workspace = torch.empty(vsa.vsa_workspace_bytes(pb, True), dtype=torch.uint8, device=dout.device)
        vsa.vsa_backward(pb, tq, tk, tv, tgc, tgf, dout, idx, out_fine, lse_fine, out_coarse, lse_coarse, dq, dk, dv, dgc,
                         dgf, workspace)
        return dq, dk, dv, dgc, dgf, None, None, None, None, None


def video_sparse_attention(q, k, v, gate_c, gate_f=None, *, grid, topk, cube=(4, 4, 4), softmax_scale=None, flags=0):
    """q, k, v, gate_c, gate_f (or None): bf16 [B, T*Hh*W, H, d] on the GPU; returns bf16 of the same shape."""
    return _VideoSparseAttention.apply(q, k, v, gate_c, gate_f, tuple(grid), int(topk), tuple(cube), softmax_scale, flags)
