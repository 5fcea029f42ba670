"""VSA_FLAG_RASTER_IO: the forward's output and the backward's dout and gradients in raster order are, bit for bit, the tiled
ones permuted -- through every kernel that writes them, with partial cubes, larger cubes, both kinds of key lists, two samples
and lists that are split among workgroups."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# B, H, grid, d, top-K, cube, flags, all lists alike
PLAIN, POOLED, KEY16 = 0, 32, 128
CASES = [
    (2, 2, (7, 14, 30), 64, 5, (4, 4, 4), PLAIN, False),     # small, coarse stage inside
    (1, 2, (7, 14, 30), 128, 9, (4, 4, 4), PLAIN, True),     # split lists
    (1, 3, (7, 22, 30), 128, 20, (4, 4, 4), PLAIN, False),   # 288 blocks: two wavefronts share a block
    (1, 7, (18, 74, 4), 128, 20, (4, 4, 4), PLAIN, False),   # 665 blocks: a wavefront each
    (1, 12, (7, 22, 30), 128, 6, (4, 4, 4), PLAIN, True),    # 1152 blocks: short lists, split
    (1, 12, (7, 22, 30), 64, 20, (4, 4, 4), PLAIN, False),
    (2, 2, (9, 13, 27), 128, 3, (4, 4, 8), PLAIN, False),
    (1, 3, (5, 17, 19), 64, 2, (4, 8, 8), PLAIN, False),
    (1, 2, (7, 14, 30), 128, 3, (4, 4, 4), POOLED, False),
    (1, 2, (7, 14, 30), 128, 21, (4, 4, 4), KEY16, False),
    (1, 9, (7, 14, 30), 64, 21, (4, 4, 4), KEY16, False),
]


@pytest.mark.parametrize("with_gate_f", [True, False])
@pytest.mark.parametrize("B,H,grid3,d,K,cube,flags,alike", CASES)
def test_raster_tensors_are_the_tiled_ones_permuted(B, H, grid3, d, K, cube, flags, alike, with_gate_f):
    import torch
    from paper_2505_13389_amd import vsa
    assert (POOLED, KEY16) == (vsa.VSA_FLAG_SELECT_POOLED_2X2, vsa.VSA_FLAG_KEY_CUBES_16)
    if flags == POOLED:
        grid3 = (7, 16, 32)
    pb = vsa.Problem(B, H, *grid3, d, K, cube, flags=flags)
    L = grid3[0] * grid3[1] * grid3[2]
    g = torch.Generator(device="cuda")
    g.manual_seed(K + H)

    def raster():
        return torch.randn((B, L, H, d), generator=g, device="cuda").bfloat16()

    tiled_buf = vsa.Buffers(pb, with_gate_f=with_gate_f)

    def tile(x):
        y = torch.empty((B, H, tiled_buf.Np, d), dtype=torch.bfloat16, device="cuda")
        vsa.vsa_tile_permute(pb, x, y, blhd=True)
        return y

    def untile(x):
        y = torch.empty((B, L, H, d), dtype=torch.bfloat16, device="cuda")
        vsa.vsa_tile_permute(pb, x, y, inverse=True, blhd=True)
        return y

    a = [tile(raster()) for _ in range(4)] + [tile(raster()) if with_gate_f else None]
    dout = raster()
    given = alike
    if alike:
        tiled_buf.block_idx[...] = torch.arange(K, dtype=torch.int32, device="cuda")
    tiled_buf.forward(*a, indices_given=given)
    tiled_buf.backward(*a, tile(dout), workspace_kept=True)

    rb = vsa.Problem(B, H, *grid3, d, K, cube, flags=flags | vsa.VSA_FLAG_RASTER_IO)
    buf = vsa.Buffers(rb, with_gate_f=with_gate_f)
    names = ["dq", "dk", "dv", "dgate_c"] + (["dgate_f"] if with_gate_f else [])
    for n in ["out"] + names:
        setattr(buf, n, torch.full((B, L, H, d), float("nan"), dtype=torch.bfloat16, device="cuda"))
    if alike:
        buf.block_idx.copy_(tiled_buf.block_idx)
    buf.forward(*a, indices_given=given)
    buf.backward(*a, dout, workspace_kept=True)
    torch.cuda.synchronize()
    assert torch.equal(buf.block_idx, tiled_buf.block_idx) and torch.equal(buf.out_fine, tiled_buf.out_fine)
    assert torch.equal(buf.lse_fine, tiled_buf.lse_fine)
    for n in ["out"] + names:
        assert torch.equal(getattr(buf, n), untile(getattr(tiled_buf, n))), n


@pytest.mark.parametrize("order", ["contiguous", "heads first", "expanded"])
def test_op_takes_gradients_and_inputs_of_any_strides(order):
    """q and dout that are views: the same results as their contiguous copies."""
    import torch
    from paper_2505_13389_amd.autograd import video_sparse_attention
    B, H, grid3, d = 2, 3, (7, 14, 30), 64
    L = grid3[0] * grid3[1] * grid3[2]
    torch.manual_seed(3)
    mk = lambda: torch.randn((B, L, H, d), device="cuda").bfloat16()
    q, k, v, gc, do = (mk() for _ in range(5))
    if order == "heads first":
        q, do = (x.transpose(1, 2).contiguous().transpose(1, 2) for x in (q, do))
    if order == "expanded":
        do = do[:, :1, :1].expand(B, L, H, d)
    def run(q, do):
        leaves = [x.detach().requires_grad_(True) for x in (q, k, v, gc)]
        out = video_sparse_attention(*leaves, grid=grid3, topk=6)
        return [out] + list(torch.autograd.grad(out, leaves, do))
    for got, want in zip(run(q, do), run(q.contiguous(), do.contiguous())):
        assert got.shape == want.shape and torch.equal(got, want)
