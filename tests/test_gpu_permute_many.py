"""Several tensors in one permutation launch: each bit for bit what the oracle makes of it, from one tensor to the most a call
takes, below and above the size that goes past the caches, on grids no axis of which fits the cubes."""
import numpy as np
import pytest

from oracle import vsa_oracle as orc
from oracle.vsa_oracle import Grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,H,grid,d,n", [(1, 1, (3, 5, 6), 64, 1), (2, 3, (5, 7, 9), 128, 5), (1, 2, (5, 7, 9), 64, 8),
                                          (1, 20, (6, 30, 31), 128, 2)])
@pytest.mark.parametrize("token_major", [False, True])
def test_every_tensor_of_a_launch(B, H, grid, d, n, token_major):
    import torch
    from paper_2505_13389_amd import vsa
    g = Grid(*grid, 4, 4, 4)
    pb = vsa.Problem(B, H, *grid, d, 1)
    Np, _ = vsa.vsa_padded_tokens(pb)
    src = [np.random.default_rng(i).integers(0, 1 << 16, (B, H, g.L, d), dtype=np.uint16) for i in range(n)]
    raster = [np.ascontiguousarray(x.transpose(0, 2, 1, 3)) if token_major else x for x in src]
    dev = [torch.from_numpy(x.view(np.int16)).cuda().view(torch.bfloat16) for x in raster]
    bits = lambda x: x.view(torch.int16).cpu().numpy().view(np.uint16)
    out = [torch.full((B, H, Np, d), 7.0, dtype=torch.bfloat16, device="cuda") for _ in range(n)]
    vsa.vsa_tile_permute_many(pb, dev, out, blhd=token_major)
    back = [torch.full_like(x, 7.0) for x in dev]
    vsa.vsa_tile_permute_many(pb, out, back, inverse=True, blhd=token_major)
    for i in range(n):
        assert np.array_equal(bits(out[i]), orc.tile_u16(g, src[i]))
        assert np.array_equal(bits(back[i]), raster[i])
