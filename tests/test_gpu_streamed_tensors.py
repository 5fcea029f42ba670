"""The permutation of tensors too large for the caches (40 MiB and more): bit for bit, on a grid no axis of which fits the
cubes, just above and below the limit."""
import numpy as np
import pytest

from oracle import vsa_oracle as orc
from oracle.vsa_oracle import Grid

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H", [(128, 20), (128, 19), (64, 40), (64, 39)])  # 8 x 32 x 32 padded tokens: 40 MiB, 38, 40, 39
@pytest.mark.parametrize("token_major", [False, True])
def test_permute_of_large_tensors(d, H, token_major):
    import torch
    from paper_2505_13389_amd import vsa
    g = Grid(6, 30, 31, 4, 4, 4)
    pb = vsa.Problem(1, H, 6, 30, 31, d, 1)
    Np, _ = vsa.vsa_padded_tokens(pb)
    src = np.random.default_rng(H).integers(0, 1 << 16, (1, H, g.L, d), dtype=np.uint16)
    tiled = orc.tile_u16(g, src)
    raster = np.ascontiguousarray(src.transpose(0, 2, 1, 3)) if token_major else src
    dev = lambda x: torch.from_numpy(x.view(np.int16)).cuda().view(torch.bfloat16)
    bits = lambda x: x.view(torch.int16).cpu().numpy().view(np.uint16)
    out = torch.full((1, H, Np, d), 7.0, dtype=torch.bfloat16, device="cuda")
    vsa.vsa_tile_permute(pb, dev(raster), out, blhd=token_major)
    assert np.array_equal(bits(out), tiled)
    back = torch.full(raster.shape, 7.0, dtype=torch.bfloat16, device="cuda")
    vsa.vsa_tile_permute(pb, out, back, inverse=True, blhd=token_major)
    assert np.array_equal(bits(back), raster)
