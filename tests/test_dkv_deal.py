"""Host replay of how the dK/dV launch deals heads to XCDs, on both sides of the head size from which four of them are in
flight instead of eight, for every remainder of heads: each item of each head belongs to exactly one workgroup."""
import numpy as np
import pytest


@pytest.mark.parametrize("grid3,d", [((20, 48, 60), 128), ((21, 48, 64), 128), ((28, 64, 64), 64), ((32, 64, 64), 64)])  # 900, 1152, 1792, 2048 blocks
@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 7, 8, 11])
def test_every_item_is_dealt_once(grid3, d, H):
    from paper_2505_13389_amd import vsa
    pb = vsa.Problem(1, H, *grid3, d, 1)
    _, Nc = vsa.vsa_padded_tokens(pb)
    idx = np.random.default_rng(H).integers(0, Nc, (1, H, Nc, 1), dtype=np.int32)
    rc, rep = vsa.vsa_host_replay_lists(pb, idx)
    assert rc == 0 and rep["violations"] == 0, rep
