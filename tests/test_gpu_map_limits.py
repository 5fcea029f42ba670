"""The transposed block map on both sides of the limit below which it shares the preprocess launch (384 blocks), with
lists that name a few key blocks very often (split lists) and some never; and the coarse backward by itself, in one
launch (one chunk of 256 cubes, two and three) and in three."""
import numpy as np
import pytest

from helpers import assert_close, bf16_to_np, grid_of, problem_of, tiled_bits, to_dev, widen
from oracle import vsa_oracle as orc
from paper_2505_13389_amd.synth import Workload
from test_gpu_dkv_units import lists_of_spread_degrees

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grid,blocks,d", [((4, 4, 7), 2, 64), ((4, 4, 7), 2, 128), ((23, 32, 30), 384, 64),
                                           ((23, 32, 30), 384, 128), ((20, 27, 44), 385, 64)])
def test_map_on_both_sides_of_the_limit(grid, blocks, d):
    import torch
    from paper_2505_13389_amd import vsa
    K = min(5, blocks)
    wl = Workload("map_limit", 1, 3, *grid, d, K)  # an odd number of cubes in all: the last workgroup has a spare half
    g = grid_of(wl)
    assert g.Nc == blocks
    bits = tiled_bits(wl, seed=blocks, pad_garbage=True)
    x, dev = widen(bits), to_dev(bits)
    if blocks > 8:
        idx = lists_of_spread_degrees(np.random.default_rng(blocks), 3, g.Nc, K)
    else:
        idx = np.tile(np.arange(K, dtype=np.int32), (1, 3, g.Nc, 1))
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], idx, K, real="f32")
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(*a, indices_given=True)
    buf.workspace[vsa.vsa_workspace_bytes(problem_of(wl), False):].fill_(0xFF)  # nothing of the backward's part is kept
    buf.backward(*a, dev["dout"])
    torch.cuda.synchronize()
    for n in ("dq", "dk", "dv", "dgate_c", "dgate_f"):
        assert_close(bf16_to_np(getattr(buf, n)), ref[n], n)


@pytest.mark.parametrize("grid,blocks", [((4, 4, 7), 2), ((20, 12, 68), 255), ((4, 4, 1028), 257), ((23, 32, 30), 384),
                                         ((20, 27, 44), 385), ((21, 30, 52), 624)])
@pytest.mark.parametrize("d,H", [(64, 3), (64, 4), (128, 1), (128, 2)])  # 624 blocks: one launch, three, one, three
@pytest.mark.parametrize("planted", [False, True])
def test_coarse_gradients_alone(grid, blocks, d, H, planted):
    """Gate G_f = 0: nothing comes through the fine stage, dq, dk and dv are the pooled coarse gradients.  They are fp32 sums
    rounded to bf16 once, so off by at most 2^-9 of themselves and what the sums lose (1e-4 of the whole)."""
    import torch
    from paper_2505_13389_amd import vsa
    K = min(5, blocks)
    wl = Workload("coarse_alone", 1, H, *grid, d, K, planted=planted)
    g = grid_of(wl)
    assert g.Nc == blocks
    bits = tiled_bits(wl, seed=blocks + d, pad_garbage=True)
    bits["gate_f"][:] = 0
    x, dev = widen(bits), to_dev(bits)
    idx = np.tile(np.arange(K, dtype=np.int32), (1, H, g.Nc, 1))
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], idx, K, real="f64")
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(*a, indices_given=True)
    buf.backward(*a, dev["dout"])
    torch.cuda.synchronize()
    for n in ("dq", "dk", "dv"):
        assert np.abs(ref[n]).max() > 0
        assert_close(bf16_to_np(getattr(buf, n)), ref[n], n, rel_l2=2.0 ** -9 + 1e-4)


@pytest.mark.parametrize("d", [64, 128])
def test_an_infinite_gradient_of_the_last_cube(d):
    """175 cubes, not a multiple of 16: an infinite dO in the last one makes that column of dv infinite, not NaN."""
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("coarse_inf", 1, 1, 20, 20, 28, d, 8)
    g = grid_of(wl)
    assert g.Nc == 175
    dev = to_dev(tiled_bits(wl, seed=d))
    dev["dout"][:, :, 64 * 174, 3] = float("inf")
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"].abs() + 0.1, dev["gate_f"].abs() + 0.1)
    buf.forward(*a)
    buf.backward(*a, dev["dout"])
    torch.cuda.synchronize()
    dv = bf16_to_np(buf.dv)
    assert (dv[..., 3] == np.inf).all()
    assert np.isfinite(np.delete(dv, 3, axis=-1)).all()
