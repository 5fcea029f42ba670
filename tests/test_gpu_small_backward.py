"""The backward of small problems in one launch, with the coarse backward inside (up to 64 cubes) and without, on both sides
of the limits, with lists that are split among workgroups (all query cubes select the same few key cubes); the same bits
whatever the order in which the runs of a split list end."""
import numpy as np
import pytest

from helpers import assert_close, bf16_to_np, grid_of, problem_of, tiled_bits, to_dev, widen
from oracle import vsa_oracle as orc
from paper_2505_13389_amd.synth import Workload

pytestmark = pytest.mark.gpu

# grid (cubes), heads: 64 cubes up to and beyond 256 blocks, 65 cubes, partial cubes, one cube
GRIDS = [((16, 16, 16), 4), ((16, 16, 16), 5), ((20, 52, 4), 3), ((7, 22, 30), 2), ((5, 9, 13), 1), ((3, 4, 2), 2)]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("sinks", [False, True])
@pytest.mark.parametrize("grid3,H", GRIDS)
def test_backward_of_small_problems(grid3, H, sinks, d):
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("small_bwd", 1, H, *grid3, d, 1)
    g = grid_of(wl)
    K = min(9, g.Nc)
    wl = Workload("small_bwd", 1, H, *grid3, d, K)
    bits = tiled_bits(wl, seed=g.Nc + H + d, pad_garbage=True)
    x, dev = widen(bits), to_dev(bits)
    rng = np.random.default_rng(g.Nc)
    idx = np.sort(rng.permuted(np.tile(np.arange(g.Nc, dtype=np.int32), (1, H, g.Nc, 1)), axis=-1)[..., :K])
    if sinks:
        idx[...] = np.sort(rng.permutation(g.Nc)[:K])
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], idx, K, real="f32")
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(*a, indices_given=True)
    first = None
    for _ in range(5):
        buf.backward(*a, dev["dout"], workspace_kept=True)
        torch.cuda.synchronize()
        got = {n: getattr(buf, n).clone() for n in ("dq", "dk", "dv")}
        first = first or got
        assert all(torch.equal(got[n], first[n]) for n in got)
    for n in got:
        assert_close(bf16_to_np(got[n]), ref[n], n)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid3,H", GRIDS[:3] + GRIDS[4:5])
def test_coarse_gradients_alone(grid3, H, d):
    """G_f = 0: dQ, dK and dV are the pooled-gradient terms and nothing else."""
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("small_coarse", 1, H, *grid3, d, 2)
    g = grid_of(wl)
    bits = tiled_bits(wl, seed=7 + g.Nc + d)
    bits["gate_f"][...] = 0
    x, dev = widen(bits), to_dev(bits)
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.forward(*a)
    buf.backward(*a, dev["dout"], workspace_kept=True)
    torch.cuda.synchronize()
    idx = buf.block_idx.cpu().numpy()
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], idx, 2, real="f32")
    for n in ("dq", "dk", "dv"):
        got, want = bf16_to_np(getattr(buf, n)).astype(np.float64), ref[n].astype(np.float64)
        # one rounding to bf16 of sums in fp32: 2^-9 an element, 2^-8.5 with the fp32 sums' own error to spare
        assert np.sqrt(((got - want) ** 2).sum()) <= 2.0 ** -8.5 * np.sqrt((want ** 2).sum()), n
