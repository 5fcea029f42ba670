"""dK/dV pass: transposed lists of every length from none to all query blocks (a wavefront's share of a list is
then 0, 1, 2, ... units), on both sides of the workgroup-size rule and for head counts that the XCD mapping
deals as whole, half, quarter and eighth heads."""
import numpy as np
import pytest

from helpers import assert_close, bf16_to_np, grid_of, problem_of, tiled_bits, to_dev, widen
from oracle import vsa_oracle as orc
from paper_2505_13389_amd.synth import Workload

pytestmark = pytest.mark.gpu


def lists_of_spread_degrees(rng, H, Nc, K):
    """Key block j is taken with a weight that falls by a factor of about 100 over the blocks; the last two never."""
    w = np.exp(-4.6 * np.arange(Nc) / Nc)
    w[-2:] = 0
    out = np.zeros((1, H, Nc, K), np.int32)
    for h in range(H):
        p = w[rng.permutation(Nc)]
        p = p / p.sum()
        for c in range(Nc):
            out[0, h, c] = np.sort(rng.choice(Nc, size=K, replace=False, p=p))
    return out


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H", [1, 2, 3, 7, 9])  # 96 blocks: up to 2 heads four wavefronts per workgroup, then two
def test_dkv_lists_of_every_length(d, H):
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("dkv_units", 1, H, 7, 22, 30, d, 6)
    bits = tiled_bits(wl, seed=70 + d + H, pad_garbage=True)
    x, dev, g = widen(bits), to_dev(bits), grid_of(wl)
    idx = lists_of_spread_degrees(np.random.default_rng(d + H), H, g.Nc, wl.topk)
    deg = np.bincount(idx[0, 0].ravel(), minlength=g.Nc)
    assert deg.min() == 0 and {1, 2, 3, 4} <= set(deg) and deg.max() > 16
    fwd = orc.forward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], wl.topk, real="f32", block_idx=idx)
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], idx, wl.topk, real="f32")
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(*a, indices_given=True)
    buf.backward(*a, dev["dout"], workspace_kept=True)
    torch.cuda.synchronize()
    assert_close(bf16_to_np(buf.out), fwd["out"], "out")
    for n in ("dq", "dk", "dv"):
        assert_close(bf16_to_np(getattr(buf, n)), ref[n], n)


def test_four_heads_at_a_time(d=128, H=5, K=3):
    """960 blocks, d = 128: from this head size on four heads are in flight, not eight.  Two heads of the group of four and the one
    left over; lists of three, whose transposed lists are short and sometimes empty, and in the last head three sinks, split
    among workgroups."""
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("dkv_four", 1, H, 20, 48, 64, d, K)
    bits = tiled_bits(wl, seed=77)
    x, dev, g = widen(bits), to_dev(bits), grid_of(wl)
    assert g.Nc * 64 * d * 4 == 30 << 20
    rng = np.random.default_rng(4)
    idx = np.sort(np.stack([rng.permutation(g.Nc)[:K] for _ in range(H * g.Nc)]).reshape(1, H, g.Nc, K).astype(np.int32), axis=-1)
    idx[0, H - 1] = np.sort(rng.permutation(g.Nc)[:K])
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(*a, indices_given=True)
    buf.backward(*a, dev["dout"], workspace_kept=True)
    torch.cuda.synchronize()
    heads = [0, 3, H - 1]
    x = {n: np.ascontiguousarray(v[:, heads]) for n, v in x.items()}
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], np.ascontiguousarray(idx[:, heads]), K, real="f32")
    for n in ("dq", "dk", "dv"):
        for i, h in enumerate(heads):
            assert_close(bf16_to_np(getattr(buf, n)[:, h]), ref[n][:, i], f"{n} of head {h}")


# d = 128, both sides of the lines between the 32x32x16 and the 16x16x32 matrix instruction: one launch with dQ (up to 256 blocks, with the coarse
# backward up to 64 cubes a head), two launches.  Heads, grid of a head (tokens), entries.
@pytest.mark.parametrize("H,grid3,K", [(1, (16, 16, 16), 25), (1, (16, 16, 16), 62), (3, (8, 16, 16), 16), (3, (8, 16, 16), 17), (2, (14, 15, 16), 12),
                                       (2, (14, 15, 16), 13), (3, (16, 16, 16), 8), (3, (16, 16, 16), 9), (1, (7, 22, 30), 16), (1, (7, 22, 30), 17),
                                       (2, (7, 22, 30), 8), (2, (7, 22, 30), 9), (3, (7, 22, 30), 8), (3, (7, 22, 30), 9),
                                       (4, (7, 22, 30), 8), (4, (7, 22, 30), 9), (7, (16, 16, 16), 8)])
def test_either_matrix_instruction(H, grid3, K, d=128):
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("dkv_instruction", 1, H, *grid3, d, K)
    bits = tiled_bits(wl, seed=H + K, pad_garbage=True)
    x, dev, g = widen(bits), to_dev(bits), grid_of(wl)
    idx = lists_of_spread_degrees(np.random.default_rng(H + K), H, g.Nc, K)
    ref = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], idx, K, real="f32")
    buf = vsa.Buffers(problem_of(wl))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(*a, indices_given=True)
    buf.backward(*a, dev["dout"], workspace_kept=True)
    torch.cuda.synchronize()
    for n in ("dq", "dk", "dv"):
        assert_close(bf16_to_np(getattr(buf, n)), ref[n], n)
