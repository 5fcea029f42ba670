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
