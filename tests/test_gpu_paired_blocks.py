"""Forward and dQ where a workgroup takes two query blocks, one per wavefront: odd numbers of blocks, launches whose last
blocks are shared by two wavefronts, short walks, lists of several chunks, lists of all blocks, and V of any magnitude."""
import numpy as np
import pytest

from helpers import assert_close, bf16_to_np, grid_of, problem_of, tiled_bits, to_dev, widen
from oracle import vsa_oracle as orc
from paper_2505_13389_amd import synth
from paper_2505_13389_amd.synth import Workload

pytestmark = pytest.mark.gpu

# d, heads of 95 query blocks, list length, what the forward (None: not a matter of pairs) and dQ do with the blocks
ALL, SOME, NONE = "all paired", "full generations paired, the rest shared", "all shared"
CASES = ([(128, 7, K, ALL, ALL) for K in (1, 2, 3, 17, 18, 65, 95)] +  # (the last workgroup has one block)
         [(128, 11, 1, None, SOME), (128, 11, 50, SOME, SOME)] + [(128, 15, K, SOME, SOME) for K in (1, 2, 5)] +
         [(64, 17, K, None, ALL) for K in (1, 2, 9)] + [(64, 22, 3, None, SOME), (64, 25, 3, None, NONE)])


def assert_pairs(wl, forward, dq):
    from paper_2505_13389_amd import vsa
    blocks = wl.H * grid_of(wl).Nc
    route = vsa.vsa_host_routes(problem_of(wl), indices_given=True)
    of = lambda pairs: ALL if 2 * pairs >= blocks else SOME if pairs else NONE
    assert route["dq_waves"] == 2 and of(route["dq_pairs"]) == dq, route
    assert forward is None or (route["fwd_waves"] == 2 and of(route["fwd_pairs"]) == forward), route


def check_heads(wl, bits, idx, heads):
    import torch
    from paper_2505_13389_amd import vsa
    dev, g = to_dev(bits), grid_of(wl)
    buf = vsa.Buffers(problem_of(wl))
    buf.block_idx.copy_(torch.from_numpy(idx))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.forward(*a, indices_given=True)
    buf.backward(*a, dev["dout"], workspace_kept=True)
    torch.cuda.synchronize()
    x = {n: np.ascontiguousarray(v[:, heads]) for n, v in widen(bits).items()}
    lists = np.ascontiguousarray(idx[:, heads])
    ref = orc.forward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], wl.topk, real="f32", block_idx=lists)
    grad = orc.backward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], x["dout"], lists, wl.topk, real="f32")
    for n in ("out", "out_fine"):
        assert_close(bf16_to_np(getattr(buf, n))[:, heads], ref[n], n)
    assert np.abs(buf.lse_fine.cpu().numpy()[:, heads] - ref["lse_fine"]).max() < 1e-3  # (as in test_gpu_fwd_units.py)
    for n in ("dq", "dk", "dv"):
        assert_close(bf16_to_np(getattr(buf, n))[:, heads], grad[n], n)


@pytest.mark.parametrize("d,H,K,forward,dq", CASES)
def test_blocks_of_their_own(d, H, K, forward, dq):
    wl = Workload("paired", 1, H, 18, 74, 4, d, K)
    g = grid_of(wl)
    assert_pairs(wl, forward, dq)
    rng = np.random.default_rng(K)
    idx = np.sort(rng.permuted(np.tile(np.arange(g.Nc, dtype=np.int32), (1, H, g.Nc, 1)), axis=-1)[..., :K])
    check_heads(wl, tiled_bits(wl, seed=500 + K + H, pad_garbage=True), idx, [0, H // 2, H - 2, H - 1])


@pytest.mark.parametrize("scale", [2.0 ** 60, 2.0 ** 110])
def test_values_of_any_magnitude_per_wavefront(scale, d=128, H=7, K=40):
    """Rising logits (see test_gpu_fwd_units.py) in every second block's wavefront alone: one of a workgroup's two does its
    block again while the other is done."""
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("paired_big", 1, H, 18, 74, 4, d, K)
    g = grid_of(wl)
    assert_pairs(wl, ALL, ALL)
    bits = tiled_bits(wl, seed=9, pad_garbage=True)
    rng = np.random.default_rng(4)
    ramp = np.linspace(-20.0, 20.0, g.Nc)
    u = rng.choice([-1.0, 1.0], size=d)
    k = np.repeat(ramp, 64)[None, None, :, None] * u / np.sqrt(d) + 0.1 * rng.standard_normal((1, H, g.Np, d))
    q = u * (np.arange(g.Np) // 64 % 2)[None, None, :, None] + 0.1 * rng.standard_normal((1, H, g.Np, d))
    bits["q"], bits["k"] = synth.f32_to_bf16_bits(q.astype(np.float32)), synth.f32_to_bf16_bits(k.astype(np.float32))
    x = widen(bits)
    idx = np.sort(rng.permuted(np.tile(np.arange(g.Nc, dtype=np.int32), (1, H, g.Nc, 1)), axis=-1)[..., :K])
    big = {**x, "v": x["v"] * np.float32(scale)}
    dev = to_dev({**bits, "v": synth.f32_to_bf16_bits(big["v"])})
    buf = vsa.Buffers(problem_of(wl))
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"], indices_given=True)
    torch.cuda.synchronize()
    ref = orc.forward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], K, real="f32", block_idx=idx)
    got = bf16_to_np(buf.out_fine).astype(np.float64) / scale  # (a power of two: exact)
    assert_close(got, ref["out_fine"], "out_fine")
