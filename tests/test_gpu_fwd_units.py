"""Forward: list walks of every length around the unrolled loop, on both sides of the rules that choose the kernel, and the
reference of the online softmax: first units without a valid key, and logits that outgrow the reference again and
again along the walk."""
import numpy as np
import pytest

from helpers import assert_close, bf16_to_np, grid_of, problem_of, tiled_bits, to_dev, widen
from oracle import vsa_oracle as orc
from paper_2505_13389_amd import synth
from paper_2505_13389_amd.synth import Workload

pytestmark = pytest.mark.gpu


SHORT, TWO, FOUR = 0, 2, 4  # the kernel for short lists; the general one, by wavefronts per workgroup


def assert_kernel(wl, waves, paired=False):
    from paper_2505_13389_amd import vsa
    route = vsa.vsa_host_routes(problem_of(wl), indices_given=True)
    assert (route["fwd_waves"], route["fwd_pairs"] > 0) == (waves, paired), route


def run_and_check(wl, bits, idx, heads=None):
    """`heads`: those compared with the oracle (all)."""
    import torch
    from paper_2505_13389_amd import vsa
    dev, g, heads = to_dev(bits), grid_of(wl), list(range(wl.H)) if heads is None else heads
    x = {n: np.ascontiguousarray(v[:, heads]) for n, v in widen(bits).items()}
    ref = orc.forward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], wl.topk, real="f32",
                      block_idx=np.ascontiguousarray(idx[:, heads]))
    buf = vsa.Buffers(problem_of(wl))
    buf.block_idx.copy_(torch.from_numpy(idx))
    buf.forward(dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"], indices_given=True)
    torch.cuda.synchronize()
    assert_close(bf16_to_np(buf.out)[:, heads], ref["out"], "out")
    assert_close(bf16_to_np(buf.out_fine)[:, heads], ref["out_fine"], "out_fine")
    # fp32 sums of up to a few thousand terms, logits of magnitude up to 500 (log2 units): 1e-3 is 8 spacings there
    assert np.abs(buf.lse_fine.cpu().numpy()[:, heads] - ref["lse_fine"]).max() < 1e-3


def random_lists(wl, g, seed):
    rng = np.random.default_rng(seed)
    return np.sort(rng.permuted(np.tile(np.arange(g.Nc, dtype=np.int32), (1, wl.H, g.Nc, 1)), axis=-1)[..., :wl.topk])


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H", [1, 3])  # 96 query blocks each: four wavefronts (d = 128, 3 heads: two; few tiles: short lists)
@pytest.mark.parametrize("K", [1, 2, 3, 4, 5, 6, 7, 8, 65])
def test_walks_of_every_length(K, H, d):
    wl = Workload("fwd_units", 1, H, 7, 22, 30, d, K)
    g = grid_of(wl)
    run_and_check(wl, tiled_bits(wl, seed=K + d + H, pad_garbage=True), random_lists(wl, g, K))


# d, heads of 96 query blocks, list lengths: the general kernel with two wavefronts per workgroup
TWO_WAVES = [(128, 3, K) for K in (9, 10, 11, 12, 13, 14, 65)] + [(64, 9, K) for K in (3, 4, 5, 6, 7, 8, 65)]


@pytest.mark.parametrize("d,H,K", TWO_WAVES)
def test_walks_of_two_wavefronts(d, H, K):
    wl = Workload("fwd_two", 1, H, 7, 22, 30, d, K)
    g = grid_of(wl)
    assert_kernel(wl, TWO)
    run_and_check(wl, tiled_bits(wl, seed=300 + K + d, pad_garbage=True), random_lists(wl, g, K))


# d, heads of 96 query blocks, list length, kernel, whether workgroups take two blocks
RULE = [(128, 5, 10, SHORT, False), (128, 5, 11, TWO, False), (128, 12, 20, SHORT, False), (128, 12, 21, TWO, True),
        (128, 24, 12, SHORT, False), (128, 24, 13, TWO, True), (128, 28, 4, SHORT, False), (128, 28, 5, TWO, True),
        (128, 5, 16, TWO, False), (128, 5, 17, TWO, False), (128, 12, 44, TWO, True), (128, 12, 45, TWO, True),
        (128, 24, 26, TWO, True), (128, 24, 27, TWO, True), (128, 28, 18, TWO, True), (128, 28, 19, TWO, True),
        (64, 6, 16, SHORT, False), (64, 6, 17, FOUR, False), (64, 12, 14, SHORT, False), (64, 12, 15, FOUR, False),
        (64, 28, 9, SHORT, False), (64, 28, 10, TWO, False)]


@pytest.mark.parametrize("d,H,K,waves,paired", RULE)
def test_both_sides_of_the_short_list_rule(d, H, K, waves, paired):
    wl = Workload("fwd_rule", 1, H, 7, 22, 30, d, K)
    g = grid_of(wl)
    assert_kernel(wl, waves, paired)
    run_and_check(wl, tiled_bits(wl, seed=400 + K + d, pad_garbage=True), random_lists(wl, g, K), heads=[0, H // 2, H - 1])


# 576, 1152 and 480 query blocks: the kernel for short lists, and lists that it leaves to the general one
SHORT_WALKS = ([(d, H, K, SHORT, False) for d, H in ((64, 6), (128, 12)) for K in (1, 2, 12, 13)] +
               [(128, 5, K, SHORT, False) for K in (1, 2, 9)] + [(128, 5, K, TWO, False) for K in (12, 13)])


@pytest.mark.parametrize("d,H,K,waves,paired", SHORT_WALKS)
def test_short_walks_of_larger_launches(K, d, H, waves, paired):
    wl = Workload("fwd_short", 1, H, 7, 22, 30, d, K)
    g = grid_of(wl)
    assert_kernel(wl, waves, paired)
    run_and_check(wl, tiled_bits(wl, seed=200 + K + d, pad_garbage=True), random_lists(wl, g, K))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H", [1, 3])
def test_walks_that_begin_without_a_valid_key(H, d, K=9):
    """6 frames: in the last layer of cubes slots 32..63 are pads, so the wavefronts of the second key half meet only
    pads in lists of that layer (even rows) and a valid key late in the others."""
    wl = Workload("fwd_dead", 1, H, 6, 22, 30, d, K)
    g = grid_of(wl)
    idx = random_lists(wl, g, 5)
    layer = np.arange(g.Nc // 2, g.Nc)
    rng = np.random.default_rng(1)
    for h in range(H):
        for c in range(g.Nc):
            pick = rng.permutation(layer)[:wl.topk].astype(np.int32)
            if c % 2:
                pick[-1] = c % (g.Nc // 2)  # (the order of a list is free)
            idx[0, h, c] = pick
    run_and_check(wl, tiled_bits(wl, seed=3, pad_garbage=True), idx)


@pytest.mark.parametrize("d,H,K,waves", [(64, 9, 9, TWO), (64, 9, 14, TWO), (64, 6, 9, SHORT), (128, 5, 9, SHORT), (128, 12, 9, SHORT),
                                         (128, 3, 14, TWO)])
def test_walks_of_two_wavefronts_that_begin_without_a_valid_key(d, H, K, waves):
    """Two wavefronts, and the kernel for short lists."""
    assert_kernel(Workload("fwd_dead", 1, H, 6, 22, 30, d, K), waves)
    test_walks_that_begin_without_a_valid_key(H, d, K)


@pytest.mark.parametrize("order", ["rising", "falling", "mixed"])
def test_reference_of_two_wavefronts(order):
    test_reference_follows_the_logits(order, 9, 64)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("H", [1, 3])
@pytest.mark.parametrize("order", ["rising", "falling", "mixed"])
def test_reference_follows_the_logits(order, H, d):
    """Logits between -290 and 290 (log2 units), constant per key cube up to noise: rising lists grow by
    about 15 per entry, mixed ones jump by up to 580, more than fp32 holds."""
    wl = Workload("fwd_ramp", 1, H, 7, 22, 30, d, 40)
    g = grid_of(wl)
    bits = tiled_bits(wl, seed=d)
    rng = np.random.default_rng(d + H)
    ramp = np.linspace(-200.0, 200.0, g.Nc)
    if order == "falling":
        ramp = ramp[::-1]
    if order == "mixed":
        ramp = rng.permutation(ramp)
    u = rng.choice([-1.0, 1.0], size=d)
    # q.k = d * 8 / sqrt(d) * ramp / 8, times log2(e) / sqrt(d): 1.44 * ramp
    k = np.repeat(ramp, g.Np // g.Nc)[None, None, :, None] * u / np.sqrt(d) + 0.3 * rng.standard_normal((1, H, g.Np, d))
    q = u + 0.1 * rng.standard_normal((1, H, g.Np, d))
    bits["q"], bits["k"] = synth.f32_to_bf16_bits(q.astype(np.float32)), synth.f32_to_bf16_bits(k.astype(np.float32))
    run_and_check(wl, bits, random_lists(wl, g, 11))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("waves", [4, 2])
@pytest.mark.parametrize("scale", [2.0 ** 60, 2.0 ** 110])
def test_values_of_any_magnitude(scale, waves, d):
    """Rising logits, up to 57 (log2 units) above the first unit's: V of magnitude 2^60 still fits beside them before O is
    normalised, 2^110 does not."""
    H = 1 if waves == 4 else {64: 9, 128: 3}[d]
    wl = Workload("fwd_big", 1, H, 7, 22, 30, d, 40)
    g = grid_of(wl)
    assert_kernel(wl, waves)
    bits = tiled_bits(wl, seed=d + 1, pad_garbage=True)
    rng = np.random.default_rng(d + H)
    ramp = np.linspace(-20.0, 20.0, g.Nc)
    u = rng.choice([-1.0, 1.0], size=d)
    k = np.repeat(ramp, g.Np // g.Nc)[None, None, :, None] * u / np.sqrt(d) + 0.1 * rng.standard_normal((1, H, g.Np, d))
    q = u + 0.1 * rng.standard_normal((1, H, g.Np, d))
    bits["q"], bits["k"] = synth.f32_to_bf16_bits(q.astype(np.float32)), synth.f32_to_bf16_bits(k.astype(np.float32))
    bits["v"] = synth.f32_to_bf16_bits(widen(bits)["v"] * np.float32(scale))
    run_and_check(wl, bits, random_lists(wl, g, 11))


@pytest.mark.parametrize("H,K,d,waves", [(1, 9, 64, FOUR), (1, 9, 128, FOUR), (6, 5, 64, SHORT), (5, 5, 128, SHORT), (9, 20, 64, TWO),
                                         (3, 20, 128, TWO)])
def test_rows_whose_logits_are_all_minus_infinity(H, K, d, waves):
    """As a row without a valid key: O_f = 0, lse = 0, and no NaN in the gradients of the keys."""
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("fwd_minf", 1, H, 7, 22, 30, d, K)
    g = grid_of(wl)
    assert_kernel(wl, waves)
    bits = tiled_bits(wl, seed=K + d)
    valid, _ = orc.valid_mask(g)
    V = g.Np // g.Nc
    bits["q"] = synth.f32_to_bf16_bits(np.abs(widen(bits)["q"]) + np.float32(0.01))
    k = widen(bits)["k"]
    n = max(12, K)
    k[:, :, :n * V, 0] = np.where(valid[:n * V], -np.inf, 0.0)
    bits["k"] = synth.f32_to_bf16_bits(k)
    idx = random_lists(wl, g, K)
    idx[:, :, :4] = np.arange(K)  # the lists of the first cubes name only such keys
    with np.errstate(invalid="ignore"):
        x = widen(bits)
        ref = orc.forward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], K, real="f32", block_idx=idx)
    dev, buf = to_dev(bits), vsa.Buffers(problem_of(wl))
    buf.block_idx.copy_(torch.from_numpy(idx))
    a = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.forward(*a, indices_given=True)
    torch.cuda.synchronize()
    of, lse = bf16_to_np(buf.out_fine), buf.lse_fine.cpu().numpy()
    assert (of[:, :, :4 * V] == 0).all() and (lse[:, :, :4 * V] == 0).all()
    # (elsewhere a list may still name nothing but those cubes: compared where the oracle has a result)
    rest = np.isfinite(ref["lse_fine"][:, :, 4 * V:])
    assert rest.mean() > 0.9 and np.isfinite(of).all() and np.isfinite(lse).all()
    assert_close(of[:, :, 4 * V:][rest], ref["out_fine"][:, :, 4 * V:][rest], "out_fine")
    buf.backward(*a, dev["dout"], workspace_kept=True)
    torch.cuda.synchronize()
    assert np.isfinite(bf16_to_np(buf.dk)).all() and np.isfinite(bf16_to_np(buf.dv)).all()


LARGE, GANGS = (2, 24, 48, 80), (1, 24, 64, 88)  # heads of 1440 blocks; of 2112 blocks, whose workgroups start in gangs


@pytest.mark.parametrize("d,K,shape", [(64, 300, LARGE), (128, 150, LARGE), (128, 20, LARGE), (128, 300, GANGS),
                                       (128, 150, GANGS), (128, 30, GANGS)])
def test_gangs_of_large_heads(d, K, shape):
    """Large heads without gangs, and with (every one, every second, every ninth; the last gang of an XCD is not a whole
    one).  Sampled query cubes against the oracle; graph replays, with the counters' memory poisoned in between,
    bit-identical."""
    import torch
    from paper_2505_13389_amd import vsa
    wl = Workload("fwd_gang", 1, *shape, d, K)
    g = grid_of(wl)
    bits = tiled_bits(wl, seed=K)
    x, dev = widen(bits), to_dev(bits)
    idx = random_lists(wl, g, K)
    cubes = np.array([0, 1, 511, 512, 777, g.Nc - 1], np.int32)
    ref = orc.forward(g, x["q"], x["k"], x["v"], x["gate_c"], x["gate_f"], K, real="f32", block_idx=idx, cubes=cubes)
    buf = vsa.Buffers(problem_of(wl))
    buf.block_idx.copy_(torch.from_numpy(idx))
    args = (dev["q"], dev["k"], dev["v"], dev["gate_c"], dev["gate_f"])
    buf.forward(*args, indices_given=True)
    torch.cuda.synchronize()
    V = g.Np // g.Nc
    rows = (cubes[:, None] * V + np.arange(V)).ravel()
    assert_close(bf16_to_np(buf.out)[:, :, rows], ref["out"][:, :, rows], "out")
    eager = buf.out.clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        buf.forward(*args, indices_given=True)
    for rep in range(3):
        buf.out.fill_(float("nan"))
        buf.workspace.fill_(0xFF)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(buf.out.view(torch.int16), eager.view(torch.int16)), f"replay {rep}"


@pytest.mark.parametrize("K,waves", [(20, SHORT), (21, TWO)])
def test_both_sides_of_the_line_of_large_heads(K, waves):
    wl = Workload("fwd_gang", 1, *GANGS, 128, K)
    assert_kernel(wl, waves, waves == TWO)
    test_gangs_of_large_heads(128, K, GANGS)


# d = 128, heads of 96 query blocks, list length, kernel, whether workgroups take two blocks: the lines of 369 to 448, 1153 to 1280, 2049 to
# 2304, 2305 to 2560, 2816 to 3071, 3073 to 3264 and 4097 to 4608 blocks
LATER_LINES = [(4, 4, SHORT, False), (4, 5, TWO, False), (13, 10, SHORT, False), (13, 11, TWO, True), (22, 12, SHORT, False), (22, 13, TWO, True),
               (25, 5, SHORT, False), (25, 6, TWO, True), (25, 7, TWO, True), (30, 3, SHORT, False), (30, 4, TWO, True),
               (33, 6, SHORT, False), (33, 7, TWO, True), (47, 3, SHORT, False), (47, 4, TWO, True)]


@pytest.mark.parametrize("H,K,waves,paired", LATER_LINES)
def test_both_sides_of_the_lines_drawn_later(H, K, waves, paired):
    test_both_sides_of_the_short_list_rule(128, H, K, waves, paired)
