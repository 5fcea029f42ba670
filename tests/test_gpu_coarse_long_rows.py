"""Coarse stage in one launch for 513 to 768 cubes.  With d = 128 and more than 256 workgroups (here: 8 heads) its third step requests rows of V_c
four groups of 16 at a time, else one: first and last number of cubes, whole and broken groups, rounds and shares of a wavefront, against
float64.  And shorter and longer rows."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [2, 8])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [(1, 19, 27), (2, 16, 17), (3, 11, 17), (7, 9, 10), (8, 8, 10), (13, 59, 1), (8, 8, 12)])  # 513 to 768 cubes
def test_coarse_stage_of_long_rows(n, d, H):
    Nc = n[0] * n[1] * n[2]
    assert 512 < Nc <= 768 and (H * ((Nc + 15) // 16) > 256) == (H == 8)
    check(n, d, H)


# groups of 16 rows, whole and not, fewer and more than wavefronts share them, in every instance by the length of a row
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [(1, 1, 3), (1, 3, 5), (2, 2, 4), (1, 1, 17), (1, 1, 31), (3, 3, 7), (4, 4, 4), (1, 5, 13), (3, 5, 5), (4, 4, 5), (1, 1, 127),
                               (4, 4, 8), (3, 1, 43), (5, 6, 8), (1, 1, 257), (8, 8, 8), (1, 1, 769), (13, 7, 11), (1, 25, 41), (16, 12, 8)])
def test_coarse_stage_by_groups_of_rows(n, d):
    check(n, d, 3)


def check(n, d, H, K=3):
    import torch
    from paper_2505_13389_amd import vsa
    pb = vsa.Problem(1, H, 4 * n[0], 4 * n[1], 4 * n[2], d, K, flags=vsa.VSA_FLAG_COARSE_FUSED)
    Np, Nc = vsa.vsa_padded_tokens(pb)
    assert Nc == n[0] * n[1] * n[2]
    g = torch.Generator(device="cuda")
    g.manual_seed(Nc + d)
    q, k, v, gate = (torch.randn((1, H, Np, d), generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    buf = vsa.Buffers(pb, with_gate_f=False)
    buf.forward(q, k, v, gate, None)
    torch.cuda.synchronize()
    qc, kc, vc = (x[0].double().view(H, Nc, 64, d).mean(2) for x in (q, k, v))
    S = torch.bmm(qc, kc.transpose(1, 2).contiguous()) * d ** -0.5
    # float32 sums of 64, d and Nc terms of order one: off by some 1e-6; 2e-5 is a wide margin for them and far below a missing row
    oc = torch.bmm(torch.softmax(S, -1), vc)
    got = buf.out_coarse[0].double()
    assert float((got - oc).norm() / oc.norm()) < 2e-5
    assert float((buf.lse_coarse[0].double() - torch.logsumexp(S, -1)).abs().max()) < 2e-5
    idx = buf.block_idx[0].long()
    least = torch.gather(S, 2, idx).min(-1).values
    assert bool((least >= torch.topk(S, K, -1).values[..., -1] - 1e-5).all()) and bool((idx[..., 1:] > idx[..., :-1]).all())
