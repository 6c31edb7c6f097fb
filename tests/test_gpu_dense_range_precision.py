"""Dense attention: values near the end of the range, infinite elements in the last row of a sequence, and
scores as exact as sums in fp32."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def full_attention(q, K, V, starts, lens):
    """q [B][Hq][d], K, V [Hkv][pool][d] (bf16, on the CPU) -> the library's output as float64."""
    import paper_2510_18413_amd as A
    (Hkv, pool, d), (B, Hq, _) = K.shape, q.shape
    cfg = A.Config.make(Hq, Hkv, pool, head_dim=d)
    out = torch.full((B, Hq, d), -7.0, device="cuda")
    ws = torch.full((A.adamas_full_attn_workspace_bytes(cfg, B, max(lens)),), 0xA5, dtype=torch.uint8, device="cuda")
    A.adamas_full_attn(cfg, q.cuda(), K.cuda(), V.cuda(), torch.tensor(starts, dtype=torch.int64).cuda(),
                       torch.tensor(lens, dtype=torch.int32).cuda(), out, max(lens), ws)
    return out.cpu().double()


@pytest.mark.parametrize("G", [1, 4, 5, 6, 8])
def test_values_near_the_end_of_the_range(G):
    """A wave meets token 0 first and token 130, 2^7 times its weight, in its next step: the weighted sum may
    not pass the largest V by the ratio of the two weights."""
    d, L, Hkv = 128, 300, 2
    K = torch.zeros(Hkv, L, d)
    K[:, :, 0] = -40 / (d ** -0.5 * 1.4426950408889634)
    K[:, 0, 0] = 0
    K[:, 130, 0] = 7 / (d ** -0.5 * 1.4426950408889634)
    V = torch.full((Hkv, L, d), 1e30)
    V[:, 0] = 1e38
    V[:, 130] = 3e38
    V[:, :, 1::2] *= -1
    q = torch.zeros(1, Hkv * G, d)
    q[:, :, 0] = 1
    q, K, V = q.bfloat16(), K.bfloat16(), V.bfloat16()
    out = full_attention(q, K, V, [0], [L])
    for h in range(Hkv * G):
        ref = torch.softmax(K[h // G].double() @ q[0, h].double() / d ** 0.5, 0) @ V[h // G].double()
        # weights and sums in fp32, 300 tokens: below 310 roundings of 2^-24 each
        assert float(((out[0, h] - ref) / ref).abs().max()) < 310 * 2.0 ** -24


@pytest.mark.parametrize("G", [1, 5, 8])
@pytest.mark.parametrize("d", [64, 128, 192])
def test_an_infinite_element_in_the_last_row(G, d):
    gen = torch.Generator().manual_seed(G + d)
    lens, Hkv = [1, 33, 200, 64, 127], 2
    starts = [0] + list(np.cumsum(lens)[:-1])
    K, V = (torch.randn(Hkv, sum(lens), d, generator=gen).bfloat16() for _ in range(2))
    q = torch.randn(len(lens), Hkv * G, d, generator=gen).bfloat16()
    inf = float("inf")
    for s, L in zip(starts, lens):
        V[0, s + L - 1, 3] = inf
        V[1, s + L - 1, 8] = -inf
    out = full_attention(q, K, V, starts, lens)
    assert torch.all(out[:, :G, 3] == inf) and torch.all(out[:, G:, 8] == -inf)
    fine = torch.ones_like(out, dtype=torch.bool)
    fine[:, :G, 3] = fine[:, G:, 8] = False
    assert torch.isfinite(out[fine]).all()


def fp32_scores(q, k, lanes):
    """Scores of pairs of rows as sums in fp32: `lanes` chains of fused multiply-adds, joined pairwise."""
    d = q.shape[-1]
    q, k = q.double().view(-1, lanes, d // lanes), k.double().view(-1, lanes, d // lanes)
    acc = torch.zeros(q.shape[:2])
    for j in range(d // lanes):
        acc = (acc.double() + q[:, :, j] * k[:, :, j]).float()     # the product of two bf16 numbers is exact
    while acc.shape[1] > 1:
        acc = acc[:, 0::2] + acc[:, 1::2]
    return acc[:, 0]


@pytest.mark.parametrize("G,d", [(1, 64), (4, 64), (8, 64), (1, 128), (4, 128), (8, 128), (4, 192), (1, 256), (4, 256), (8, 256)])
def test_scores_are_as_exact_as_sums_in_fp32(G, d):
    """Sequences of two tokens with V = 0 and V = 1: the output is the second one's weight, and its logit the
    difference of the two scores.  Rows near the query, with a few large channels: large scores that differ little,
    so that what their sums lose shows."""
    gen = torch.Generator().manual_seed(100 * G + d)
    B, Hkv = 2048, 2
    n = lambda *s: torch.randn(*s, generator=gen)
    scale = torch.ones(Hkv, d).scatter_(1, torch.rand(Hkv, d, generator=gen).topk(4).indices, 8.0)
    base = n(B, Hkv, d) * scale
    K = (base[:, :, None] + 0.1 * n(B, Hkv, 2, d)).permute(1, 0, 2, 3).reshape(Hkv, 2 * B, d).bfloat16().contiguous()
    q = (base[:, :, None] + 0.1 * n(B, Hkv, G, d)).reshape(B, Hkv * G, d).bfloat16()
    V = torch.zeros(Hkv, 2 * B, d)
    V[:, 1::2] = 1
    w = full_attention(q, K, V.bfloat16(), [2 * b for b in range(B)], [2] * B)[:, :, 0]
    got = torch.log(w) - torch.log1p(-w)
    rows = K.view(Hkv, B, 2, d).permute(1, 0, 2, 3).repeat_interleave(G, 1)              # [B][Hq][2][d]
    exact = (rows.double() * q.double()[:, :, None]).sum(-1) / d ** 0.5
    flat = fp32_scores(q[:, :, None].expand(rows.shape).reshape(-1, d), rows.reshape(-1, d), d // 8 if d & (d - 1) == 0 else 8)
    fp32 = (flat * np.float32(d ** -0.5 * 1.4426950408889634)).double().view(exact.shape) * np.log(2.0)
    rms = lambda x: float(x.square().mean().sqrt())
    mine, theirs = rms(got - (exact[..., 1] - exact[..., 0])), rms((fp32 - exact)[..., 1] - (fp32 - exact)[..., 0])
    print("score error, rms: %.3e, sums in fp32 %.3e" % (mine, theirs))
    # one more rounding of the weights and of the quotient, 2^-24 of a number of about one half each
    assert mine <= theirs * 1.02 + 2.0 ** -24
