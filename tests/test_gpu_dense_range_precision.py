"""Dense attention: values near the end of the range, infinite elements in the last row of a sequence."""

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
