"""Stand-alone sparse attention where the number of workgroups per head changes: one per head (no merge), one per 32
rows, at most eight or sixteen; lists with padding in them."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,k", [(8, 32, 8, 256), (8, 32, 8, 257), (8, 31, 31, 256), (16, 32, 8, 40),
                                        (33, 32, 4, 33), (2, 32, 8, 512), (1, 8, 8, 700), (40, 32, 32, 1), (17, 32, 8, 513),
                                        (32, 32, 32, 896), (3, 32, 8, 900), (10, 32, 8, 400), (10, 32, 8, 257)])
def test_sparse_attention_over_lists_of_every_plan(B, Hq, Hkv, k):
    import paper_2510_18413_amd as A
    L, d, G = 900, 128, Hq // Hkv
    gen = torch.Generator().manual_seed(B * 1000 + k)
    K = (torch.randn(Hkv, B * L, d, generator=gen) * 2).to(torch.bfloat16)
    V = torch.randn(Hkv, B * L, d, generator=gen).to(torch.bfloat16)
    q = torch.randn(B, Hq, d, generator=gen).to(torch.bfloat16)
    idx = torch.rand(B, Hq, L, generator=gen).topk(k, dim=-1).indices.sort(-1).values.to(torch.int32)
    idx[torch.rand(idx.shape, generator=gen) < 0.1] = -1      # padding anywhere in a list
    idx[0, 0] = -1                                            # a list of nothing else: zeros
    cfg = A.Config.make(Hq, Hkv, B * L)
    out = torch.full((B, Hq, d), 7.0, device="cuda")
    ws = torch.full((A.adamas_workspace_bytes(cfg, B, L, k),), 0xA5, dtype=torch.uint8, device="cuda")
    A.adamas_sparse_attn(cfg, q.cuda(), K.cuda(), V.cuda(), (torch.arange(B) * L).cuda(), idx.cuda(), out, L, ws)
    ref = torch.zeros(B, Hq, d, dtype=torch.float64)
    for b in range(B):
        for h in range(Hq):
            t = idx[b, h][idx[b, h] >= 0].long() + b * L
            if t.numel():
                w = torch.softmax(K[h // G, t].double() @ q[b, h].double() / d ** 0.5, 0)
                ref[b, h] = w @ V[h // G, t].double()
    got = out.cpu().double()
    # scores in fp64; a weight carries a few roundings to fp32 (2^-24 each), its sums at most k more
    assert float((got - ref).abs().max()) <= (k + 16) * 2.0 ** -23 * 5
    assert float((got - ref).norm() / ref.norm()) <= 1e-6
