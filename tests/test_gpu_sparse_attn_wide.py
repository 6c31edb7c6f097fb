"""Stand-alone sparse attention with one workgroup per head, of four waves for short lists and of sixteen for long ones: at
the limits between them and to several workgroups, lists with padding, of one row and of padding only."""

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,k,d", [(1, 128, 128), (1, 129, 128), (63, 256, 128), (64, 129, 128), (64, 256, 128), (64, 257, 128),
                                       (191, 300, 128), (192, 300, 128), (256, 1025, 128), (257, 300, 128), (255, 1, 128),
                                       (64, 257, 64), (70, 512, 64), (66, 300, 96), (200, 103, 160), (65, 160, 192), (256, 65, 256),
                                       # several passes of the compaction, on both sides of the limits by rows
                                       (192, 1024, 64), (208, 2047, 64), (208, 2048, 64), (193, 4096, 64)])
def test_one_workgroup_per_head(heads, k, d):
    import paper_2510_18413_amd as A
    L = max(1200, k + 50)
    gen = torch.Generator().manual_seed(heads * 1000 + k)
    K = (torch.randn(1, heads * L, d, generator=gen) * 2).to(torch.bfloat16)
    V = torch.randn(1, heads * L, d, generator=gen).to(torch.bfloat16)
    q = torch.randn(heads, 1, d, generator=gen).to(torch.bfloat16)
    idx = torch.rand(heads, 1, L, generator=gen).topk(k, dim=-1).indices.sort(-1).values.to(torch.int32)
    idx[torch.rand(idx.shape, generator=gen) < 0.1] = -1
    idx[-1, 0] = -1                  # nothing but padding: zeros
    if heads > 1:
        idx[0, 0] = -1
        idx[0, 0, k // 2] = 7        # one row: that row of V
    cfg = A.Config.make(1, 1, heads * L, head_dim=d)
    out = torch.full((heads, 1, d), 7.0, device="cuda")
    ws = torch.full((A.adamas_workspace_bytes(cfg, heads, L, k),), 0xA5, dtype=torch.uint8, device="cuda")
    A.adamas_sparse_attn(cfg, q.cuda(), K.cuda(), V.cuda(), (torch.arange(heads) * L).cuda(), idx.cuda(), out, L, ws)
    ref = torch.zeros(heads, 1, d, dtype=torch.float64)
    for b in range(heads):
        t = idx[b, 0][idx[b, 0] >= 0].long() + b * L
        if t.numel():
            ref[b, 0] = torch.softmax(K[0, t].double() @ q[b, 0].double() / d ** 0.5, 0) @ V[0, t].double()
    got = out.cpu().double()
    # scores in fp64; a weight carries a few roundings to fp32 (2^-24 each), its sums at most k more; |V| < 5
    assert float((got - ref).abs().max()) <= (k + 16) * 2.0 ** -23 * 5
    if float(ref.norm()) > 0:
        assert float((got - ref).norm() / ref.norm()) <= 1e-6
