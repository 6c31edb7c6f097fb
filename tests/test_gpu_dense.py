"""Dense attention at the edges of its steps: 16-token blocks, 32-token steps, 128-token rounds of a
workgroup and 256-token splits, every group size (one or two sets of head columns), every head
dimension, and elements that are not finite."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

LENS = [1, 2, 15, 16, 17, 31, 32, 33, 63, 65, 127, 128, 129, 255, 256, 257, 513, 0]


def run(G, d, lens, seed, spoil=None, bound=None):
    """(library's output, the same in float64) for Hkv = 2; sequences packed back to back."""
    import paper_2510_18413_amd as A
    rng = np.random.default_rng(seed)
    Hkv, B = 2, len(lens)
    starts = np.concatenate([[0], np.cumsum(lens)[:-1]]).astype(np.int64)
    pool = int(sum(lens))
    bf = lambda *s: torch.from_numpy(rng.standard_normal(s, dtype=np.float32)).to(torch.bfloat16)
    K, V, q = bf(Hkv, pool, d) * 3, bf(Hkv, pool, d), bf(B, Hkv * G, d)
    if spoil is not None:
        spoil(K, V, q, starts)
    cfg = A.Config.make(Hkv * G, Hkv, pool, head_dim=d)
    out = torch.full((B, Hkv * G, d), -7.0, device="cuda")
    ws = torch.full((A.adamas_full_attn_workspace_bytes(cfg, B, bound or max(lens)),), 0xA5, dtype=torch.uint8, device="cuda")
    A.adamas_full_attn(cfg, q.cuda(), K.cuda(), V.cuda(), torch.from_numpy(starts).cuda(),
                       torch.tensor(lens, dtype=torch.int32).cuda(), out, bound or max(lens), ws)
    ref = torch.zeros(B, Hkv * G, d, dtype=torch.float64)
    for b, L in enumerate(lens):
        for h in range(Hkv * G if L else 0):
            s = slice(int(starts[b]), int(starts[b]) + L)
            w = torch.softmax(K[h // G, s].double() @ q[b, h].double() / d ** 0.5, 0)
            ref[b, h] = w @ V[h // G, s].double()
    return out.cpu().double(), ref


@pytest.mark.parametrize("G,d", [(g, 128) for g in range(1, 9)] + [(1, 64), (8, 64), (5, 96), (7, 96), (4, 160),
                                                                   (6, 160), (3, 192), (8, 192), (2, 256), (8, 256)])
def test_dense_attention_at_the_edges_of_its_steps(G, d):
    out, ref = run(G, d, LENS, 40 + G + d)
    # A score is a sum of d products with |k| about 3: it is off by at most (d + 1) * 2^-23 * sum |q k| (each
    # of its additions and the alignment inside the matrix instruction lose less than 2^-23 of what they add),
    # about 3 * 0.64 * d * 2^-23 * (d + 1); divided by sqrt(d) that is the relative error of a weight, which
    # moves the output by at most that times the largest |V| (below 6).  At d = 256: 0.00094 * 6.
    bound = 6 * 1.92 * d * (d + 1) / d ** 0.5 * 2.0 ** -23
    assert float((out - ref).abs().max()) <= bound
    assert float((out - ref).norm() / ref.norm()) <= 4e-6    # typical: 1e-6, as with fp32 sums in any order


@pytest.mark.parametrize("G", [1, 4, 8])
def test_dense_attention_with_elements_that_are_not_finite(G):
    inf = float("inf")

    def spoil(K, V, q, starts):
        V[0, starts[0] + 40, 3] = inf           # an infinite element of V: that output dim of head 0's group
        V[1, starts[1] + 5, 9] = -inf
        V[0, starts[2] + 64, 0] = float("nan")
        q[3] = q[3].abs()                       # scores of -inf: that token has weight zero
        K[1, starts[3] + 17] = -inf
    out, _ = run(G, 128, [200, 40, 70, 60], 5, spoil)
    clean, ref = run(G, 128, [200, 40, 70, 60], 5, lambda K, V, q, starts: (q[3].abs_(), K[1, starts[3] + 17].fill_(-1e30)))
    assert torch.all(out[0, :G, 3] == inf) and torch.all(out[1, G:, 9] == -inf) and torch.all(torch.isnan(out[2, :G, 0]))
    fine = torch.ones_like(out, dtype=torch.bool)
    fine[0, :G, 3] = fine[1, G:, 9] = fine[2, :G, 0] = False
    assert torch.isfinite(out[fine]).all()
    assert float((out - ref)[fine].abs().max()) < 1e-3


@pytest.mark.parametrize("bound", [513, 768, 5000, 65536, 100001, 1 << 20])
def test_dense_attention_of_lengths_far_below_the_bound(bound):
    """The splits follow each sequence's own length, whatever max_seq_len allows for."""
    out, ref = run(4, 128, LENS, 7, bound=bound)
    assert float((out - ref).abs().max()) <= 6 * 1.92 * 128 * 129 / 128 ** 0.5 * 2.0 ** -23      # as above
    assert float((out - ref).norm() / ref.norm()) <= 4e-6
    assert torch.all(out[LENS.index(0)] == 0)
