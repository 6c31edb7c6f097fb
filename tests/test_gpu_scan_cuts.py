"""The scan's cuts, by tile (1024, 2048 or 4096 tokens) and by parts of the query group (1, 2 or 4): distances, selected
positions and outputs against the oracle where each cut is chosen, one token before, on and after the edge of a tile, of
a wave's 256 tokens and of a lane's eight.  Calls of short contexts run as one launch and have no cut: their steps are
also run as the two kernels, one by one."""

import numpy as np
import pytest
import torch

import paper_2510_18413_amd as A
import plan_query as P
import synth_inputs as synth

# B, query heads, KV heads, length, head dimension; (tile, parts) of the step, of top-k, of the distances alone
CUTS = [
    ((2, 3, 1, 1023, 64), (2048, 1), (1024, 1), (1024, 1)),         # one tile
    ((1, 2, 1, 1017, 128), (2048, 2), (1024, 2), (1024, 2)),        # a head per workgroup
    ((1, 8, 1, 1023, 128), (2048, 4), (1024, 4), (1024, 4)),        # two heads of eight
    ((1, 4, 1, 2049, 128), (2048, 4), (1024, 4), (1024, 4)),
    ((1, 8, 1, 2304, 128), (2048, 4), (1024, 4), (1024, 4)),
    ((1, 8, 1, 8191, 64), (2048, 4), (1024, 4), (1024, 4)),
    ((2, 12, 4, 4097, 128), (2048, 1), (1024, 1), (1024, 1)),       # a group of three is not cut
    ((3, 24, 4, 4105, 128), (2048, 2), (1024, 2), (1024, 2)),       # a group of six: halves only
    ((40, 4, 1, 5000, 128), (2048, 2), (1024, 1), (1024, 1)),
    ((5, 16, 2, 33000, 128), (4096, 2), (4096, 2), (4096, 2)),      # halves of eight heads
    ((1, 16, 2, 65537, 128), (4096, 4), (4096, 4), (2048, 2)),      # quarters of eight heads, seventeen tiles
    ((1, 4, 1, 40003, 128), (4096, 4), (4096, 4), (1024, 4)),       # quarters of four heads
    ((9, 32, 8, 4096, 128), (4096, 2), (2048, 1), (2048, 1)),       # halves of four heads
    ((3, 32, 8, 30001, 128), (4096, 1), (4096, 1), (4096, 1)),      # four heads together, sixteen waves
    ((70, 3, 3, 4095, 128), (4096, 1), (2048, 1), (2048, 1)),       # one head per row, sixteen waves
    ((9, 32, 8, 4097, 96), (2048, 1), (2048, 1), (2048, 1)),
    ((16, 32, 8, 8200, 128), (2048, 1), (2048, 1), (2048, 1)),      # more workgroups than compute units
    ((33, 16, 8, 2049, 256), (2048, 1), (2048, 1), (2048, 1)),      # uint16 distances
    # six, nine, ten and thirteen tiles of histograms: as many at once as the select kernel's instance takes
    ((1, 4, 1, 12001, 128), (2048, 4), (1024, 4), (1024, 4)), ((1, 4, 1, 17001, 96), (2048, 4), (2048, 4), (1024, 4)),
    ((1, 4, 1, 26001, 64), (2048, 4), (2048, 4), (1024, 4)),
    # seventeen: a second batch of them
    ((2, 8, 2, 66001, 128), (4096, 2), (4096, 2), (2048, 1)), ((2, 32, 4, 66001, 64), (4096, 1), (4096, 1), (4096, 1)),
    ((2, 64, 8, 66001, 64), (2048, 1), (4096, 1), (2048, 1)),       # segments of 16384 tokens, 33 and seventeen tiles
    # contexts from which on few heads run as two kernels, for the cuts of the smaller tiles
    ((1, 1, 1, 10241, 128), (2048, 1), (1024, 1), (1024, 1)), ((1, 2, 1, 10239, 128), (2048, 2), (1024, 2), (1024, 2)),
    ((1, 2, 1, 14337, 128), (2048, 2), (1024, 2), (1024, 2)), ((1, 4, 1, 12287, 64), (2048, 4), (1024, 4), (1024, 4)),
    ((1, 1, 1, 20481, 128), (2048, 1), (2048, 1), (1024, 1)), ((1, 2, 1, 22527, 128), (2048, 2), (2048, 2), (1024, 2)),
    ((2, 6, 2, 13313, 160), (2048, 1), (1024, 1), (1024, 1)),
]
K = 96


def of(shape):
    B, Hq, Hkv, L, d = shape
    return P.config(Hq, Hkv, head_dim=d), B, L, min(K, L - 3 * B)


def test_every_cut_is_here():
    """Among the calls that run as two kernels."""
    run = {P.STEP: set(), P.TOPK: set()}
    for shape, *cuts in CUTS:
        cfg, B, L, k = of(shape)
        for use, want in zip((P.STEP, P.TOPK, P.DISTANCES), cuts):
            got = P.cut(cfg, B, L, use)
            assert (got.tile, got.parts) == want, (shape, use)
            if use != P.DISTANCES and P.waves(cfg, B, L, k, use) == 0:
                run[use].add(want)
    every = {(tile, parts) for tile in (1024, 2048, 4096) for parts in (1, 2, 4)}
    assert run[P.STEP] == {c for c in every if c[0] > 1024}        # no tiles of 1024 in the step
    assert run[P.TOPK] == every


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,L,d", [c[0] for c in CUTS])
def test_step_at_every_cut_of_the_scan(oracle, B, Hq, Hkv, L, d):
    from gpu_harness import ATTN_TOL, POISON, DeviceCase, attn_rel_err, oracle_step, two_kernels
    G = Hq // Hkv
    lens = [max(2, L - 3 * i) for i in range(B)]
    case = synth.make_case("cut", 7000 + L + B, B, Hq, Hkv, lens, [0],
                           lambda b, Lc, h, rng: rng.choice(Lc, size=(G, 1), replace=False), append=True, head_dim=d)
    k = of((B, Hq, Hkv, L, d))[-1]
    want = oracle_step(case, k)
    one = P.waves(P.config(Hq, Hkv, head_dim=d), B, L, k) != 0
    for staged in (False, True) if one else (False,):
        dc = DeviceCase(case, k)
        if staged:
            for stages in (A.STAGE_SCAN, A.STAGE_SELECT_ATTN):
                A.adamas_decode_step_stages(dc.cfg, dc.q, dc.K, dc.V, dc.codes, dc.seq_start, dc.seq_len, k, dc.out, dc.max_len,
                                            dc.workspace, k_new=dc.k_new, v_new=dc.v_new, idx_out=dc.idx, stages=stages)
            out, idx = dc.out.cpu().numpy(), dc.idx.cpu().numpy()
        else:
            out, idx = dc.decode_step()
        assert two_kernels(dc.workspace) == (staged or not one)
        assert np.array_equal(idx, want["idx"])
        assert attn_rel_err(out, want["out"]) <= ATTN_TOL
        got_rows = dc.codes.cpu().numpy()
        for b in range(B):       # the appended row is in the cache
            at = int(case.seq_start[b]) + lens[b] - 1
            assert np.array_equal(got_rows[:, at], want["rows"][:, at])
    # the distances themselves, of the stand-alone scan and of top-k
    qcodes = torch.zeros(B, Hq, dc.cfg.code_row_bytes, dtype=torch.uint8, device="cuda")
    A.adamas_encode_query(dc.cfg, dc.q, qcodes)
    dist = torch.zeros(B, Hq, dc.max_len, dtype=torch.uint16, device="cuda")
    A.adamas_manhattan_distance(dc.cfg, qcodes, dc.codes, dc.seq_start, dc.seq_len, dist)
    dist2, idx2 = torch.zeros_like(dist), torch.zeros_like(dc.idx)
    dc.workspace.fill_(POISON)
    A.adamas_select_topk(dc.cfg, qcodes, dc.codes, dc.seq_start, dc.seq_len, k, idx2, dc.max_len, dc.workspace, dist_out=dist2)
    assert two_kernels(dc.workspace) == (P.waves(P.config(Hq, Hkv, head_dim=d), B, L, k, P.TOPK) == 0)
    assert np.array_equal(idx2.cpu().numpy(), want["idx"])
    for got in (dist, dist2):
        got = got.cpu().view(torch.int16).numpy().view(np.uint16).astype(np.int32)
        for b in range(B):
            assert np.array_equal(got[b, :, :lens[b]], want["dist"][b][:, :lens[b]])


def test_the_static_array_takes_every_shape_that_fits_with_the_fewest_histograms():
    """Tiles of 4096 tokens need the least scratch: the static call is never refused because the plan would rather have
    smaller ones.  (No pointer is given, so a call that fits ends at the check behind the one of its scratch.)"""
    lib = A.library()

    def fits(cfg, batch, L):
        rc = lib.adamas_decode_step_static(cfg, None, None, None, None, None, None, None, None, batch, 64, None, None, L, None)
        assert rc in (-1, -3)
        return rc == -1

    for group, kv, batch in [(1, 32, 1), (4, 8, 3), (4, 8, 11), (8, 2, 20), (2, 8, 7), (4, 1, 150), (4, 8, 16), (4, 8, 41)]:
        heads = batch * kv * group
        cfg = A.Config.make(kv * group, kv, 1 << 22)
        for L in range(700, 1 << 17, 1777):
            tiles = -(-L // 4096)
            least = heads * (-(-L // 128) * 128) * 9 // 8 + (heads * tiles + 16) * 193 * 4 + heads * 16 * 132 * 4 + 4 * 256
            if least <= A.STATIC_SCRATCH_BYTES:
                assert fits(cfg, batch, L), (group, kv, batch, L)
            if A.adamas_workspace_bytes(cfg, batch, L, 64) <= A.STATIC_SCRATCH_BYTES:
                assert fits(cfg, batch, L), (group, kv, batch, L)


# sequences, context, shortest sequence
FEWEST = [(12, 24000, 2000), (41, 2560, 2360)]      # as two kernels, as one launch


def test_the_static_step_with_the_fewest_histograms_has_another_cut():
    cfg = P.config(32, 8)
    for (B, L, _), two in zip(FEWEST, (True, False)):
        assert P.cut(cfg, B, L).tile == 2048 and P.cut(cfg, B, L, P.STATIC).tile == 4096
        assert (P.waves(cfg, B, L, 48) == 0) == two


@pytest.mark.gpu
@pytest.mark.parametrize("B,L,least", FEWEST)
def test_the_static_step_with_the_fewest_histograms(oracle, B, L, least):
    """A shape that fits the static array only with tiles of 4096 tokens, while the plan takes 2048: same results."""
    from gpu_harness import ATTN_TOL, DeviceCase, attn_rel_err, oracle_step
    k = 48
    case = synth.make_case("static cut", 31, B, 32, 8, [L - (L - least) * b // (B - 1) for b in range(B)], [0],
                           lambda b, Lc, h, rng: rng.choice(Lc, size=(4, 1), replace=False), append=True)
    dc = DeviceCase(case, k)
    assert A.adamas_workspace_bytes(dc.cfg, B, dc.max_len, k) > A.STATIC_SCRATCH_BYTES
    A.adamas_decode_step_static(dc.cfg, dc.q, dc.K, dc.V, dc.codes, dc.seq_start, dc.seq_len, k, dc.out, dc.max_len,
                                k_new=dc.k_new, v_new=dc.v_new, idx_out=dc.idx)
    torch.cuda.synchronize()
    want = oracle_step(case, k)
    assert np.array_equal(dc.idx.cpu().numpy(), want["idx"])
    assert attn_rel_err(dc.out.cpu().numpy(), want["out"]) <= ATTN_TOL
