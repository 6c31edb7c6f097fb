"""The scan's plan (csrc/plan.hpp) without a GPU."""

import pytest

import plan_query as P
import paper_2510_18413_amd as A


@pytest.mark.parametrize("heads,kv,d", [(1, 1, 128), (32, 8, 128), (24, 8, 96), (16, 2, 64), (14, 2, 256)])
def test_every_cut_divides_the_group_and_covers_the_context(heads, kv, d):
    for batch in (1, 3, 16, 200):
        for L in (1, 63, 1024, 1025, 4097, 32771, 200001, 1 << 20):
            c = P.cut(P.config(heads, kv, head_dim=d), batch, L)
            assert c.tile in (1024, 2048, 4096) and (heads // kv) % c.parts == 0
            assert (c.n_tiles - 1) * c.tile < L <= c.n_tiles * c.tile
            assert c.scratch <= A.adamas_workspace_bytes(P.config(heads, kv, head_dim=d), batch, L, 64)


@pytest.mark.parametrize("batch,L", [(16, 17408), (12, 24576), (41, 2560)])
def test_the_static_array_does_not_decide_the_cut_of_other_calls(batch, L):
    """These need just over the static array's bytes with the tiles that take the least time, and less with the largest."""
    c = P.cut(P.config(32, 8), batch, L)
    assert (c.tile, c.parts) == (2048, 1) and c.scratch > A.STATIC_SCRATCH_BYTES


@pytest.mark.parametrize("heads,kv,kw", [(32, 8, {}), (32, 32, {}), (8, 1, {}), (6, 2, dict(head_dim=256)), (12, 4, dict(variant=A.VARIANT_L2)),
                                         (5, 1, dict(code_bits=1, thr_k=(0.0,)))])
def test_a_workspace_for_the_largest_call_serves_the_smaller_ones(heads, kv, kw):
    cfg = P.config(heads, kv, context=1 << 20, **kw)
    need = lambda batch, L: A.adamas_workspace_bytes(cfg, batch, L, 64)
    for batch in (1, 2, 8, 16, 61):
        last = 0
        for L in list(range(1, 60000, 509)) + [1 << 17, 200000, 1 << 20]:
            here = need(batch, L)
            assert here >= last and here >= P.cut(cfg, batch, L).scratch, (batch, L)
            last = here
    for L in (700, 1024, 2560, 8192, 21248, 32768):
        sizes = [need(batch, L) for batch in range(1, 80)]
        assert sizes == sorted(sizes), L
    # refused and served at these before: 16 sequences with a workspace for 24576 tokens, eight with one for 32768
    if (heads, kv) == (32, 8):
        assert max(need(16, L) for L in range(21248, 22529, 128)) <= need(16, 24576)
        assert max(need(b, 32768) for b in range(1, 12)) <= need(12, 32768)
    if (heads, kv) == (32, 32):
        assert max(need(8, L) for L in range(28800, 30721, 128)) <= need(8, 32768)
