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
