"""The scan's plan (csrc/plan.hpp) without a GPU."""

import ctypes

import pytest

import plan_query as P
import paper_2510_18413_amd as A


@pytest.mark.parametrize("heads,kv,d", [(1, 1, 128), (32, 8, 128), (24, 8, 96), (16, 2, 64), (14, 2, 256)])
def test_every_cut_divides_the_group_and_covers_the_context(heads, kv, d):
    for batch in (1, 3, 16, 200):
        for L in (1, 63, 1024, 1025, 4097, 32771, 200001, 1 << 20):
            for use in (P.STEP, P.TOPK, P.DISTANCES, P.STATIC):
                c = P.cut(P.config(heads, kv, head_dim=d), batch, L, use)
                assert c.tile in ((2048, 4096) if use in (P.STEP, P.STATIC) else (1024, 2048, 4096)) and (heads // kv) % c.parts == 0
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
            assert here >= last and here >= max(P.cut(cfg, batch, L, use).scratch for use in range(4)), (batch, L)
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


# The shapes that the plan was measured at (see scan_cost; calls of the shorter ones run as one launch, and have these cuts where a
# profiling call cuts them in two): use, heads, KV heads, batch, context, (tile, parts) chosen
MEASURED = [
    (P.STEP, 32, 8, 1, 4000, (2048, 4)), (P.STEP, 32, 8, 1, 16384, (2048, 4)), (P.STEP, 32, 8, 1, 20000, (2048, 2)),
    (P.STEP, 32, 8, 1, 24576, (2048, 2)), (P.STEP, 32, 8, 1, 32768, (4096, 4)), (P.STEP, 32, 8, 1, 32771, (4096, 2)),
    (P.STEP, 32, 8, 1, 65540, (4096, 1)), (P.STEP, 32, 8, 1, 100000, (4096, 1)), (P.STEP, 32, 8, 2, 20011, (4096, 2)),
    (P.STEP, 32, 8, 4, 8000, (2048, 2)), (P.STEP, 32, 8, 8, 4000, (2048, 2)), (P.STEP, 32, 8, 4, 60000, (4096, 1)),
    (P.STEP, 32, 8, 16, 17408, (2048, 1)), (P.STEP, 32, 8, 16, 32768, (4096, 1)), (P.STEP, 32, 8, 41, 2560, (2048, 1)),
    (P.STEP, 32, 8, 48, 6001, (2048, 1)), (P.STEP, 32, 32, 1, 32768, (2048, 1)), (P.STEP, 32, 32, 4, 32768, (4096, 1)),
    (P.TOPK, 32, 8, 1, 4000, (1024, 4)), (P.TOPK, 32, 8, 2, 20011, (4096, 2)), (P.TOPK, 32, 8, 16, 3000, (2048, 1)),
    (P.DISTANCES, 16, 8, 4, 8000, (1024, 1)),
]


@pytest.mark.parametrize("use,heads,kv,batch,L,chosen", MEASURED)
def test_the_cut_that_was_measured_as_the_best_is_the_one_chosen(use, heads, kv, batch, L, chosen):
    c = P.cut(P.config(heads, kv), batch, L, use)
    assert (c.tile, c.parts) == chosen


def test_cuts_of_spilling_instances():
    three = dict(code_bits=3, thr_k=(-1.5, -1.0, -0.5, 0.0, 0.5, 1.0, 1.5), head_dim=256)
    c = P.cut(P.config(32, 32, **three), 1, 32771)
    assert (c.tile, c.parts) == (2048, 1)


def test_a_group_that_cannot_be_shared_evenly_has_no_heads_per_part():
    assert [P.heads_per_part(8, s) for s in range(4)] == [8, 4, 2, 1]
    assert [P.heads_per_part(6, s) for s in range(4)] == [6, 3, 0, 0]
    assert P.heads_per_part(1, 1) == P.heads_per_part(8, -1) == P.heads_per_part(8, 4) == 0


def test_the_launcher_takes_only_cuts_that_have_a_kernel():
    """Asked without a GPU and for cuts that do not exist: false, and no launch is tried."""
    lib = A.library()
    of = getattr(lib, "_ZN6adamas10kernel_setILi128ELi0EEERKNS_9KernelSetEv")
    of.restype = ctypes.c_void_p
    # the table's first entry; a dim3 (three 32-bit words) travels as two 64-bit words
    address = ctypes.cast(of(), ctypes.POINTER(ctypes.c_void_p))[0]
    scan = ctypes.CFUNCTYPE(ctypes.c_bool, ctypes.c_bool, ctypes.c_int, ctypes.c_int, ctypes.c_uint64, ctypes.c_uint64,
                            ctypes.c_void_p, ctypes.c_void_p)(address)
    params = (ctypes.c_char * 4096)()
    for fused in (False, True):
        for heads, tile in [(0, 2048), (9, 2048), (-1, 4096), (16, 1024), (1, 0), (4, 512), (8, 8192)]:
            assert scan(fused, heads, tile, 1 | 1 << 32, 1, None, params) is False, (fused, heads, tile)
    for heads in range(1, 9):           # the step's smallest tiles are of 2048 tokens
        assert scan(True, heads, 1024, 1 | 1 << 32, 1, None, params) is False, heads


@pytest.mark.parametrize("heads,k,d,parts", [
    (1, 128, 128, 1), (1, 129, 128, 5), (63, 256, 128, 8), (64, 129, 128, -1), (64, 256, 128, -1), (64, 257, 128, 9), (128, 512, 128, 8),
    (192, 1024, 128, -1), (192, 1025, 128, 8), (207, 2047, 64, 8), (208, 2047, 64, -1), (256, 2047, 256, -1), (192, 4096, 128, 8),
    (256, 2048, 64, 8), (256, 4096, 256, 8), (257, 300, 128, 8), (512, 512, 128, 1), (256, 64, 64, 1)])
def test_workgroups_of_the_stand_alone_attention(heads, k, d, parts):
    assert P.sparse_parts(heads, k, d) == parts
