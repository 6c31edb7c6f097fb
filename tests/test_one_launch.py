"""The step and top-k as one launch, a workgroup per query head: the rule that chooses it, and its results against those of the
scan and select kernels (the profiling hook runs them one by one) where it can go wrong: contexts around a wave's 64 tokens, a
batch of four of them, what a thread looks at (4, 8 or 16 tokens) and a second pass; planes that do not fill a row of eight
workgroups; ties, short lists, empty sequences."""

import ctypes
import random

import pytest
import torch

import paper_2510_18413_amd as A
from plan_query import STEP, TOPK, one_launch_lib, waves

THR = {1: (0.0,), 2: (-1.0, 0.0, 1.0), 3: (-1.5, -1.0, -0.5, 0.0, 0.5, 1.0, 1.5)}


def config(heads, kv, d=128, bits=2, variant=0, pool=1 << 20):
    return A.Config.make(heads, kv, pool, thr_k=THR[bits], head_dim=d, variant=variant, code_bits=0 if bits == 2 else bits)


# heads, KV heads, sequences, context, k, use, waves
MEASURED = [(1, 1, 1, 1024, 64, STEP, 8), (32, 8, 1, 4000, 256, STEP, 16), (32, 8, 1, 8000, 128, STEP, 16), (32, 8, 1, 12000, 128, STEP, 16),
            (32, 8, 1, 16384, 128, STEP, 0), (32, 32, 1, 16384, 256, STEP, 0), (32, 8, 8, 8000, 256, STEP, 16), (32, 8, 16, 16469, 40, STEP, 8),
            (32, 8, 16, 24000, 128, STEP, 0), (32, 8, 48, 6001, 256, STEP, 4), (32, 32, 1, 32768, 256, STEP, 0),
            (32, 8, 1, 8000, 512, TOPK, 8), (32, 8, 1, 12000, 512, TOPK, 0), (32, 8, 2, 20011, 512, TOPK, 0), (32, 8, 8, 24000, 512, TOPK, 16)]


@pytest.mark.parametrize("heads,kv,batch,L,k,use,want", MEASURED)
def test_the_form_that_was_measured_as_the_best_is_chosen(heads, kv, batch, L, k, use, want):
    assert waves(config(heads, kv), batch, L, k, use) == want


# Calls that one launch takes longer for than two: head dimension, bits, heads, KV heads, sequences, context, k, page, use; us as one, as two
SLOWER = [((64, 1), (48, 8, 14, 26137, 491, 0, STEP), 57.4, 40.2), ((64, 1), (64, 8, 33, 23812, 16, 64, STEP), 76.6, 55.1),
          ((64, 2), (96, 16, 8, 27440, 355, 0, STEP), 59.4, 43.3), ((64, 2), (8, 1, 139, 21187, 25, 0, STEP), 44.8, 34.7),
          ((64, 2), (6, 2, 534, 25990, 42, 0, STEP), 178.1, 137.7), ((160, 1), (256, 32, 12, 7350, 61, 0, STEP), 86.3, 66.3),
          ((128, 1), (16, 4, 41, 25530, 331, 64, STEP), 56.2, 45.0), ((96, 1), (112, 16, 12, 16330, 41, 0, TOPK), 44.7, 26.8),
          ((96, 3), (24, 8, 1, 8925, 18, 0, TOPK), 16.8, 10.6), ((256, 2), (48, 16, 2, 15190, 910, 0, TOPK), 25.6, 17.1),
          ((160, 1), (64, 8, 5, 17395, 819, 0, TOPK), 27.5, 18.5), ((96, 3), (32, 8, 44, 7100, 394, 0, TOPK), 72.2, 50.2),
          ((96, 2), (7, 1, 408, 16330, 870, 0, TOPK), 98.4, 73.2), ((160, 2), (64, 8, 2, 13312, 36, 0, TOPK), 13.6, 10.9),
          # rows of pieces of four bytes
          ((160, 3), (4, 4, 26, 5791, 84, 0, TOPK), 21.0, 14.6), ((96, 3), (48, 8, 10, 13187, 339, 0, TOPK), 47.2, 35.1),
          ((160, 1), (3, 1, 5, 8963, 39, 0, TOPK), 9.8, 7.4), ((160, 1), (8, 8, 8, 10363, 35, 0, TOPK), 10.3, 7.7)]


@pytest.mark.parametrize("code,call,one,two", SLOWER)
def test_calls_that_one_launch_takes_longer_for_run_as_two(code, call, one, two):
    heads, kv, batch, L, k, page, use = call
    assert one > two and waves(config(heads, kv, *code), batch, L, k, use, page > 0) == 0


def test_the_rule_knows_how_many_waves_the_registers_leave_room_for():
    import kernel_resources as R
    for metric in range(4):
        for d in (64, 96, 128, 160, 192, 256):
            for fused, paged in ((True, False), (True, True), (False, False)):
                k = R.kernels()["one_launch_kernel<8, %s, %d, %s, %d>" % (str(fused).lower(), metric, str(paged).lower(), d)]
                assert one_launch_lib().one_launch_waves_per_simd(int(fused), metric, d) <= R.waves_per_simd(k), (metric, d, fused, k)


def test_a_launch_never_asks_for_more_lds_than_it_may_have_or_a_grid_that_does_not_exist():
    for d, bits, variant in [(64, 1, 0), (128, 2, 0), (128, 2, A.VARIANT_L2), (256, 3, 0), (256, 2, A.VARIANT_L2)]:
        for heads, kv in [(1, 1), (32, 8), (64, 64)]:
            c = config(heads, kv, d, bits, variant)
            for batch in (1, 7, 40, 1000):
                for L in (1, 900, 7000, 15000, 19999, 26000, 1 << 20):
                    for k in (1, 500, 4096):
                        for use, paged in ((STEP, False), (STEP, True), (TOPK, False)):
                            w = waves(c, batch, L, k, use, paged)
                            assert w in (0, 4, 8, 16)
                            assert w == 0 or one_launch_lib().one_launch_lds(ctypes.byref(c), w, ctypes.c_int64(L), k, use, int(paged)) <= 65536
    assert waves(config(64, 64), 65535, 100, 10) == 0                    # 4 Mi planes
    assert waves(config(32768, 32768), 16, 100, 10) == 0                 # a plane times the KV heads beyond 2^32
    assert waves(config(64, 64), 8191, 100, 10) == 4


def test_no_call_of_32768_tokens_runs_as_one_launch():
    """What tests of the two kernels give as max_seq_len when their sequences are shorter."""
    for d in (64, 96, 128, 160, 192, 256):
        for bits, variant in ((1, 0), (2, 0), (2, A.VARIANT_L2), (3, 0)):
            for heads, kv in ((1, 1), (8, 1), (32, 8), (64, 64)):
                for batch in (1, 9, 300):
                    for k in (1, 4096):
                        for use, paged in ((STEP, False), (STEP, True), (TOPK, False)):
                            assert waves(config(heads, kv, d, bits, variant), batch, 32768, k, use, paged) == 0
                for batch, L in ((1, 10240), (3, 10240)):           # top-k of a few heads
                    assert batch * heads > 17 or waves(config(heads, kv, d, bits, variant), batch, L, 300, TOPK) == 0


class Case:
    """A cache on the GPU, contiguous and (page > 0) paged, with the same rows."""

    def __init__(self, heads, kv, lens, d=128, bits=2, variant=0, k=40, append=True, page=0, bound=0, seed=1):
        gen, r = torch.Generator().manual_seed(seed), random.Random(seed)
        G, nb = heads // kv, len(lens)
        g = lambda *s: torch.randn(*s, generator=gen)
        starts, at = [], 0
        for n in lens:
            starts.append(at)
            at += n + 9
        at = max(at, 64) + 55 & ~15
        self.cfg, self.k, self.d, self.lens = config(heads, kv, d, bits, variant, pool=at), k, d, lens
        K = g(kv, at, d)
        q = g(nb, heads, d)
        for b, n in enumerate(lens):        # rows near the queries
            for h in range(heads):
                if n > 1:
                    K[h // G, starts[b] + r.randrange(n - 1)] = q[b, h] + 0.1 * g(d)
        to = lambda x: x.to(torch.bfloat16).cuda()
        self.K, self.V, self.q = to(K), to(g(kv, at, d)), to(q)
        self.k_new, self.v_new = (to(g(nb, kv, d)), to(g(nb, kv, d))) if append else (None, None)
        self.starts = torch.tensor(starts, dtype=torch.int64, device="cuda")
        self.L = torch.tensor(lens, dtype=torch.int32, device="cuda")
        self.bound = max(bound, max(lens), 1)
        self.codes = torch.zeros(kv, at, self.cfg.code_row_bytes, dtype=torch.uint8, device="cuda")
        A.adamas_encode_keys(self.cfg, self.K, self.codes, 0, at)
        self.ws = torch.full((A.adamas_workspace_bytes(self.cfg, nb, self.bound, k),), 0xA5, dtype=torch.uint8, device="cuda")
        self.page = page
        if page:
            need = [max(1, -(-n // page)) for n in lens]
            order = list(range(sum(need)))
            r.shuffle(order)
            table = torch.full((nb, -(-self.bound // page)), -1, dtype=torch.int32)
            rows = torch.zeros(sum(need) * page, dtype=torch.long)
            for b, n in enumerate(lens):
                for p in range(need[b]):
                    table[b, p] = order.pop()
                for t in range(n):
                    rows[int(table[b, t // page]) * page + t % page] = starts[b] + t
            rows = rows.cuda()
            self.table = table.cuda()
            self.paged_cfg = config(heads, kv, d, bits, variant, pool=rows.numel())
            self.paged = [x[:, rows].contiguous() for x in (self.K, self.V, self.codes)]
            self.rows = rows

    def buffers(self):
        nb, heads = len(self.lens), self.cfg.num_q_heads
        return (torch.full((nb, heads, self.d), float("nan"), device="cuda"),
                torch.full((nb, heads, self.k), -7, dtype=torch.int32, device="cuda"))

    def step(self, two):
        out, idx = self.buffers()
        K, V, codes = self.K.clone(), self.V.clone(), self.codes.clone()
        for stages in ((A.STAGE_SCAN, A.STAGE_SELECT_ATTN) if two else (A.STAGE_ALL,)):
            A.adamas_decode_step_stages(self.cfg, self.q, K, V, codes, self.starts, self.L, self.k, out, self.bound, self.ws,
                                        k_new=self.k_new, v_new=self.v_new, idx_out=idx, stages=stages)
        return out, idx, K, V, codes

    def step_paged(self):
        out, idx = self.buffers()
        A.adamas_decode_step_paged(self.paged_cfg, self.q, *self.paged, self.table, self.page, self.L, self.k, out, self.bound, self.ws,
                                   k_new=self.k_new, v_new=self.v_new, idx_out=idx)
        return out, idx

    def topk(self):
        qc = torch.zeros(len(self.lens), self.cfg.num_q_heads, self.cfg.code_row_bytes, dtype=torch.uint8, device="cuda")
        A.adamas_encode_query(self.cfg, self.q, qc)
        idx = self.buffers()[1]
        dist = torch.full((len(self.lens), self.cfg.num_q_heads, self.bound), 9999, dtype=torch.uint16, device="cuda")
        want = dist.clone()
        A.adamas_select_topk(self.cfg, qc, self.codes, self.starts, self.L, self.k, idx, self.bound, self.ws, dist_out=dist)
        A.adamas_manhattan_distance(self.cfg, qc, self.codes, self.starts, self.L, want)
        return idx, dist, want


FORMS = [
    # lengths around a step of a wave, a batch of four, the tokens of a thread (4, 8, 16) and a second pass of each wave count
    dict(heads=1, kv=1, lens=[1], k=3), dict(heads=1, kv=1, lens=[63], k=64), dict(heads=2, kv=1, lens=[64, 65, 0, 2], k=5),
    dict(heads=4, kv=1, lens=[2047, 2048, 2049, 512], k=64), dict(heads=4, kv=2, lens=[4096, 4097, 1025], k=33),
    dict(heads=3, kv=1, lens=[8192, 8193], k=100), dict(heads=8, kv=1, lens=[4095, 4099], k=600), dict(heads=5, kv=1, lens=[8193, 9000], k=700),
    dict(heads=32, kv=8, lens=[1024 * 4 + 1] * 20, k=16), dict(heads=24, kv=8, lens=[1023, 1024, 1025, 2049, 7] * 6, k=20),
    dict(heads=64, kv=8, lens=[5000, 4096, 1, 0] * 3, k=9), dict(heads=2, kv=2, lens=[12001], k=12),
    # sixteen waves beyond 16384 tokens: two passes of 16 tokens a thread
    dict(heads=64, kv=16, lens=[17001, 16385, 16384, 3], k=80, append=False),
    # short lists, all rows, more than all rows, the longest list, a bound far above the lengths
    dict(heads=6, kv=2, lens=[300, 41], k=1), dict(heads=6, kv=2, lens=[300, 41], k=300), dict(heads=2, kv=1, lens=[4500], k=4096),
    dict(heads=4, kv=4, lens=[70, 300], k=400, bound=9000), dict(heads=7, kv=1, lens=[130, 129], k=64, append=False),
    # head dimensions, code formats and estimators
    *[dict(heads=4, kv=2, lens=[1500, 777], d=d, bits=bits, variant=v, k=50, append=ap)
      for d in (64, 96, 128, 160, 192, 256)
      for bits, v, ap in ((2, 0, True), (1, 0, False), (3, 0, True), (2, A.VARIANT_L2, True), (2, A.VARIANT_NO_HADAMARD, False))],
    dict(heads=8, kv=1, lens=[9000], d=64, bits=1, k=2000), dict(heads=4, kv=4, lens=[3000] * 3, d=256, variant=A.VARIANT_L2, k=700),
    # many heads: four waves
    dict(heads=64, kv=8, lens=[200 + 37 * i for i in range(11)], k=31), dict(heads=64, kv=64, lens=[1025, 64, 2000] * 4, d=96, k=77),
    # paged
    dict(heads=4, kv=2, lens=[64, 65, 1, 0], k=20, page=64), dict(heads=8, kv=2, lens=[4097, 2000], k=128, page=64),
    dict(heads=3, kv=1, lens=[9001], d=64, k=300, page=256), dict(heads=64, kv=8, lens=[700, 64, 1] * 5, k=90, page=128),
    dict(heads=4, kv=4, lens=[2500, 3], d=192, bits=3, k=60, page=64, append=False),
]


@pytest.mark.gpu
@pytest.mark.parametrize("form", FORMS, ids=lambda f: " ".join("%s=%s" % (a, b if a != "lens" else "%d..%d" % (len(b), max(b))) for a, b in f.items()))
def test_one_launch_gives_what_two_give(form):
    c = Case(**form)
    nb = len(c.lens)
    assert waves(c.cfg, nb, c.bound, c.k)
    want = c.step(two=True)
    got = c.step(two=False)
    assert torch.equal(got[1], want[1])
    # fp32 weights and sums in another order: 1e-6 of the output's norm per head is several times what they show
    err = (got[0] - want[0]).norm(dim=-1) / want[0].norm(dim=-1).clamp(min=1e-30)
    assert err.max().item() <= 1e-6
    for a, b in zip(got[2:], want[2:]):
        assert torch.equal(a, b)
    idx, dist, all_dist = c.topk()
    live = [b for b, n in enumerate(c.lens) if n]
    assert torch.equal(dist.view(torch.int16), all_dist.view(torch.int16))   # and nothing beyond the lengths
    if c.k_new is None:
        assert torch.equal(idx, want[1])
    else:                                   # the cache before the append: against the distances
        for b in live:
            order = all_dist[b, :, :c.lens[b]].to(torch.int32).sort(dim=-1, stable=True).indices[:, :c.k].sort(dim=-1).values
            assert torch.equal(idx[b, :, :order.shape[1]], order.to(torch.int32))
            assert (idx[b, :, order.shape[1]:] == -1).all()
    if c.page:
        assert waves(c.paged_cfg, nb, c.bound, c.k, paged=True)
        out, idx = c.step_paged()
        assert torch.equal(idx, want[1])
        err = (out - want[0]).norm(dim=-1) / want[0].norm(dim=-1).clamp(min=1e-30)
        assert err.max().item() <= 1e-6
        for b, n in enumerate(c.lens):      # the rows are where the table says
            t = torch.arange(n, device="cuda")
            at = c.table[b].long()[t // c.page] * c.page + t % c.page
            for paged, flat in zip(c.paged, want[2:]):
                assert torch.equal(paged[:, at], flat[:, int(c.starts[b]):int(c.starts[b]) + n])


@pytest.mark.gpu
def test_ties_infinite_elements_and_lengths_that_do_not_fit():
    """Every distance the same: the lowest positions.  A row with an infinity among the selected gives the same as two launches, and a
    length beyond the bound, or a start outside the pool, counts as empty."""
    c = Case(heads=4, kv=2, lens=[700, 90], k=130, append=False)
    c.codes.zero_()
    out, idx = c.step(two=False)[:2]
    assert torch.equal(idx[0], torch.arange(130, dtype=torch.int32, device="cuda").expand(4, 130))
    assert torch.equal(idx[1, :, :90], torch.arange(90, dtype=torch.int32, device="cuda").expand(4, 90)) and (idx[1, :, 90:] == -1).all()
    c.V[0, 5, 3] = float("inf")
    c.K[1, 7, 2] = float("-inf")
    got, want = c.step(two=False)[0], c.step(two=True)[0]
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    c.L[0] = 701                            # beyond the bound
    c.starts[1] = -1
    got, idx = c.step(two=False)[:2]
    assert (got == 0).all() and (idx == -1).all()


@pytest.mark.gpu
def test_replays_of_a_graph_and_two_streams():
    """No scratch: calls on two streams at once, with one workspace between them, and replays, all give the same."""
    c = Case(heads=8, kv=2, lens=[2000, 1500, 64], k=90)
    want = c.step(two=False)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    K, V, codes = c.K.clone(), c.V.clone(), c.codes.clone()
    bufs = [c.buffers() for _ in streams]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for _ in range(10):
        for s, (out, idx) in zip(streams, bufs):
            A.adamas_decode_step(c.cfg, c.q, K, V, codes, c.starts, c.L, c.k, out, c.bound, c.ws, k_new=c.k_new, v_new=c.v_new,
                                 idx_out=idx, stream=s)
    torch.cuda.synchronize()
    for out, idx in bufs:
        assert torch.equal(out, want[0]) and torch.equal(idx, want[1])
    out, idx = c.buffers()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        A.adamas_decode_step(c.cfg, c.q, K, V, codes, c.starts, c.L, c.k, out, c.bound, c.ws, k_new=c.k_new, v_new=c.v_new, idx_out=idx)
    for _ in range(4):
        out.zero_(), idx.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[0]) and torch.equal(idx, want[1])
