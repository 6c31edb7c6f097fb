"""The binding's native argument marshalling against its own checks: what it takes gives the same results, what it does not
take is refused, or accepted, by the checks as if it were not there."""

import pytest
import torch

import paper_2510_18413_amd as A
from paper_2510_18413_amd import binding


def test_it_is_built_and_takes_nothing_that_is_not_a_gpu_tensor():
    A.library()
    m = binding._marshal
    assert m is not None
    cfg = A.Config.make(4, 2, 64)
    x, codes = torch.zeros(2, 64, 128, dtype=torch.bfloat16), torch.zeros(2, 64, 32, dtype=torch.uint8)
    assert m.encode_keys(cfg, x, codes, 0, 64, None) is None           # host memory
    assert m.encode_keys(cfg, None, codes, 0, 64, None) is None
    assert m.encode_keys(b"x" * 88, x, codes, 0, 64, None) is None     # not a Config
    assert m.encode_keys(cfg, x) is None
    assert m.decode_step(*([cfg] + [None] * 14)) is None
    assert m.decode_step_paged(*([cfg] + [x] * 16)) is None
    assert m.full_attn(*([cfg] + [3] * 9)) is None
    with pytest.raises(ValueError, match="K must live on the GPU"):
        A.adamas_encode_keys(cfg, x, codes, 0, 64)
    with pytest.raises(ValueError, match="q must live on the GPU"):
        A.adamas_decode_step(cfg, x[:1, :4].contiguous(), None, x, codes, None, None, 4, x, 64, codes)


def _call(L=300, k=40, page=64):
    gen = torch.Generator().manual_seed(5)
    g = lambda *s: torch.randn(*s, generator=gen).to(torch.bfloat16).cuda()
    pool = 320
    cfg = A.Config.make(4, 2, pool)
    c = dict(cfg=cfg, q=g(1, 4, 128), K=g(2, pool, 128), V=g(2, pool, 128),
             codes=torch.zeros(2, pool, 32, dtype=torch.uint8, device="cuda"),
             seq_start=torch.zeros(1, dtype=torch.int64, device="cuda"),
             seq_len=torch.full((1,), L, dtype=torch.int32, device="cuda"), k=k,
             out=torch.zeros(1, 4, 128, device="cuda"), max_seq_len=L,
             workspace=torch.zeros(A.adamas_workspace_bytes(cfg, 1, L, k), dtype=torch.uint8, device="cuda"),
             k_new=g(1, 2, 128), v_new=g(1, 2, 128), idx_out=torch.zeros(1, 4, k, dtype=torch.int32, device="cuda"))
    table = torch.arange(pool // page, dtype=torch.int32, device="cuda")[None].contiguous()
    return c, table, page


@pytest.mark.gpu
def test_same_results_with_and_without_it(monkeypatch):
    def every_call():
        got = []
        c, table, page = _call()
        A.adamas_encode_keys(c["cfg"], c["K"], c["codes"], 0, 320)
        got.append(c["codes"].clone())
        for stream in (None, torch.cuda.current_stream(), torch.cuda.current_stream().cuda_stream):
            A.adamas_decode_step(**c, stream=stream)
            got += [c["out"].clone(), c["idx_out"].clone(), c["K"].clone(), c["codes"].clone()]
        p = {n: v for n, v in c.items() if n != "seq_start"}
        A.adamas_decode_step_paged(**p, page_table=table, page_tokens=page)
        got += [c["out"].clone(), c["idx_out"].clone()]
        A.adamas_decode_step(**dict(c, k_new=None, v_new=None, idx_out=None))
        got.append(c["out"].clone())
        ws = torch.zeros(A.adamas_full_attn_workspace_bytes(c["cfg"], 1, 300), dtype=torch.uint8, device="cuda")
        A.adamas_full_attn(c["cfg"], c["q"], c["K"], c["V"], c["seq_start"], c["seq_len"], c["out"], 300, ws)
        got.append(c["out"].clone())
        torch.cuda.synchronize()
        return got

    A.library()
    assert binding._marshal is not None
    native = every_call()
    monkeypatch.setattr(binding, "_marshal", None)
    for a, b in zip(native, every_call()):
        assert torch.equal(a, b)


def test_a_module_that_cannot_be_had_is_said_and_done_without(monkeypatch, tmp_path):
    lib = A.library()

    def no_compiler(*a, **k):
        raise FileNotFoundError("g++")

    with monkeypatch.context() as mp:
        mp.setattr(binding._build, "MARSHAL_LIB", tmp_path / "_marshal.so")
        mp.setattr(binding._build, "build_marshal", no_compiler)
        with pytest.warns(RuntimeWarning, match="FileNotFoundError: g"):
            assert binding._load_marshal(lib) is None
    with monkeypatch.context() as mp:       # a torch without GPU support
        mp.delattr(torch._C, "_cuda_getDevice")
        with pytest.warns(RuntimeWarning, match="_cuda_getDevice"):
            assert binding._load_marshal(lib) is None
    assert binding._load_marshal(lib) is not None


def _outcomes(call, calls, monkeypatch):
    """What every call does, with the native module and without it."""
    def outcome(kw):
        try:
            call(**kw)
        except Exception as e:
            return type(e).__name__, str(e)
        return "accepted"

    assert binding._marshal is not None
    native = [outcome(kw) for kw in calls]
    with monkeypatch.context() as mp:
        mp.setattr(binding, "_marshal", None)
        without = [outcome(kw) for kw in calls]
    torch.cuda.synchronize()
    assert native == without
    return native


@pytest.mark.gpu
def test_same_refusals_of_the_other_calls_with_and_without_it(monkeypatch):
    A.library()
    c, table, page = _call()
    p = dict({n: v for n, v in c.items() if n != "seq_start"}, page_table=table, page_tokens=page)
    bad = [{}, dict(page_tokens=64.0), dict(stages=True), dict(page_table=table[0]), dict(page_table=table.long()),
           dict(page_table=table.cpu()), dict(page_table=torch.cat([table, table])), dict(page_tokens=63), dict(page_tokens=8192),
           dict(page_tokens="64"), dict(stages=2), dict(stages=-1), dict(stages=2 ** 31), dict(max_seq_len=321), dict(q=c["q"].float()),
           dict(K=c["K"][:, ::2]), dict(V=c["V"].cpu()), dict(codes=c["codes"][:, :, :16]), dict(seq_len=c["seq_len"][:0]),
           dict(idx_out=c["idx_out"][:, :, 1:].contiguous()), dict(idx_out=None, k=0), dict(idx_out=None, k=2 ** 40), dict(v_new=None),
           dict(workspace=c["workspace"][:1000]), dict(workspace=c["workspace"][1:]), dict(out=None), dict(cfg=None), dict(stream="x")]
    got = _outcomes(A.adamas_decode_step_paged, [dict(p, **b) for b in bad], monkeypatch)
    assert [i for i, g in enumerate(got) if g == "accepted"] == [0, 1, 2, 9]

    e = dict(cfg=c["cfg"], K=c["K"], codes=c["codes"], row_begin=0, n_rows=320)
    bad = [{}, dict(row_begin=True), dict(n_rows=0), dict(K=None), dict(K=c["K"].float()), dict(K=c["K"].transpose(0, 1)), dict(K=c["K"][0]),
           dict(codes=c["codes"].cpu()), dict(codes=c["codes"][:, ::2]), dict(codes=c["codes"].view(torch.int8)), dict(n_rows=321),
           dict(row_begin=-1), dict(n_rows=-1), dict(row_begin=2 ** 70), dict(n_rows="3"), dict(cfg=b"x" * 88), dict(stream=[])]
    got = _outcomes(A.adamas_encode_keys, [dict(e, **b) for b in bad], monkeypatch)
    assert [i for i, g in enumerate(got) if g == "accepted"] == [0, 2, 13]      # (ctypes takes the low bits of a number)

    ws = torch.zeros(A.adamas_full_attn_workspace_bytes(c["cfg"], 1, 300), dtype=torch.uint8, device="cuda")
    f = dict(cfg=c["cfg"], q=c["q"], K=c["K"], V=c["V"], seq_start=c["seq_start"], seq_len=c["seq_len"], out=c["out"], max_seq_len=300,
             workspace=ws)
    bad = [{}, dict(q=c["q"][0]), dict(q=c["q"].half()), dict(K=c["K"][:1]), dict(V=None), dict(seq_start=c["seq_start"].int()),
           dict(seq_start=None), dict(seq_len=c["seq_len"].cpu()), dict(out=c["out"].double()), dict(out=c["out"].transpose(1, 2)),
           dict(max_seq_len=0), dict(max_seq_len=2 ** 21), dict(max_seq_len=3.5), dict(workspace=ws[:100]), dict(workspace=None),
           dict(workspace=ws.float()), dict(cfg="c"), dict(stream=object())]
    got = _outcomes(A.adamas_full_attn, [dict(f, **b) for b in bad], monkeypatch)
    assert [i for i, g in enumerate(got) if g == "accepted"] == [0]


@pytest.mark.gpu
def test_same_refusals_with_and_without_it(monkeypatch):
    A.library()
    c, table, page = _call()
    bad = [dict(q=c["q"].float()), dict(q=c["q"][0]), dict(K=c["K"].transpose(0, 1)), dict(K=c["K"][:, ::2]), dict(V=None),
           dict(codes=c["codes"][:1]), dict(seq_len=c["seq_len"].long()), dict(seq_start=c["seq_start"].cpu()),
           dict(idx_out=c["idx_out"][:, :, 1:].contiguous()), dict(k="4"), dict(workspace=c["workspace"][:1000]),
           dict(k=5000, idx_out=None), dict(k=0, idx_out=None), dict(max_seq_len=0), dict(k_new=None), dict(cfg=3),
           dict(out=[1.0]), dict(max_seq_len=2 ** 70), dict(k=2 ** 40, idx_out=None)]

    native = _outcomes(A.adamas_decode_step, [dict(c, **b) for b in bad], monkeypatch)
    assert native[10][0] == native[11][0] == "AdamasError"
    # a transformed tensor has no storage of its own: refused, not dereferenced
    ran = []

    def inside(q):
        with pytest.raises(Exception):
            A.adamas_decode_step(**dict(c, q=q))
        ran.append(True)
        return q

    torch.vmap(inside)(c["q"][None])
    assert ran
