"""The native argument checks of the binding: what they leave to the general
path (CPU), and that both paths give the same results and errors (GPU)."""

import ctypes

import numpy as np
import pytest
import torch

from paper_2608_08081_amd import _lib, api


def test_everything_else_goes_to_the_general_path():
    nat = _lib.native()
    t = torch.zeros(1, 16, 128)
    for fn, n in (("compress", 9), ("decode", 12), ("step", 15), ("decode_paged", 12),
                  ("step_paged", 15), ("multi", 12), ("step_multi", 15), ("rope", 13),
                  ("dequantize", 10)):
        f = getattr(nat, fn)
        assert f(*[None] * n) is None            # nothing given
        assert f(*[t] * n) is None               # host tensors
        assert f(*[object()] * n) is None
        assert f() is None and f(t) is None      # too few


def _case(b=2, hkv=2, group=8, cap=64, dev="cuda:0"):
    g = torch.Generator(device=dev).manual_seed(3)
    c = api.alloc_cache(b, hkv, cap, dev)
    quats = api.iq_make_rotation(9, hkv).to(dev)
    x = torch.randn((b, hkv, 40, 128), generator=g, device=dev).half()
    api.iq_compress_kv(x, x.flip(2).contiguous(), quats, c["k_codes"], c["k_norms"], c["v_codes"],
                       c["v_norms"])
    c["seq_lens"].fill_(40)
    q = torch.randn((b, hkv * group, 128), generator=g, device=dev)
    k = torch.randn((b, hkv, 128), generator=g, device=dev).half()
    return c, quats, q, k, torch.empty_like(q), api.alloc_workspace(b, hkv * group, hkv, cap, dev)


@pytest.mark.gpu
def test_both_paths_agree(monkeypatch):
    c, quats, q, k, out, ws = _case()
    rows = (c["k_codes"], c["k_norms"], c["v_codes"], c["v_norms"], c["seq_lens"], quats)

    class General:   # the native module that never calls
        def __getattr__(self, name):
            return lambda *a: None

    got = []
    for general in (False, True):
        if general:
            monkeypatch.setattr(_lib, "native", lambda: General())
        c["seq_lens"].fill_(40)
        a = api.iq_decode_attention(q, *rows, out=out, workspace=ws).clone()
        s = api.iq_decode_step(q, k, k, *rows, out=out, workspace=ws).clone()
        d = api.iq_dequantize_kv(*rows[:4], quats, k_out=torch.empty((2, 2, 64, 128), device="cuda:0",
                                                                      dtype=torch.float16),
                                 v_out=torch.empty((2, 2, 64, 128), device="cuda:0",
                                                   dtype=torch.float16))
        got.append((a, s, *d, c["seq_lens"].clone(), c["k_codes"].clone()))
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("wrong,error", [
    ({"q": lambda t: t.half()}, TypeError), ({"q": lambda t: t[:, :, :64]}, ValueError),
    ({"k": lambda t: t.bfloat16()}, TypeError), ({"k": lambda t: t.cpu()}, ValueError),
    ({"out": lambda t: t.transpose(0, 1)}, ValueError), ({"ws": lambda t: t.float()}, ValueError),
    ({"ws": lambda t: t[:256]}, _lib.IsoQuantError), ({"quats": lambda t: t[:1]}, ValueError),
    ({"lens": lambda t: t.long()}, TypeError), ({"most": lambda m: 65}, _lib.IsoQuantError),
])
def test_wrong_arguments_raise_as_before(wrong, error):
    c, quats, q, k, out, ws = _case()
    a = dict(q=q, k=k, quats=quats, out=out, ws=ws, lens=c["seq_lens"], most=None)
    before = c["k_codes"].clone()
    for name, f in wrong.items():
        a[name] = f(a[name])
    with pytest.raises(error):
        api.iq_decode_step(a["q"], a["k"], a["k"], c["k_codes"], c["k_norms"], c["v_codes"],
                           c["v_norms"], a["lens"], a["quats"], out=a["out"], workspace=a["ws"],
                           max_seq_len=a["most"])
    assert torch.equal(before, c["k_codes"])


@pytest.mark.gpu
def test_calls_go_to_the_current_stream():
    c, quats, q, k, out, ws = _case()
    args = (q, c["k_codes"], c["k_norms"], c["v_codes"], c["v_norms"], c["seq_lens"], quats)
    want = api.iq_decode_attention(*args, out=out, workspace=ws).clone()
    torch.cuda.synchronize()
    side, out2 = torch.cuda.Stream(), torch.zeros_like(out)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        api.iq_decode_attention(*args, out=out2, workspace=ws)
    assert not np.any(out2.cpu().numpy())   # captured, not run
    for _ in range(3):
        out2.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out2, want)


class _General:   # a native module that never calls
    def __getattr__(self, name):
        return lambda *a: None


def _paged_case(b=3, hkv=2, page=16, per=4, dev="cuda:0"):
    c, quats, q, k, out, ws = _case(b, hkv, 8, page * per)
    pool = api.alloc_paged_cache(b * per, hkv, page, dev)
    for name, x in pool.items():   # page i of sequence s: s * per + i
        y = c[name].view(b, hkv, per, page, *c[name].shape[3:]).transpose(1, 2)
        x.copy_(y.reshape(x.shape))
    tables = torch.arange(b * per, dtype=torch.int32, device=dev).view(b, per)
    return c, pool, tables, quats, q, k, out, ws


@pytest.mark.gpu
@pytest.mark.parametrize("general", [False, True])
def test_page_tables_need_a_row_per_sequence(general, monkeypatch):
    """Fewer rows than sequences are refused before anything runs; more are allowed."""
    c, pool, tables, quats, q, k, out, ws = _paged_case()
    if general:
        monkeypatch.setattr(_lib, "native", lambda: _General())
    lens = c["seq_lens"]
    want = api.iq_decode_attention(q, c["k_codes"], c["k_norms"], c["v_codes"], c["v_norms"], lens,
                                   quats).clone()
    more = torch.cat((tables, torch.full((2, tables.shape[1]), 1 << 30, dtype=torch.int32,
                                         device=tables.device)))
    for t in (tables, more):
        assert torch.equal(want, api.iq_decode_attention_paged(q, pool, t, lens, quats, out=out,
                                                               workspace=ws))
    before = {n: x.clone() for n, x in pool.items()}
    qs = torch.stack((q, q), 1)
    for t in (tables[:2], tables[:0]):
        for call in (lambda: api.iq_decode_attention_paged(q, pool, t, lens, quats, out=out,
                                                           workspace=ws),
                     lambda: api.iq_decode_step_paged(q, k, k, pool, t, lens, quats, out=out,
                                                      workspace=ws),
                     lambda: api.iq_decode_attention_multi_paged(qs, pool, t, lens, quats)):
            with pytest.raises(ValueError, match="rows for 3 sequences"):
                call()
    assert lens.tolist() == [40] * 3
    assert all(torch.equal(x, before[n]) for n, x in pool.items())


@pytest.mark.gpu
def test_an_exception_out_of_the_call_is_an_error():
    """Bound to a function that throws: the call raises, with the interpreter lock held, and is
    not made a second time by the general path."""
    c, quats, q, k, out, ws = _case()
    throw = ctypes.cast(getattr(ctypes.CDLL("libstdc++.so.6"), "_ZSt17__throw_bad_allocv"),
                        ctypes.c_void_p).value
    nat = _lib.native()
    out.fill_(7.0)
    try:
        nat.bind(*[throw] * len(_lib._BOUND))
        with pytest.raises(RuntimeError, match="bad_alloc"):
            api.iq_decode_step(q, k, k, c["k_codes"], c["k_norms"], c["v_codes"], c["v_norms"],
                               c["seq_lens"], quats, out=out, workspace=ws)
    finally:
        nat.bind(*(ctypes.cast(getattr(_lib.lib(), n), ctypes.c_void_p).value
                   for n in _lib._BOUND))
    torch.cuda.synchronize()
    assert torch.all(out == 7.0) and c["seq_lens"].tolist() == [40, 40]
    api.iq_decode_step(q, k, k, c["k_codes"], c["k_norms"], c["v_codes"], c["v_norms"],
                       c["seq_lens"], quats, out=out, workspace=ws)
    assert c["seq_lens"].tolist() == [41, 41]



def test_without_the_native_module_every_call_takes_the_general_path(monkeypatch):
    import sys

    import paper_2608_08081_amd as package
    monkeypatch.setattr(_lib, "_native", None)
    monkeypatch.delattr(package, "_bind", raising=False)
    monkeypatch.setitem(sys.modules, package.__name__ + "._bind", None)
    with pytest.warns(RuntimeWarning, match="_bind.so does not load"):
        nat = _lib.native()
    assert nat.decode(*[None] * 12) is None and _lib.native() is nat
    with pytest.raises(ValueError):   # reported by the general path
        api.iq_decode_attention(torch.zeros(1, 8, 64), *[torch.zeros(1)] * 6)


def _calls():
    """Every entry point of the native module: name -> (function, its arguments)."""
    c, pool, tables, quats, q, k, out, ws = _paged_case()
    b, hkv, cap = c["k_norms"].shape
    rows = dict(k_codes=c["k_codes"], k_norms=c["k_norms"], v_codes=c["v_codes"],
                v_norms=c["v_norms"])
    at = dict(seq_lens=c["seq_lens"], quats=quats)
    dev = q.device
    g = torch.Generator(device=dev).manual_seed(4)
    q2 = torch.randn((b, 2, 16, 128), generator=g, device=dev)
    k2 = torch.randn((b, 2, hkv, 128), generator=g, device=dev)
    ws2 = torch.empty(api.iq_decode_multi_workspace_bytes(b, 2, 16, hkv, cap), dtype=torch.uint8,
                      device=dev)
    x = torch.randn((b, hkv, 9, 128), generator=g, device=dev)
    io = dict(out=out, workspace=ws)
    io2 = dict(out=torch.empty_like(q2), workspace=ws2)
    flag = torch.zeros(1, dtype=torch.int32, device=dev)
    kv = torch.empty((b, hkv, cap, 128), dtype=torch.float16, device=dev)
    n = {}
    n["compress"] = (api.iq_compress_kv, dict(k=x, v=x, quats=quats, **rows, dst_offset=48))
    n["decode"] = (api.iq_decode_attention, dict(q=q, **rows, **at, **io))
    n["step"] = (api.iq_decode_step, dict(q=q, k_new=k, v_new=k, **rows, **at, **io, status=flag))
    n["paged"] = (api.iq_decode_attention_paged, dict(q=q, pool=pool, block_tables=tables, **at,
                                                      **io))
    n["step_paged"] = (api.iq_decode_step_paged, dict(q=q, k_new=k, v_new=k, pool=pool,
                                                      block_tables=tables, **at, **io,
                                                      status=flag))
    n["multi"] = (api.iq_decode_attention_multi, dict(q=q2, **rows, **at, **io2))
    n["step_multi"] = (api.iq_decode_step_multi, dict(q=q2, k_new=k2, v_new=k2, **rows, **at,
                                                      **io2, status=flag))
    n["rope"] = (api.iq_decode_attention_rope, dict(
        q=q, q_rope=torch.randn((b, 16, 64), generator=g, device=dev), **rows,
        k_rope=torch.randn((b, 1, cap, 64), generator=g, device=dev).half(), **at, **io))
    n["dequantize"] = (api.iq_dequantize_kv, dict(**rows, quats=quats, k_out=kv,
                                                  v_out=torch.empty_like(kv)))
    return n, (c["k_codes"], c["k_norms"], c["v_codes"], c["v_norms"], c["seq_lens"], flag,
               *pool.values())


ENTRIES = ("compress", "decode", "step", "paged", "step_paged", "multi", "step_multi", "rope",
           "dequantize")


@pytest.mark.gpu
@pytest.mark.parametrize("name", ENTRIES)
def test_every_entry_point_agrees_with_the_general_path(name, monkeypatch):
    got = []
    for general in (False, True):
        calls, state = _calls()
        if general:
            monkeypatch.setattr(_lib, "native", lambda: _General())
        else:   # the native path takes it
            nat, taken = _lib.native(), []

            class Watch:
                def __getattr__(self, fn):
                    return lambda *a: taken.append(getattr(nat, fn)(*a)) or taken[-1]

            monkeypatch.setattr(_lib, "native", lambda: Watch())
        f, kw = calls[name]
        r = f(**kw)
        if not general:
            assert taken == [0]
        outs = [] if r is None else ([r] if torch.is_tensor(r) else list(r))
        got.append([x.clone() for x in (*outs, *state)])
    assert len(got[0]) == len(got[1])
    for x, y in zip(*got):
        assert torch.equal(x, y)


@pytest.mark.gpu
@pytest.mark.parametrize("name", ENTRIES)
def test_wrong_tensors_of_every_entry_point(name, monkeypatch):
    """Each tensor in turn of another type, shape, layout or device: both paths raise the same
    error, and nothing is written."""
    wrong = {"type": lambda t: t.double(), "shape": lambda t: t.unsqueeze(0),
             "layout": lambda t: torch.stack((t, t), -1)[..., 0], "device": lambda t: t.cpu(),
             "kind": lambda t: t.cpu().numpy()}
    calls, state = _calls()
    f, kw = calls[name]
    before = [x.clone() for x in state]
    native = _lib.native
    seen = 0
    for arg, t in kw.items():
        for key in (t if isinstance(t, dict) else [None]):
            x = t[key] if key else t
            if not torch.is_tensor(x):
                continue
            for how, change in wrong.items():
                if arg == "workspace" and how in ("shape", "kind"):
                    continue   # any shape of bytes will do
                if name in ("paged", "step_paged", "rope") and arg == "workspace":
                    continue   # (these take it as it is)
                if how == "layout" and x.numel() == 1:
                    continue   # one value is contiguous whatever its stride
                bad = dict(kw)
                bad[arg] = {**t, key: change(x)} if key else change(x)
                errors = []
                for general in (False, True):
                    monkeypatch.setattr(_lib, "native", (lambda: _General()) if general else native)
                    with pytest.raises((TypeError, ValueError, AttributeError,
                                        _lib.IsoQuantError)) as e:
                        f(**bad)
                    errors.append((e.type, str(e.value)))
                assert errors[0] == errors[1], (arg, how)
                seen += 1
    assert seen > 20
    torch.cuda.synchronize()
    assert all(torch.equal(x, y) for x, y in zip(before, state))
