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
