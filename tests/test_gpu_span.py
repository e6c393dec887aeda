"""GPU parity of the span kernel (decode and fused step on long lines of work:
rows of every sequence cut into equal runs, one per workgroup) against the
oracle: lengths around every chunk, wave and batch edge, empty sequences, runs
that hold several rows and rows that cross runs, 2-, 3- and 4-bit records,
pages, head groups other than 8, and a single long sequence among empty ones."""

import os
import re

import numpy as np
import pytest
import torch

from oracle import attention as oatt
from oracle import codebook as ocb
from oracle import compress as ocz
from oracle import rotation as orot
from paper_2608_08081_amd import api
from paper_2608_08081_amd import build as B
from tests.parity import row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")

# Scores carry the query as fp16 hi + lo pairs: off by at most 2^-21 of |q||k|
# scale, below 64 in log2 units here, so weights by ln 2 * 64 * 2^-21 = 2.1e-5;
# weights themselves are cut after 20 bits.
RTOL = 5e-5

EDGES = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 511, 512, 513, 640, 1023, 1024, 1025]


def _records(rng, shape, bits):
    """Random records (every code equally often) and scales."""
    return (rng.integers(0, 256, size=(*shape, 16 * bits), dtype=np.uint8),
            (14.0 * np.exp(0.35 * rng.standard_normal(shape))).astype(np.float32))


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _lengths(kind, batch, cap):
    if kind == "edges":
        return [EDGES[i % len(EDGES)] if i % 2 else (977 * i) % (cap - 1) for i in range(batch)]
    if kind == "full":
        return [cap - 1] * batch
    return [cap - 1 if i == batch // 2 else 0 for i in range(batch)]   # "one"


def _check(rng, seq, bits, group, page, step, hkv, cap):
    """One decode or fused step of sequences of these lengths against the oracle."""
    batch = len(seq)
    kc, kn = _records(rng, (batch, hkv, cap), bits)
    vc, vn = _records(rng, (batch, hkv, cap), bits)
    quats = orot.make_quaternions(77, hkv)
    levels, thr = ocb.isoquant_codebook(128, bits)
    q = rng.standard_normal((batch, hkv * group, 128), dtype=np.float32)
    k_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32)
    v_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32)
    gk, gkn, gv, gvn = kc.copy(), kn.copy(), vc.copy(), vn.copy()
    for i, n in enumerate(seq):   # a read of a position that is not attended shows up
        gkn[i, :, n:] = np.nan
        gvn[i, :, n:] = np.nan
    lens = _dev(np.asarray(seq, np.int32))
    ws = api.alloc_workspace(batch, hkv * group, hkv, cap, DEV)
    ws.fill_(0x44)
    if page:
        per = cap // page
        table = rng.permutation(batch * per).astype(np.int32).reshape(batch, per)
        cache = {}
        for nm, x in (("k_codes", gk), ("k_norms", gkn), ("v_codes", gv), ("v_norms", gvn)):
            pool = np.empty((batch * per, hkv, page, *x.shape[3:]), x.dtype)
            pool[table.reshape(-1)] = np.moveaxis(
                x[:, :, :per * page].reshape(batch, hkv, per, page, *x.shape[3:]), 2, 1).reshape(
                    batch * per, hkv, page, *x.shape[3:])
            cache[nm] = _dev(pool)
        tab = _dev(table)
        assert max(seq) < per * page
    else:
        cache = {"k_codes": _dev(gk), "k_norms": _dev(gkn), "v_codes": _dev(gv),
                 "v_norms": _dev(gvn)}
    args = (cache["k_codes"], cache["k_norms"], cache["v_codes"], cache["v_norms"], lens,
            _dev(quats))
    if step and page:
        out = api.iq_decode_step_paged(_dev(q), _dev(k_new), _dev(v_new), cache, tab, lens,
                                       _dev(quats), workspace=ws)
    elif step:
        out = api.iq_decode_step_bits(_dev(q), _dev(k_new), _dev(v_new), *args, workspace=ws,
                                      bits=bits)
    elif page:
        out = api.iq_decode_attention_paged(_dev(q), cache, tab, lens, _dev(quats), workspace=ws)
    else:
        out = api.iq_decode_attention_bits(_dev(q), *args, workspace=ws, bits=bits)
    torch.cuda.synchronize()
    if step:
        assert lens.cpu().tolist() == [n + 1 for n in seq]
        rots = orot.rotation_matrices(quats)
        pk, nk, *_ = ocz.compress_kv(k_new[:, :, None], rots, thr)
        pv, nv, *_ = ocz.compress_kv(v_new[:, :, None], rots, thr)
        for i, n in enumerate(seq):
            kc[i, :, n], kn[i, :, n] = pk[i, :, 0], nk[i, :, 0]
            vc[i, :, n], vn[i, :, n] = pv[i, :, 0], nv[i, :, 0]
    ref = oatt.decode_fused(q, kc, kn, vc, vn, [n + step for n in seq], quats, levels)
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got))
    err = row_rel_err(got, ref)
    print(f"[span] max row rel err {err.max():.3e}", flush=True)
    assert err.max() <= RTOL


@pytest.mark.parametrize("bits,group,kind,page,step", [
    (3, 8, "edges", 0, True), (3, 8, "edges", 0, False), (3, 8, "one", 0, True),
    (3, 8, "one", 0, False), (2, 8, "edges", 0, True), (4, 8, "edges", 0, True),
    (3, 4, "edges", 16, True), (3, 16, "edges", 64, False), (3, 5, "full", 0, True),
])
def test_span_against_oracle(bits, group, kind, page, step):
    hkv, cap = 2, 2112
    rows = hkv * (2 if group > 8 else 1)
    batch = -(-49152 // (rows * (cap // 16)))   # the shortest line that takes the kernel
    seq = _lengths(kind, batch, cap)
    print(f"[span] bits={bits} group={group} {kind} page={page} step={step} batch={batch}",
          flush=True)
    _check(np.random.default_rng([5, bits, group, page]), seq, bits, group, page, step, hkv, cap)


def _short_batches(step):
    src = open(os.path.join(B.CSRC, "iq_g8_device.h")).read()
    both = re.search(r"kShortBatches = kAppend \? (\d+) : (\d+);", src)
    return int(both.group(1 if step else 2))


def _line_of(rng, batch, batches, cap, step):
    """Lengths of `batch` sequences with `batches` 16-position batches in all, empty ones and every
    remainder among them."""
    nb = rng.multinomial(batches, rng.dirichlet(np.full(batch, 4.0)))
    nb[1] += nb[0]
    nb[0] = 0
    top = (cap - 16) // 16
    while nb.max() > top:   # move what does not fit to the shortest
        i, j = int(nb.argmax()), 2 + int(nb[2:].argmin())
        nb[j] += nb[i] - top
        nb[i] = top
    n = 16 * nb - rng.integers(0, 16, size=batch)
    assert nb.sum() == batches
    return [int(max(x, 0)) for x in n]


@pytest.mark.parametrize("bits,group,page,step,over", [
    (3, 8, 0, True, 0), (3, 8, 0, True, 1), (3, 8, 0, False, 0), (3, 8, 0, False, 1),
    (3, 8, 16, True, 0), (3, 8, 16, True, 1), (3, 16, 64, False, 0), (3, 16, 64, False, 1),
    (2, 8, 0, True, 0), (2, 5, 0, False, 1), (4, 8, 0, True, 1), (4, 8, 0, False, 0),
    (3, 8, 0, True, -20000), (3, 3, 32, True, -20000), (3, 8, 0, False, -12000),
])
@pytest.mark.parametrize("batch", [40, 150])
def test_lines_around_the_shortest_of_runs(bits, group, page, step, over, batch):
    """Lines of the length from which the kernel takes equal runs (over 0), the longest that takes
    fixed splits (1 batch less; over 1) and much shorter ones, in rows that could hold more."""
    hkv = 2
    rows = batch * hkv * (2 if group > 8 else 1)
    # the shortest line that takes the kernel
    cap = -(-(-(-49152 // rows) * 16 + 64) // 64) * 64
    least = 512 * 8 * _short_batches(step) // (rows // batch)
    batches = least - (over if over >= 0 else -over // (rows // batch))
    rng = np.random.default_rng([9, bits, group, page, step, abs(over), batch])
    seq = _line_of(rng, batch, batches, cap, step)
    _check(rng, seq, bits, group, page, step, hkv, cap)


@pytest.mark.parametrize("bits,group,page,step", [(3, 8, 0, True), (3, 8, 0, False),
                                                  (2, 8, 0, True), (4, 16, 0, True),
                                                  (3, 4, 16, True), (3, 8, 64, False)])
def test_runs_with_edges(bits, group, page, step):
    """Lengths around every edge among rows long enough for equal runs."""
    hkv, cap = 2, 2112
    batch = -(-49152 // (hkv * (2 if group > 8 else 1) * (cap // 16)))
    seq = [EDGES[(i // 4) % len(EDGES)] if i % 4 == 0 else cap - 1 - (37 * i) % 300
           for i in range(batch)]
    _check(np.random.default_rng([10, bits, group, page]), seq, bits, group, page, step, hkv, cap)


@pytest.mark.parametrize("batch,hkv,group,cap,step,shift", [
    (1, 1, 1, 1, True, 0), (1, 1, 1, 5, False, 0), (1, 4, 8, 17, True, 0), (3, 2, 8, 131, True, 0),
    (2, 2, 4, 777, False, 0), (5, 2, 16, 1031, True, 0), (300, 2, 8, 103, True, 0),
    (300, 2, 8, 103, False, 0), (2, 4, 8, 9191, True, 0), (7, 2, 5, 1025, True, 1),
    (3, 2, 8, 1040, True, 1), (1, 2, 8, 641, True, 3),
])
def test_rows_of_any_length(batch, hkv, group, cap, step, shift):
    """Rows that are not whole batches of 16 positions (whose last loads end with the row; the
    buffers hold nothing past the last row) and scales that are only 4-byte aligned (shift)."""
    print(f"[rows] batch={batch} hkv={hkv} group={group} cap={cap} step={step}", flush=True)
    rng = np.random.default_rng([6, batch, cap])
    kc, kn = _records(rng, (batch, hkv, cap), 3)
    vc, vn = _records(rng, (batch, hkv, cap), 3)
    seq = [(cap - step, 0, cap // 2, cap - step, 1 % cap)[i % 5] if i < 5 else (31 * i) % cap
           for i in range(batch)]
    seq = [min(n, cap - step) for n in seq]
    quats = orot.make_quaternions(78, hkv)
    levels, thr = ocb.isoquant_codebook(128, 3)
    q = rng.standard_normal((batch, hkv * group, 128), dtype=np.float32)
    k_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32).astype(np.float16)
    v_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32).astype(np.float16)

    def scales(x):
        x = x.copy()
        for i, n in enumerate(seq):
            x[i, :, n:] = np.nan
        buf = torch.empty(x.size + shift, dtype=torch.float32, device=DEV)
        view = buf[shift:].view(x.shape)
        view.copy_(torch.from_numpy(x))
        return view

    lens = _dev(np.asarray(seq, np.int32))
    args = (_dev(kc), scales(kn), _dev(vc), scales(vn), lens, _dev(quats))
    ws = api.alloc_workspace(batch, hkv * group, hkv, cap, DEV)
    ws.fill_(0x44)
    if step:
        out = api.iq_decode_step(_dev(q), _dev(k_new), _dev(v_new), *args, workspace=ws)
    else:
        out = api.iq_decode_attention(_dev(q), *args, workspace=ws)
    torch.cuda.synchronize()
    if step:
        assert lens.cpu().tolist() == [n + 1 for n in seq]
        rots = orot.rotation_matrices(quats)
        pk, nk, *_ = ocz.compress_kv(k_new[:, :, None], rots, thr)
        pv, nv, *_ = ocz.compress_kv(v_new[:, :, None], rots, thr)
        for i, n in enumerate(seq):
            kc[i, :, n], kn[i, :, n] = pk[i, :, 0], nk[i, :, 0]
            vc[i, :, n], vn[i, :, n] = pv[i, :, 0], nv[i, :, 0]
        assert np.array_equal(args[0].cpu().numpy(), kc)   # nothing else was written
        assert np.array_equal(args[2].cpu().numpy(), vc)
    ref = oatt.decode_fused(q, kc, kn, vc, vn, [n + step for n in seq], quats, levels)
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got))
    err = row_rel_err(got, ref)
    print(f"[rows] max row rel err {err.max():.3e}", flush=True)
    assert err.max() <= RTOL


@pytest.mark.parametrize("hq,hkv,shared,kind", [(16, 16, True, "edges"), (16, 2, False, "edges"),
                                                (8, 8, True, "one"), (16, 16, True, "runs"),
                                                (16, 2, False, "runs"), (8, 8, True, "splits")])
def test_positional_split(hq, hkv, shared, kind):
    cap = 1040
    batch = -(-16384 // (hkv * (cap // 16)))   # the shortest line that takes the kernel
    if kind in ("runs", "splits"):   # the shortest line of equal runs, or the longest of splits
        seq = _line_of(np.random.default_rng(11), batch, 256 * 8 * _short_batches(False) // hkv -
                       (kind == "splits"), cap, False)
    else:
        seq = [min(n, cap) for n in _lengths(kind, batch, cap)]
    print(f"[span rope] hq={hq} hkv={hkv} shared={shared} {kind} batch={batch}", flush=True)
    rng = np.random.default_rng([7, hq, hkv])
    kc, kn = _records(rng, (batch, hkv, cap), 3)
    vc, vn = _records(rng, (batch, hkv, cap), 3)
    kr = rng.standard_normal((batch, 1 if shared else hkv, cap, 64), dtype=np.float32).astype(
        np.float16)
    quats = orot.make_quaternions(79, hkv)
    levels, _ = ocb.isoquant_codebook(128, 3)
    q = rng.standard_normal((batch, hq, 128), dtype=np.float32)
    qr = rng.standard_normal((batch, hq, 64), dtype=np.float32)
    gkn, gvn, gkr = kn.copy(), vn.copy(), kr.copy()
    for i, n in enumerate(seq):
        gkn[i, :, n:] = np.nan
        gvn[i, :, n:] = np.nan
        gkr[i, :, n:] = np.nan
    ws = api.alloc_workspace(batch, hq, hkv, cap, DEV)
    ws.fill_(0x44)
    out = api.iq_decode_attention_rope(_dev(q), _dev(qr), _dev(kc), _dev(gkn), _dev(gkr), _dev(vc),
                                       _dev(gvn), _dev(np.asarray(seq, np.int32)), _dev(quats),
                                       workspace=ws)
    torch.cuda.synchronize()
    ref = oatt.decode_fused_rope(q, qr, kc, kn, kr, vc, vn, seq, quats, levels)
    got = out.cpu().numpy()
    assert np.all(np.isfinite(got))
    err = row_rel_err(got, ref)
    print(f"[span rope] max row rel err {err.max():.3e}", flush=True)
    assert err.max() <= RTOL


def _decode(q, kc, kn, vc, vn, seq, quats):
    out = api.iq_decode_attention(_dev(q), _dev(kc), _dev(kn), _dev(vc), _dev(vn),
                                  _dev(np.asarray(seq, np.int32)), _dev(quats))
    torch.cuda.synchronize()
    return out.cpu().numpy().astype(np.float64)


def test_weights_are_not_cut():
    """One attended position (weight 1) in each of 512 sequences: over random value scales, the
    output over the scale is the output of scale 1.  Pairs of fp16 values to nearest are off by at
    most 2^-23, 2^-24 rms and 0 in the mean, so the mean of 512 is within 4 * 2^-24 / sqrt(512) =
    1.1e-8 (the roundings of the outputs themselves average out over 512 x 128); pairs that are cut
    are off by -7e-8 in the mean."""
    batch, group, cap = 512, 8, 3
    rng = np.random.default_rng(12)
    kc = rng.integers(0, 256, size=(batch, 1, cap, 48), dtype=np.uint8)
    vc = rng.integers(0, 256, size=(batch, 1, cap, 48), dtype=np.uint8)
    kn = np.ones((batch, 1, cap), np.float32)
    vn = rng.uniform(1.0, 2.0, size=(batch, 1, cap)).astype(np.float32)
    quats = orot.make_quaternions(82, 1)
    q = rng.standard_normal((batch, group, 128), dtype=np.float32)
    one = _decode(q, kc, kn, vc, kn, [1] * batch, quats)
    got = _decode(q, kc, kn, vc, vn, [1] * batch, quats) / vn[:, :, :1].astype(np.float64)
    shift = (got * one).sum() / (one * one).sum() - 1.0
    print(f"[weights] shift {shift:.2e}", flush=True)
    assert abs(shift) <= 2e-8


@pytest.mark.parametrize("ratio", [1e3, 1e5])
def test_outlier_among_the_value_scales(ratio):
    """A value scale far above the others at a position of negligible weight: weights times scales
    are kept to 2^-39 of the largest scale of a wave's stretch (2^-25 in units of which the largest
    is 2^14 to 2^15), so that n positions of levels below 0.19 and a rotation (norm 1) are off by
    at most n 2^-39 0.19 sqrt(128) of that scale, beside the usual relative error."""
    cap, n, group = 1031, 1030, 8
    rng = np.random.default_rng(13)
    kc = rng.integers(0, 256, size=(1, 1, cap, 48), dtype=np.uint8)
    vc = rng.integers(0, 256, size=(1, 1, cap, 48), dtype=np.uint8)
    kn = np.full((1, 1, cap), 14.0, np.float32)
    vn = np.full((1, 1, cap), 14.0, np.float32)
    quats = orot.make_quaternions(83, 1)
    levels, _ = ocb.isoquant_codebook(128, 3)
    rot = orot.rotation_matrices(quats)[0]
    # queries against position 5's key: its score is the lowest by far
    key = levels[ocz.unpack(kc[0, 0, 5][None], 128, 3)[0]] @ rot
    q = (rng.standard_normal((1, group, 128)) - 40.0 * key / np.linalg.norm(key)).astype(np.float32)
    vn[0, 0, 5] *= ratio
    got = _decode(q, kc, kn, vc, vn, [n], quats)
    ref = oatt.decode_fused(q, kc, kn, vc, vn, [n], quats, levels)
    bound = RTOL * np.abs(ref).max(-1) + n * 2.0 ** -39 * 0.19 * 128 ** 0.5 * 14.0 * ratio
    err = np.abs(got - ref).max(-1)
    print(f"[outlier {ratio:g}] {err.max():.3e} bound {bound.min():.3e} out {np.abs(ref).max():.3e}")
    assert np.all(err <= bound)
