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


def _check(rng, seq, bits, group, page, step, hkv, cap, most=None, unmapped=()):
    """One decode or fused step of sequences of these lengths against the oracle: outputs, lengths,
    the capacity flag, and every byte of the cache.  Positions from `most` on are not attended; the
    page of the new token is not mapped for the sequences `unmapped`."""
    batch = len(seq)
    kc, kn = _records(rng, (batch, hkv, cap), bits)
    vc, vn = _records(rng, (batch, hkv, cap), bits)
    quats = orot.make_quaternions(77, hkv)
    levels, thr = ocb.isoquant_codebook(128, bits)
    q = rng.standard_normal((batch, hkv * group, 128), dtype=np.float32)
    k_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32)
    v_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32)
    room = [step and n < cap and i not in unmapped for i, n in enumerate(seq)]
    for i, n in enumerate(seq):   # a read of a position that is not attended shows up
        end = n if most is None else min(n, most)
        kn[i, :, end:] = np.nan
        vn[i, :, end:] = np.nan
    lens = _dev(np.asarray(seq, np.int32))
    flag = torch.zeros(1, dtype=torch.int32, device=DEV)
    ws = api.alloc_workspace(batch, hkv * group, hkv, most or cap, DEV)
    ws.fill_(0x44)
    host = {"k_codes": kc, "k_norms": kn, "v_codes": vc, "v_norms": vn}
    if page:
        per = cap // page
        assert per * page == cap
        table = rng.permutation(batch * per).astype(np.int32).reshape(batch, per)

        def pool_of(x):
            y = np.empty((batch * per, hkv, page, *x.shape[3:]), x.dtype)
            y[table.reshape(-1)] = np.moveaxis(x.reshape(batch, hkv, per, page, *x.shape[3:]), 2,
                                               1).reshape(y.shape)
            return y

        cache = {nm: _dev(pool_of(x)) for nm, x in host.items()}
        mapped = table.copy()
        for i in unmapped:
            assert seq[i] % page == 0
            mapped[i, seq[i] // page:] = (-1, 1 << 30)[i % 2]
        tab = _dev(mapped)
    else:
        cache = {nm: _dev(x) for nm, x in host.items()}
    args = (*cache.values(), lens, _dev(quats))
    kw = dict(workspace=ws, max_seq_len=most)
    if step and page:
        out = api.iq_decode_step_paged(_dev(q), _dev(k_new), _dev(v_new), cache, tab, lens,
                                       _dev(quats), status=flag, **kw)
    elif step:
        out = api.iq_decode_step_bits(_dev(q), _dev(k_new), _dev(v_new), *args, status=flag,
                                      bits=bits, **kw)
    elif page:
        out = api.iq_decode_attention_paged(_dev(q), cache, tab, lens, _dev(quats), **kw)
    else:
        out = api.iq_decode_attention_bits(_dev(q), *args, bits=bits, **kw)
    torch.cuda.synchronize()
    assert lens.cpu().tolist() == [n + r for n, r in zip(seq, room)]
    assert int(flag) == (5 if step and not all(room) else 0)   # IQ_ERR_CAPACITY
    if step:
        rots = orot.rotation_matrices(quats)
        pk, nk, *_ = ocz.compress_kv(k_new[:, :, None], rots, thr)
        pv, nv, *_ = ocz.compress_kv(v_new[:, :, None], rots, thr)
        for i, n in enumerate(seq):
            if room[i]:
                kc[i, :, n], kn[i, :, n] = pk[i, :, 0], nk[i, :, 0]
                vc[i, :, n], vn[i, :, n] = pv[i, :, 0], nv[i, :, 0]
    for nm, x in host.items():   # the new records, and nothing else
        got = cache[nm].cpu().numpy()
        assert np.array_equal(got, pool_of(x) if page else x, equal_nan=nm.endswith("norms")), nm
    end = [min(n + r, most or cap) for n, r in zip(seq, room)]
    ref = oatt.decode_fused(q, kc, np.nan_to_num(kn), vc, np.nan_to_num(vn), end, quats, levels)
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
    hkv, cap = 2, 2112   # (33 pages of 64)
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
        for got, want in ((args[1], kn), (args[3], vn)):
            x = want.copy()
            for i, n in enumerate(seq):
                x[i, :, n + 1:] = np.nan
            assert np.array_equal(got.cpu().numpy(), x, equal_nan=True)
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


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("mode", ["runs", "splits"])
def test_sequences_without_room(page, mode):
    """Among others: sequences at capacity (paged: also with an unmapped page for the new token)
    are attended as they are, keep their length and raise the flag."""
    hkv, cap = 2, 2112
    batch = -(-49152 // (hkv * (cap // 16)))
    rng = np.random.default_rng([14, page])
    seq = [cap - 1 - (37 * i) % 300 if mode == "runs" else (61 * i) % 700 for i in range(batch)]
    for i in (0, 5, batch - 1):
        seq[i] = cap
    unmapped = ()
    if page:
        unmapped = (2, 3, 40)
        for i in unmapped:
            seq[i] = seq[i] // page * page
    _check(rng, seq, 3, 8, page, True, hkv, cap, unmapped=unmapped)


@pytest.mark.parametrize("page,step,most", [(0, True, 1500), (0, False, 1500), (64, True, 1472)])
def test_lengths_beyond_max_seq_len(page, step, most):
    """Lengths at and past max_seq_len: the positions before it, the new token only if it lies
    before it too (it is appended all the same)."""
    hkv, cap = 2, 2112
    batch = -(-49152 // (hkv * (most // 16)))
    rng = np.random.default_rng([15, page, step])
    seq = [(most - 1, most, most + 1, cap - 1, 17, most - 16)[i] if i < 6 else
           int(rng.integers(most - 200, cap - 1)) for i in range(batch)]
    _check(rng, seq, 3, 8, page, step, hkv, cap, most=most)


def test_page_entries_of_long_runs():
    """Runs of more than 512 batches, whose waves read their page entries in pieces of 64 batches:
    the same bits as on rows."""
    batch, hkv, group, page, n = 2, 8, 2, 32, 270000
    cap = -(-n // page) * page
    g = torch.Generator(device=DEV).manual_seed(16)
    per = cap // page
    order = torch.randperm(batch * per, generator=g, device=DEV).view(batch, per)
    rows, pool = [], {}
    for side in ("k", "v"):
        codes = torch.randint(0, 256, (batch, hkv, cap, 48), generator=g, device=DEV,
                              dtype=torch.uint8)
        norms = 14.0 * torch.exp(0.35 * torch.randn((batch, hkv, cap), generator=g, device=DEV))
        for name, x in (("codes", codes), ("norms", norms)):
            y = x.view(batch, hkv, per, page, *x.shape[3:]).transpose(1, 2).flatten(0, 1)
            pool[f"{side}_{name}"] = torch.empty_like(y)
            pool[f"{side}_{name}"][order.view(-1)] = y
            rows.append(x)
    q = torch.randn((batch, hkv * group, 128), generator=g, device=DEV)
    lens = torch.tensor([n, n - 12345], dtype=torch.int32, device=DEV)
    quats = api.iq_make_rotation(17, hkv).to(DEV)
    want = api.iq_decode_attention(q, *rows, lens, quats)
    got = api.iq_decode_attention_paged(q, pool, order.int(), lens, quats)
    torch.cuda.synchronize()
    assert torch.isfinite(want).all() and want.abs().min(-1).values.max() > 0
    assert torch.equal(got, want)


@pytest.mark.parametrize("step", [False, True])
def test_more_sequences_than_the_line_holds(step):
    """513 sequences of split rows of odd capacity: the vector-unit path."""
    hkv, cap, batch = 1, 1001, 513
    rng = np.random.default_rng([18, step])
    seq = [(cap - 1, 0, 1, 512, 513)[i] if i < 5 else int(rng.integers(0, cap)) for i in
           range(batch)]
    if step:
        seq[6] = cap   # no room
    _check(rng, seq, 3, 8, 0, step, hkv, cap)


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


@pytest.mark.parametrize("page", [0, 16])
def test_captured_step_follows_the_lengths(page):
    """One captured step replayed on short lines (fixed splits) and long ones (equal runs) in turn,
    with the program's own work between: every replay as the eager call on the same cache."""
    hkv, group, cap = 2, 8, 2112
    batch = -(-49152 // (hkv * (cap // 16)))
    g = torch.Generator(device=DEV).manual_seed(19)
    shape = (batch * cap // page, hkv, page) if page else (batch, hkv, cap)
    cache = {}
    for side in ("k", "v"):
        cache[f"{side}_codes"] = torch.randint(0, 256, (*shape, 48), generator=g, device=DEV,
                                               dtype=torch.uint8)
        cache[f"{side}_norms"] = 14.0 * torch.exp(0.35 * torch.randn(shape, generator=g, device=DEV))
    tab = torch.randperm(batch * cap // (page or cap), generator=g, device=DEV).int().view(batch, -1)
    q = torch.randn((batch, hkv * group, 128), generator=g, device=DEV)
    k, v = (torch.randn((batch, hkv, 128), generator=g, device=DEV) for _ in range(2))
    quats = api.iq_make_rotation(20, hkv).to(DEV)
    lens = torch.zeros(batch, dtype=torch.int32, device=DEV)
    ws = api.alloc_workspace(batch, hkv * group, hkv, cap, DEV)
    out, ws2 = torch.empty_like(q), torch.empty_like(ws)

    def step(lens, out, ws):
        if page:
            api.iq_decode_step_paged(q, k, v, cache, tab, lens, quats, out=out, workspace=ws)
        else:
            api.iq_decode_step(q, k, v, *cache.values(), lens, quats, out=out, workspace=ws)

    sizes = [torch.randint(lo, hi, (batch,), generator=g, device=DEV).int()
             for lo, hi in ((0, 300), (1700, cap - 1), (500, 900), (1500, cap - 1), (0, 40))]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(lens, out, ws)
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(lens, out, ws)
    for n in sizes:
        want, eager = torch.empty_like(q), n.clone()
        lens.copy_(n)
        out.zero_()
        graph.replay()
        step(eager, want, ws2)   # (appends the same token at the same place again)
        torch.cuda.synchronize()
        assert torch.equal(out, want) and torch.isfinite(out).all() and out.abs().max() > 0
        assert torch.equal(lens, n + 1) and torch.equal(lens, eager)
