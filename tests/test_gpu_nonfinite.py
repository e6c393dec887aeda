"""Non-finite inputs of the span kernel: they stay visible in the rows that attend them and
nowhere else; a score of -inf has weight 0; an empty sequence gives zeros."""

import numpy as np
import pytest
import torch

from oracle import attention as oatt
from oracle import codebook as ocb
from oracle import compress as ocz
from oracle import rotation as orot
from paper_2608_08081_amd import api
from tests.parity import row_rel_err

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")
RTOL = 5e-5   # as in test_gpu_span.py


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


# (capacity, lengths): one span per row, whole rows by workgroup, rows over several runs
@pytest.mark.parametrize("cap,seq", [(17, [17, 3]), (1031, [1030, 515]), (3001, [2999, 70]),
                                     (103, [102, 33] * 200)])
@pytest.mark.parametrize("step", [False, True])
def test_non_finite_rows_of_any_length(cap, seq, step):
    batch, hkv, group = len(seq), 2, 4
    seq = [n - 1 for n in seq] + [0]   # the last sequence is empty
    batch += 1
    rng = np.random.default_rng([8, cap, step])
    kc = rng.integers(0, 256, size=(batch, hkv, cap, 48), dtype=np.uint8)
    vc = rng.integers(0, 256, size=(batch, hkv, cap, 48), dtype=np.uint8)
    kn = (14.0 * np.exp(0.35 * rng.standard_normal((batch, hkv, cap)))).astype(np.float32)
    vn = (14.0 * np.exp(0.35 * rng.standard_normal((batch, hkv, cap)))).astype(np.float32)
    quats = orot.make_quaternions(80, hkv)
    levels, thr = ocb.isoquant_codebook(128, 3)
    q = rng.standard_normal((batch, hkv * group, 128), dtype=np.float32)
    k_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32)
    v_new = rng.standard_normal((batch, hkv, 128), dtype=np.float32)
    ws = api.alloc_workspace(batch, hkv * group, hkv, cap, DEV)

    def run(q, kn, vn, k_new=k_new, v_new=v_new):
        ws.fill_(0x44)
        lens = _dev(np.asarray(seq, np.int32))
        args = (_dev(kc), _dev(kn), _dev(vc), _dev(vn), lens, _dev(quats))
        if step:
            out = api.iq_decode_step(_dev(q), _dev(k_new), _dev(v_new), *args, workspace=ws)
        else:
            out = api.iq_decode_attention(_dev(q), *args, workspace=ws)
        torch.cuda.synchronize()
        return out.cpu().numpy()

    fk, fkn, fv, fvn = kc.copy(), kn.copy(), vc.copy(), vn.copy()
    if step:
        rots = orot.rotation_matrices(quats)
        pk, nk, *_ = ocz.compress_kv(k_new[:, :, None], rots, thr)
        pv, nv, *_ = ocz.compress_kv(v_new[:, :, None], rots, thr)
        for i, n in enumerate(seq):
            fk[i, :, n], fkn[i, :, n] = pk[i, :, 0], nk[i, :, 0]
            fv[i, :, n], fvn[i, :, n] = pv[i, :, 0], nv[i, :, 0]
    ref = oatt.decode_fused(q, fk, fkn, fv, fvn, [n + step for n in seq], quats, levels)

    def check(got, bad):
        """bad [batch][heads]: the rows that attend something non-finite."""
        assert np.all(np.isnan(got[bad]).any(-1)), "a non-finite input left no trace"
        assert np.all(np.isfinite(got[~bad])), "rows without non-finite inputs changed"
        assert row_rel_err(got[~bad], ref[~bad]).max() <= RTOL

    none = np.zeros((batch, hkv * group), bool)
    attends = np.asarray(seq) + step > 0
    check(run(q, kn, vn), none)
    assert step or not run(q, kn, vn)[-1].any()   # the empty sequence
    # a query: its row only
    for value in (np.nan, np.inf):
        x, bad = q.copy(), none.copy()
        x[:, 1, 5] = value
        bad[:, 1] = attends
        check(run(x, kn, vn), bad)
    # one scale of KV head 1 at one attended position: its four query heads
    at = [min(n - 1, 40) for n in seq]
    for side, value in (("k", np.nan), ("v", np.nan), ("v", np.inf)):
        x = {"k": kn.copy(), "v": vn.copy()}
        bad = none.copy()
        for i, t in enumerate(at):
            if t >= 0:
                x[side][i, 1, t] = value
                bad[i, group:] = True
        check(run(q, x["k"], x["v"]), bad)
    # every key scale of a row
    x, bad = kn.copy(), none.copy()
    for i, n in enumerate(seq):
        x[i, 0, :n] = np.nan
        bad[i, :group] = n > 0
    check(run(q, x, vn), bad)
    if step:   # the new token's key or value (also of the sequence that was empty)
        bad = none.copy()
        bad[:, :group] = True
        for which in range(2):
            y = [k_new.copy(), v_new.copy()]
            y[which][:, 0, 3] = np.nan
            check(run(q, kn, vn, *y), bad)


def test_a_score_of_minus_infinity_has_weight_zero():
    """An infinite key scale makes its position's score +inf (NaN out) or -inf (weight 0) by the
    sign of the product, also where the position is the only one of its chunk or span."""
    cap, n, group = 1031, 1025, 8
    rng = np.random.default_rng(9)
    kc = rng.integers(0, 256, size=(1, 1, cap, 48), dtype=np.uint8)
    vc = rng.integers(0, 256, size=(1, 1, cap, 48), dtype=np.uint8)
    kn = np.full((1, 1, cap), 14.0, np.float32)
    vn = np.full((1, 1, cap), 14.0, np.float32)
    quats = orot.make_quaternions(81, 1)
    levels, _ = ocb.isoquant_codebook(128, 3)
    q = rng.standard_normal((1, group, 128), dtype=np.float32)
    rot = orot.rotation_matrices(quats)[0]
    for t in (0, 500, n - 1):
        x = kn.copy()
        x[0, 0, t] = np.inf
        out = api.iq_decode_attention(_dev(q), _dev(kc), _dev(x), _dev(vc), _dev(vn),
                                      _dev(np.asarray([n], np.int32)), _dev(quats))
        torch.cuda.synchronize()
        got = out.cpu().numpy()[0]
        dots = (q[0] @ rot.T) @ levels[ocz.unpack(kc[0, 0, t][None], 128, 3)[0]]
        assert np.abs(dots).min() > 1e-3
        x[0, 0, t] = 0.0
        keep = [i for i in range(n) if i != t]
        ref = oatt.decode_fused(q, kc[:, :, keep], kn[:, :, keep], vc[:, :, keep], vn[:, :, keep],
                                [n - 1], quats, levels)[0]
        assert np.all(np.isnan(got[dots > 0]).any(-1))
        assert row_rel_err(got[dots < 0], ref[dots < 0]).max() <= RTOL
