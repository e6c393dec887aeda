"""GPU parity with fitted codebooks (Sec. 3.2 Step 3 on calibration data):
iq_fit_codebook's levels drive compression (iq_compress_kv_cb), decode
(iq_decode_attention_cb, groups of 8 and of 4 query heads), the
fused step (iq_decode_step_cb) and materialization (iq_dequantize_kv_cb),
each against the oracle run with the oracle's own fitted codebook (equal to
the library's bit for bit, pinned on the CPU)."""

import numpy as np
import pytest
import torch

from oracle import attention as oatt
from oracle import codebook as ocb
from oracle import compress as ocz
from oracle import rotation as orot
from paper_2608_08081_amd import api, synth
from tests.parity import check_attention, check_codes, check_norms

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(DEV)


def _fitted(w, quats, bits, seed):
    """Calibration keys of the workload's distribution (a different seed from
    the cache), the library's fitted codebook and the oracle's."""
    cal = synth.kv_tensor(seed + 1000, w, "k", n_tokens=2048, batch=1)[0].astype(np.float32)
    cb = api.iq_fit_codebook(cal, quats, bits)
    rots = orot.rotation_matrices(quats)
    y = np.concatenate([ocb.rotated_coordinates(cal[h], rots[h]) for h in range(w.n_kv_heads)])
    levels, thr, _ = ocb.empirical_isoquant_codebook(y, bits)
    lv, th = api.codebook_arrays(cb)
    assert np.array_equal(lv.astype(np.float64), levels)
    assert np.array_equal(th.astype(np.float64), thr)
    return cb, levels, thr


@pytest.mark.parametrize("bits,hq,hkv,seq", [
    (3, 16, 2, [1000, 17, 0]),        # group 8: matrix-core path
    (3, 8, 2, [700, 333]),            # group 4
    (2, 16, 2, [512, 31]),
    (4, 32, 4, [1500]),
])
def test_fitted_codebook_compress_and_decode(bits, hq, hkv, seq):
    seed = 30 + bits
    cap = (max(max(seq), 1) + 15) // 16 * 16 + 16
    w = synth.Workload(93, "cbgpu", len(seq), hq, hkv, cap, "f16", kv_dist="heavy_tailed",
                       rotation_seed=77)
    quats = orot.make_quaternions(w.rotation_seed, hkv)
    cb, levels, thr = _fitted(w, quats, bits, seed)
    k = synth.kv_tensor(seed, w, "k", n_tokens=cap)
    v = synth.kv_tensor(seed, w, "v", n_tokens=cap)
    qt = _dev(quats)
    cache = api.alloc_cache(len(seq), hkv, cap, DEV, bits=bits)
    print(f"[codebook] b={bits} hq={hq} hkv={hkv} seq={seq}", flush=True)
    api.iq_compress_kv_cb(_dev(k), _dev(v), qt, cb, cache["k_codes"], cache["k_norms"],
                          cache["v_codes"], cache["v_norms"])
    cache["seq_lens"].copy_(torch.tensor(seq, dtype=torch.int32))
    q = synth.queries(seed, w)[0]
    out = api.iq_decode_attention_cb(_dev(q), cache["k_codes"], cache["k_norms"],
                                     cache["v_codes"], cache["v_norms"], cache["seq_lens"], qt,
                                     cb, max_seq_len=cap)
    torch.cuda.synchronize()
    rots = orot.rotation_matrices(quats)
    kp, kn, kc, ky, ks = ocz.compress_kv(k, rots, thr)
    vp, vn, vc, vy, vs = ocz.compress_kv(v, rots, thr)
    check_codes(cache["k_codes"].cpu().numpy(), kc, ky, thr, f"k b{bits}")
    check_codes(cache["v_codes"].cpu().numpy(), vc, vy, thr, f"v b{bits}")
    check_norms(cache["k_norms"].cpu().numpy(), ks, "k scale")
    # the oracle's attention on the oracle's records with the fitted levels
    ref = oatt.decode_fused(q, kp, kn, vp, vn, seq, quats, levels)
    check_attention(out.cpu().numpy(), ref, f"decode b{bits}")
    # the library's codebook gives a different answer on these records
    if bits == 3:
        plain = api.iq_decode_attention(_dev(q), cache["k_codes"], cache["k_norms"],
                                        cache["v_codes"], cache["v_norms"], cache["seq_lens"],
                                        qt, max_seq_len=cap).cpu().numpy()
        assert not np.allclose(plain, out.cpu().numpy(), rtol=1e-3, atol=1e-4)


@pytest.mark.parametrize("hq,hkv,seq0,cap", [(32, 4, [2999, 7], 3008), (8, 2, [300], 320)])
def test_fitted_codebook_fused_step(hq, hkv, seq0, cap):
    """Fused step with the fitted codebook: the new records and the
    attention over the advanced lengths, against the oracle; cache tails
    past the lengths poisoned."""
    seed = 50
    w = synth.Workload(94, "cbstep", len(seq0), hq, hkv, cap, "f16", rotation_seed=78)
    quats = orot.make_quaternions(w.rotation_seed, hkv)
    cb, levels, thr = _fitted(w, quats, 3, seed)
    k = synth.kv_tensor(seed, w, "k", n_tokens=cap)
    v = synth.kv_tensor(seed, w, "v", n_tokens=cap)
    rots = orot.rotation_matrices(quats)
    kp, kn, kc, ky, ks = ocz.compress_kv(k, rots, thr)
    vp, vn, vc, vy, vs = ocz.compress_kv(v, rots, thr)
    rng = np.random.default_rng(seed)
    gk, gv, gkn, gvn = kp.copy(), vp.copy(), kn.copy(), vn.copy()
    for i, n in enumerate(seq0):
        gk[i, :, n:] = rng.integers(0, 256, size=gk[i, :, n:].shape, dtype=np.uint8)
        gv[i, :, n:] = rng.integers(0, 256, size=gv[i, :, n:].shape, dtype=np.uint8)
        gkn[i, :, n:] = np.nan
        gvn[i, :, n:] = np.nan
    cache = dict(k_codes=_dev(gk), k_norms=_dev(gkn), v_codes=_dev(gv), v_norms=_dev(gvn),
                 seq_lens=_dev(np.asarray(seq0, np.int32)))
    k_new = np.stack([k[i, :, n] for i, n in enumerate(seq0)])
    v_new = np.stack([v[i, :, n] for i, n in enumerate(seq0)])
    q = synth.queries(seed, w)[0]
    out = api.iq_decode_step_cb(_dev(q), _dev(k_new), _dev(v_new), cache["k_codes"],
                                cache["k_norms"], cache["v_codes"], cache["v_norms"],
                                cache["seq_lens"], _dev(quats), cb, max_seq_len=cap)
    torch.cuda.synchronize()
    assert cache["seq_lens"].cpu().numpy().tolist() == [n + 1 for n in seq0]
    for i, n in enumerate(seq0):
        for side, c, y, s in (("k", kc, ky, ks), ("v", vc, vy, vs)):
            got = cache[f"{side}_codes"][i, :, n].cpu().numpy()
            check_codes(got[None, :, None], c[i:i + 1, :, n:n + 1], y[i:i + 1, :, n:n + 1], thr,
                        f"step new {side}")
            check_norms(cache[f"{side}_norms"][i, :, n].cpu().numpy(), s[i, :, n], "step scale")
    ref = oatt.decode_fused(q, kp, kn, vp, vn, [n + 1 for n in seq0], quats, levels)
    check_attention(out.cpu().numpy(), ref, f"step hq{hq}")


def test_fitted_codebook_dequantize():
    """Materialization with the fitted codebook: s R^T C_fit[code] against
    the oracle's reconstruction of the oracle's records."""
    seed = 60
    w = synth.Workload(95, "cbdeq", 1, 16, 2, 640, "f32", rotation_seed=79)
    quats = orot.make_quaternions(w.rotation_seed, 2)
    cb, levels, thr = _fitted(w, quats, 3, seed)
    k = synth.kv_tensor(seed, w, "k")
    rots = orot.rotation_matrices(quats)
    kp, kn, *_ = ocz.compress_kv(k, rots, thr)
    got, _ = api.iq_dequantize_kv_cb(_dev(kp), _dev(kn), None, None, _dev(quats), cb,
                                     out_dtype=torch.float32)
    torch.cuda.synchronize()
    want = ocz.reconstruct_kv(kp, kn, rots, levels)
    err = np.max(np.abs(got.cpu().numpy() - want)) / np.max(np.abs(want))
    assert err < 1e-5, err
