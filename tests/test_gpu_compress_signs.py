"""Edges of the bulk quantizer, which reads codes off the signs of y and |y| -
T_k: every bit position of a record (identity rotation, unit vectors with ties
on zero), values around each threshold, both zeros, blocks of zeros, fp32 inputs
near the top and the bottom of the range."""

import numpy as np
import pytest
import torch

from oracle import codebook as ocb
from oracle import compress as ocz
from oracle import rotation as orot
from paper_2608_08081_amd import api
from tests.parity import check_codes

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda:0")


def _vectors(rng, dtype):
    """[n][128]: rows whose rotated coordinates cover signs, zeros and thresholds."""
    had = np.array([[1.0]])
    for _ in range(7):
        had = np.block([[had, had], [had, -had]])
    rows = [np.eye(128)[i] * s for i in range(128) for s in (1.0, -1.0)]
    rows += [had[i] * s for i in range(128) for s in (1.0, -1.0)]       # one coordinate left
    rows += [had[i] + had[j] for i, j in rng.integers(0, 128, (64, 2))]  # most coordinates zero
    rows += list(rng.standard_normal((256, 128)))
    rows += [np.zeros(128), -np.zeros(128)]
    x = np.array(rows)
    if dtype == np.float32:
        x = np.concatenate((x, x * 2.0 ** 110, x * 2.0 ** -110, x[:256] * 2.0 ** 120))
    return x.astype(dtype)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
@pytest.mark.parametrize("identity", [True, False])
def test_codes_at_the_edges(bits, dtype, identity):
    x = _vectors(np.random.default_rng(bits), dtype)[None, None]
    quats = orot.make_quaternions(5, 1)
    if identity:
        quats = np.zeros_like(quats)
        quats[..., 0] = 1.0
    _, thr = ocb.isoquant_codebook(128, bits)
    _, _, codes, y, _ = ocz.compress_kv(x.astype(np.float64), orot.rotation_matrices(quats), thr)
    c = api.alloc_cache(1, 1, x.shape[2], DEV, bits=bits)
    xd = torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    api.iq_compress_kv_bits(xd, xd, torch.from_numpy(quats).to(DEV), c["k_codes"], c["k_norms"],
                            c["v_codes"], c["v_norms"], bits=bits)
    torch.cuda.synchronize()
    got = c["k_codes"].cpu().numpy()
    assert np.array_equal(got, c["v_codes"].cpu().numpy())
    # a coordinate that is exactly zero in the kernel's sums may be +-1e-17 in
    # the oracle's products: both round to the levels beside zero
    g = ocz.unpack(got, 128, bits)
    near = np.abs(y) < 1e-6
    assert np.all(np.isin(g[near], (2 ** (bits - 1) - 1, 2 ** (bits - 1))))
    if identity:   # sums of signs, without rounding: zero takes the upper level
        exact = near & (np.abs(x).max(-1, keepdims=True) > 0)
        had_rows = slice(0, 512)
        assert np.all(g[0, 0, had_rows][exact[0, 0, had_rows]] == 2 ** (bits - 1))
    keep = ~near.any(-1)
    check_codes(got[keep][None, None], codes[keep][None, None], y[keep][None, None], thr,
                f"signs b={bits}")
    far = ~near
    assert np.all((g == codes)[far] | (np.abs(np.abs(y[far])[:, None] - np.abs(thr)).min(-1) < 1e-6))


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("exponent", [60, 100, 123])
def test_small_entries_decide_where_large_ones_cancel(bits, exponent):
    """x0 = x1 = 2^e and x2 = -1e-30, identity blocks: coordinates whose signs of x0 and x1 differ
    are +-x2 exactly, so their codes are the levels beside zero on x2's side."""
    x = np.zeros((1, 1, 128, 128), np.float32)
    x[..., 0] = x[..., 1] = 2.0 ** exponent
    x[..., 2] = -1e-30
    quats = np.zeros((1, 32, 2, 4), np.float32)
    quats[..., 0] = 1.0
    c = api.alloc_cache(1, 1, 128, DEV, bits=bits)
    xd = torch.from_numpy(x).to(DEV)
    api.iq_compress_kv_bits(xd, xd, torch.from_numpy(quats).to(DEV), c["k_codes"], c["k_norms"],
                            c["v_codes"], c["v_norms"], bits=bits)
    torch.cuda.synchronize()
    had = orot.hadamard(128)
    cancel = had[:, 0] * had[:, 1] < 0
    want = 2 ** (bits - 1) - (had[cancel, 2] > 0)
    got = ocz.unpack(c["k_codes"].cpu().numpy(), 128, bits)[0, 0]
    assert np.array_equal(got[:, cancel], np.broadcast_to(want, got[:, cancel].shape))
